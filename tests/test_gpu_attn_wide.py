"""GPU parity of the attention kernel of passes with many row tiles (two workgroups of four heads per compute unit, key
tiles in pairs): head sizes 32, 64 and 128, 1 to 8 query heads per kv head, odd and even numbers of key tiles, key
ranges split over workgroups or not, and short sequences beside long ones, against the oracle."""
import numpy as np
import pytest

import deer_inputs as di
from gpu_common import StoredWeights, gpu_available, make_engine, make_pair

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# (query heads, kv heads, head_dim, prompt lengths): the pass has more than 256 (row tile, query head) items
CASES = [
    (16, 2, 64, [520, 3, 33]),     # 8 heads per kv head: two workgroups; 17 key tiles, split ranges
    (14, 2, 64, [608]),            # 7: the second workgroup has an idle wave; 19 tiles
    (12, 12, 32, [736, 1]),        # 1: three idle waves; 23 tiles
    (6, 2, 128, [1377]),           # 3; 44 tiles (an even number) of which the last holds one key
    (32, 8, 128, [288, 65, 31]),   # 4, the 8B shape's heads: 9 + 3 + 1 tiles
]


@pytest.mark.parametrize("hq,hkv,hd,lens", CASES)
def test_wide_attention(hq, hkv, hd, lens):
    import torch
    t = di.ModelShape(2, 256, hq, hkv, hd, 512, 1024, rope_base=1e4)
    d, k = di.CONFIGS["tiny"]["drafter"], 8
    assert sum(-(-(n - 1) // 32) for n in lens) * hq > 256
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(d, di.DRAFTER_SEED, "bf16")
    eng = make_engine(t, d, wt, wd, len(lens), 1472, k)
    prompts = [di.prompt_ids(t.vocab, n, seq=40 + b) for b, n in enumerate(lens)]
    blocks = np.random.default_rng(3).integers(0, t.vocab, (len(lens), k)).astype(np.int32)
    eng.prefill(prompts)
    eng.draft_block(k, 0.0, 0)
    eng.verify_block(k, 0.0, torch.from_numpy(blocks).cuda())
    z = eng.debug_get_logits(0, k)
    for b, prompt in enumerate(prompts):
        pair = make_pair(t, d, wt, wd, 1472)
        pair.prefill(prompt)
        want = pair.verify_logits([int(v) for v in blocks[b]])
        assert np.abs(z[b] - want).max() < 2e-3, (b, np.abs(z[b] - want).max())   # the tiny shapes' bound elsewhere
    eng.close()


@pytest.mark.parametrize("k", [1, 5, 31, 32])
def test_blocks_of_fewer_rows_than_a_tile(k):
    """A batch's verify pass (9 tiles of 32 heads): tiles of which some rows do not exist, key ranges split over workgroups, of
    which the short sequences have none in the later ranges, beside ranges that end inside a tile."""
    import torch
    t = di.ModelShape(1, 256, 32, 8, 128, 512, 1024, rope_base=1e4)
    d, lens = di.CONFIGS["tiny"]["drafter"], [700, 3, 33, 64, 129, 1, 290, 511, 96]
    assert len(lens) * t.n_q_heads > 256
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(d, di.DRAFTER_SEED, "bf16")
    eng = make_engine(t, d, wt, wd, len(lens), 768, 32)
    eng._workspace.fill_(255)          # NaN patterns where no pass writes, in the memory that the next engine gets
    at = eng._workspace.data_ptr()
    eng.close()
    del eng
    eng = make_engine(t, d, wt, wd, len(lens), 768, 32)
    assert eng._workspace.data_ptr() == at
    prompts = [di.prompt_ids(t.vocab, n, seq=80 + b) for b, n in enumerate(lens)]
    blocks = np.random.default_rng(5).integers(0, t.vocab, (len(lens), k)).astype(np.int32)
    eng.prefill(prompts)
    eng.draft_block(k, 0.0, 0)
    eng.verify_block(k, 0.0, torch.from_numpy(blocks).cuda())
    z = eng.debug_get_logits(0, k)
    for b, prompt in enumerate(prompts):
        pair = make_pair(t, d, wt, wd, 768)
        pair.prefill(prompt)
        want = pair.verify_logits([int(v) for v in blocks[b]])
        assert np.abs(z[b] - want).max() < 2e-3, (b, np.abs(z[b] - want).max())
    eng.close()
