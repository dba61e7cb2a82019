"""GPU parity of the blocked GEMM (128-row workgroups, two per compute unit) where the default dispatch takes it: prompts
and batches of a few row tiles at real layer widths, where K is split over workgroups, the last row block is ragged
and the accumulators are folded, against the weight-streaming kernels on the same state."""
import numpy as np
import pytest

import deer_inputs as di
from gpu_common import StoredWeights, gpu_available, make_engine

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# Both kernels sum the same bf16 products in fp32, in different order, and what differs by more than that is a K or V value
# near the middle of two bf16 values that goes either way.  One such value (up to 4, off by 2^-8 of it) that is a row's
# only key moves the residual stream by 0.02 * 2^-6 = 3e-4 per channel of about 1.6, i.e. the row by 2e-4 of its norm (less
# with more keys); a hundred of them by 2e-3.  A wrong index or a missing k-step changes a row by more than 1e-2.
TOL = 2e-3


@pytest.fixture(scope="module")
def engine():
    t = di.scaled(di.CONFIGS["qwen3_8b"]["target"], n_layers=2, vocab=16384)
    d = di.scaled(di.DRAFTER_05B, n_layers=2, vocab=16384)      # d = 896: an odd number of column groups
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(d, di.DRAFTER_SEED, "bf16")
    eng = make_engine(t, d, wt, wd, 9, 1536, 32)
    yield eng, t
    eng.close()


def _pass(eng, prompts, k, T, blocks, torch):
    eng.prefill(prompts)
    eng.draft_block(k, T, 3)
    zd = eng.debug_get_logits(1, k)
    eng.verify_block(k, T, torch.from_numpy(blocks).cuda())
    zt = eng.debug_get_logits(0, k)
    eng.accept_and_commit(k, T, 3)
    return zd, zt


@pytest.mark.parametrize("lens,k", [
    ([97], 32),                                   # 4 row tiles (the target's 3 + 0 rows of the fourth)
    ([161, 33], 5),                               # 5 + 1 and 6 + 2 tiles: ragged row blocks
    ([225], 1),                                   # 7 and 8 tiles
    ([511], 17),                                  # 16 tiles: K split over workgroups for some matrices, whole for others
    ([40, 300, 77, 129, 65, 31, 2, 1, 200], 32),  # nine sequences: decode passes of 9 tiles, the LM head among them
    ([1200], 32),                                 # 38 tiles: more than one band of row blocks, 256-column workgroups
])
def test_blocked_and_streaming_kernels_agree(engine, lens, k):
    import torch
    eng, t = engine
    prompts = [di.prompt_ids(t.vocab, n, seq=b) for b, n in enumerate(lens)]
    blocks = np.random.default_rng(1).integers(0, t.vocab, (len(lens), k)).astype(np.int32)
    eng.debug_gemm_tiled(0)
    zd0, zt0 = _pass(eng, prompts, k, 0.0, blocks, torch)
    eng.debug_gemm_tiled(128)
    zd1, zt1 = _pass(eng, prompts, k, 0.0, blocks, torch)
    eng.debug_gemm_tiled(1)
    zd2, zt2 = _pass(eng, prompts, k, 0.0, blocks, torch)
    eng.debug_gemm_tiled(128)
    for a, b in ((zd0, zd1), (zt0, zt1), (zd0, zd2), (zt0, zt2)):
        off = np.linalg.norm(a - b, axis=-1) / np.linalg.norm(a, axis=-1)   # per row
        assert np.isfinite(b).all() and float(off.max()) < TOL, (lens, float(off.max()))


@pytest.mark.parametrize("lens", [[7], [65], [190, 3], [700, 33, 1]])
def test_grouped_gemms_of_a_mixture(lens):
    """Experts with fewer and more than 32 and 64 pairs, 384 = one and a half 256-column blocks, an expert width of three
    64-channel groups: gathered rows and blocked gate/up (from 14 pairs per expert on) against the streaming gate/up and
    the oracle."""
    import torch
    from gpu_common import make_pair
    t = di.ModelShape(2, 384, 6, 3, 64, 0, 1024, n_experts=12, top_k=3, d_ff_expert=192, rope_base=1e4)
    d, k = di.CONFIGS["tiny"]["drafter"], 8
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(d, di.DRAFTER_SEED, "bf16")
    eng = make_engine(t, d, wt, wd, len(lens), 1024, k)
    prompts = [di.prompt_ids(t.vocab, n, seq=20 + b) for b, n in enumerate(lens)]
    blocks = np.random.default_rng(2).integers(0, t.vocab, (len(lens), k)).astype(np.int32)
    got = []
    for mode in (0, 128):
        eng.debug_gemm_tiled(mode)
        got.append(_pass(eng, prompts, k, 0.0, blocks, torch)[1])
    for b, prompt in enumerate(prompts):
        pair = make_pair(t, d, wt, wd, 1024)
        pair.prefill(prompt)
        z = pair.verify_logits([int(v) for v in blocks[b]])
        for g in got:
            assert np.abs(g[b] - z).max() < 2e-3, (lens, b, np.abs(g[b] - z).max())   # the small mixture's bound in the lock-step test
    eng.close()
