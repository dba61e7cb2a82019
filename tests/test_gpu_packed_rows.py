"""GPU parity where a pass's GEMM rows are packed over the sequences: blocks that do not fill a row tile, sequences that
straddle tiles, committed tokens of unequal number that the drafter takes in (in the MASK rows' attention tile where they fit
for every sequence, else in one of their own), the bonus row, and one sequence without new tokens, against the oracle."""
import numpy as np
import pytest

import deer_inputs as di
from oracle import deer_oracle as O
from gpu_common import StoredWeights, gpu_available, lockstep_commit, make_engine, make_pair

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

TOL = 2e-3   # as for the tiny shapes elsewhere


@pytest.mark.parametrize("lens,k,bonus,wanted", [
    ([40, 7, 33], 20, 0, [[20, 0, 13], [11, 12, 19], [3, 0, 0]]),                 # commits of up to 20: an attention tile of their own, then one
    ([21, 64, 5, 1, 32, 9, 50], 9, 0, [[9, 0, 3, 1, 8, 2, 5], [0, 9, 9, 9, 0, 9, 1]]),   # 63 MASK rows, 28 and 40 committed tokens behind them
    ([31, 12, 60, 2, 17], 1, 0, [[1, 0, 1, 1, 0], [0, 1, 1, 0, 1]]),              # five rows in one tile
    ([30, 44], 15, 1, [[15, 4], [2, 15], [0, 0]]),                                # bonus: 16 rows per sequence, one full tile
    ([19, 70, 3], 31, 1, [[31, 30, 0], [0, 31, 1]]),                              # bonus: full tiles; 31 MASK rows leave room for one token
])
def test_packed_rows(lens, k, bonus, wanted):
    import torch
    t, d = di.CONFIGS["tiny"]["target"], di.CONFIGS["tiny"]["drafter"]
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(d, di.DRAFTER_SEED, "bf16")
    eng = make_engine(t, d, wt, wd, len(lens), 256, 32)
    prompts = [di.prompt_ids(t.vocab, n, seq=60 + b) for b, n in enumerate(lens)]
    pairs = [make_pair(t, d, wt, wd, 256) for _ in lens]
    for pair, prompt in zip(pairs, prompts):
        pair.prefill(prompt)
    eng.prefill(prompts)
    if bonus:
        eng.set_bonus_token(True)
    dec = O.Decoder(t, wt.as_f32, np.float64, "bf16")
    for a_want in wanted:
        eng.draft_block(k, 0.0, 0)
        gzd = eng.debug_get_logits(1, k)
        blocks, refs = [], []
        for b, pair in enumerate(pairs):
            block = list(O.ar_decode(dec, pair.prefix(), k))
            if a_want[b] < k:
                block[a_want[b]] = (block[a_want[b]] + 1) % t.vocab
            blocks.append(block)
            refs.append(O.deer_iteration(pair, k, 0.0, None, draft_override=block, bonus=bool(bonus)))
            assert np.abs(gzd[b] - refs[b]["draft_logits"]).max() < TOL, b
        eng.verify_block(k, 0.0, torch.tensor(blocks, dtype=torch.int32, device="cuda"))
        rows = k + bonus
        gzt = np.empty((len(lens), rows, t.vocab), dtype=np.float32)
        eng._check(eng.lib.deer_debug_get_logits(eng.ctx, 0, gzt.ctypes.data, gzt.size))
        for b in range(len(lens)):
            assert np.abs(gzt[b] - refs[b]["target_logits"]).max() < TOL, b
        lockstep_commit(eng, k, gzt, refs, blocks, bool(bonus))
        assert eng.get_lengths().tolist() == [len(p.prefix()) for p in pairs]
    eng.close()
