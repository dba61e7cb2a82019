"""The merge of a row's results over the column groups, up to and beyond the groups that a thread holds in registers (2048 of
128 columns), and the drafter's tokens that the same launch writes: against the device's own logits."""
import numpy as np
import pytest

import deer_inputs as di
from gpu_common import gpu_available
from oracle import deer_oracle as O

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("vocab", [128, 1152, 32768, 262144, 262400])   # 1, 9, 256, 2048 and 2050 groups
def test_tokens_and_acceptance(vocab):
    import torch
    from paper_2512_15176_amd import DeerEngine
    t, B, k, seed = di.ModelShape(1, 128, 4, 2, 32, 128, vocab, rope_base=1e4), 2, 5, 11
    eng = DeerEngine(t, t, B, 64, k, vocab - 1, keep_logits=True)
    for m in range(2):
        gen = torch.Generator(device="cuda").manual_seed(7 + m)
        w = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(0.1)   # noqa: E731
        for name, layer, r, c in (("embed", -1, vocab, 128), ("lm_head", -1, 128, vocab), ("wq", 0, 128, 128), ("wk", 0, 128, 64), ("wv", 0, 128, 64),
                                  ("wo", 0, 128, 128), ("wg", 0, 128, 128), ("wu", 0, 128, 128), ("wd", 0, 128, 128)):
            eng.load_tensor(m, name, layer, -1, w(r, c))
    for T in (0.0, 0.7):
        eng.prefill([di.prompt_ids(vocab, 20, seq=b) for b in range(B)])
        drafts = eng.draft_block(k, T, seed)
        zd = eng.debug_get_logits(1, k).astype(np.float64)
        got = drafts.cpu().numpy()
        eng.verify_block(k, T, drafts)
        zt = eng.debug_get_logits(0, k).astype(np.float64)
        accepted, committed = eng.accept_and_commit(k, T, seed)[:2]
        for b in range(B):
            rng = O.CounterRng(seed, b)
            a, slack = k, np.inf
            for i in range(k):
                p = zd[b, i] if T == 0.0 else zd[b, i] / T + rng._gumbel(O.TAG_DRAFT, 20 + i, vocab)
                top = np.partition(p, -2)[-2:]
                # 32-bit logarithms near 1 and sums of a dozen: 1e-4 of a Gumbel value of up to 17 at most
                assert got[b, i] == O.argmax_lowest(p) or (T > 0.0 and top[1] - top[0] < 2e-3), (T, b, i)
                if a < k:
                    continue
                if T == 0.0:
                    a = i if O.argmax_lowest(zt[b, i]) != got[b, i] else k
                else:
                    la = O.log_alpha(O.log_softmax(zt[b, i] / T)[got[b, i]], O.log_softmax(zd[b, i] / T)[got[b, i]])
                    lu = float(np.log(O.uniforms(O.row_key(seed, O.TAG_ACCEPT, b, 20 + i), 0)))
                    slack = min(slack, abs(lu - la) if la < 0 else np.inf)
                    a = k if lu <= la else i
            assert accepted[b] == a or slack < 1e-3, (T, b, accepted[b], a)
            assert [int(v) for v in committed[b][:a]] == got[b, :a].tolist() or slack < 1e-3
    eng.close()
