"""The LM head of passes of one and two row tiles over more than 32768 columns (columns streamed by one wave each): logits against 64 bits, no further off
than the weight-streaming kernel's, and the tokens drawn from them the same; vocabularies that leave half a workgroup without
columns, ragged numbers of rows, both ways to fold.  Its input is exact: a model whose layer adds nothing (zero output and down
projections) hands it the embedding rows themselves.  And (on the CPU) which passes take it."""
import os
import sys

import numpy as np
import pytest

import deer_inputs as di
from gpu_common import gpu_available

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub"))
from host_engine import run_script   # noqa: E402

# Mean over 64 rows of a row's relative error: its spread between two sets of weights is below 3 % (over 512 rows 1 %).
BOUND = 1.05


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("d,vocab", [(256, 33024), (896, 32896), (896, 49152), (1536, 33024), (1664, 32896), (4096, 49152)])
def test_logits_and_draws(d, vocab):
    import torch
    from paper_2512_15176_amd import DeerEngine, binding
    t = di.ModelShape(1, d, 4, 1, 64, 128, vocab, rope_base=1e4)
    gen = torch.Generator(device="cuda").manual_seed(d + vocab)
    w = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(0.02)   # noqa: E731
    zero = lambda *s: torch.zeros(*s, device="cuda", dtype=torch.bfloat16)   # noqa: E731
    embed, head = w(vocab, d), w(d, vocab)
    eng = DeerEngine(t, t, 3, 128, 32, vocab - 1, keep_logits=True)
    for m in (binding.DEER_TARGET, binding.DEER_DRAFTER):
        for name, layer, x in (("embed", -1, embed), ("lm_head", -1, head), ("wq", 0, w(d, 256)), ("wk", 0, w(d, 64)), ("wv", 0, w(d, 64)),
                               ("wo", 0, zero(256, d)), ("wg", 0, w(d, 128)), ("wu", 0, w(d, 128)), ("wd", 0, zero(128, d))):
            eng.load_tensor(m, name, layer, -1, x)
    for B, k in ((1, 1), (1, 32), (3, 13), (2, 31), (2, 32)):
        blocks = torch.randint(0, vocab, (B, k), generator=gen, device="cuda", dtype=torch.int32)
        last = [int(v) for v in np.random.default_rng(d + B).integers(0, vocab, B)]
        x = embed[torch.cat([torch.tensor(last, device="cuda")[:, None], blocks[:, :-1].long()], 1)].double()
        want = (x * torch.rsqrt(x.square().mean(-1, keepdim=True) + t.rms_eps)) @ head.double()
        err, out = {}, {}
        for T in (0.0, 0.8):
            for mode in (0, 128):   # streaming, the choice
                eng.debug_gemm_tiled(mode)
                eng.set_prefilled([40] * B, last)
                drafts = eng.draft_block(k, T, 5).clone()
                eng.verify_block(k, T, blocks)
                z = torch.from_numpy(eng.debug_get_logits(0, k)).cuda().double()
                rows = (z - want).norm(dim=-1) / want.norm(dim=-1)
                assert float(rows.max()) < 2e-6, (B, k, T, mode, float(rows.max()))   # a wrong fragment is off by more than 1e-2
                err[mode] = float(rows.mean())
                acc, committed = eng.accept_and_commit(k, T, 5)[:2]
                out[mode] = (drafts.cpu().tolist(), [int(v) for v in acc], [[int(v) for v in c] for c in committed])
            # the draws' margins: a difference of 1e-6 between two of them decides once in some 1e5 rows
            assert out[0] == out[128], (B, k, T)
        if B * k == 64:
            print(f"\n[d {d}, vocab {vocab}] streaming {err[0]:.3e}, here {err[128]:.3e}, ratio {err[128] / err[0]:.3f}")
            assert err[128] < BOUND * err[0]
    eng.close()


def test_which_passes_take_it(tmp_path):
    out = run_script(tmp_path, """
import deer_inputs as di
def engine(vocab):
    return HostEngine(di.ModelShape(1, 1664, 4, 2, 64, 256, vocab, rope_base=1e4), di.ModelShape(1, 256, 4, 2, 64, 256, vocab, rope_base=1e4), 3, 128)
e = engine(32896)
def heads(call):
    e.stub.stub_reset()
    assert call() == 0
    return [n.split("k_lm_head")[1][:17] for n, _ in e.launches() if "k_lm_head" in n]
for B, k, on in ((1, 1, 1), (1, 32, 1), (2, 16, 1), (2, 17, 2), (2, 32, 2), (3, 21, 2), (3, 22, 0)):
    assert e.set_prefilled([40] * B, [3] * B) == 0
    d, v = heads(lambda: e.draft_block(k)), heads(lambda: e.verify_block(k))
    assert d == ["ILi4ELi%dELi2ELb1E" % on] * (on > 0) and v == ["ILi4ELi%dELi2ELb0E" % on] * (on > 0), (B, k, d, v)
e.lib.deer_debug_gemm_tiled(e.ctx, 0)
assert e.set_prefilled([40], [3]) == 0 and heads(lambda: e.draft_block(8)) == []
for vocab in (1152, 32000, 32768):   # one round of the streaming kernel's workgroups
    e = engine(vocab)
    assert e.set_prefilled([40], [3]) == 0 and heads(lambda: e.draft_block(32)) == heads(lambda: e.verify_block(32)) == []
print("checked")
""")
    assert out == "checked\n"
