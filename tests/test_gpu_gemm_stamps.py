"""The clock stamps of streaming launches (deer_debug_gemm_stamps): every workgroup of the chosen launch leaves its own, in order,
also in the kernels that stream columns by one wave each (gate/up of two row tiles, in shares of K and not; LM heads)."""
import pytest

import deer_inputs as di
from gpu_common import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def stamps(eng, launch, B, torch):
    k = 32
    eng.debug_gemm_stamps(0, launch)
    eng.set_prefilled([40] * B, [3] * B)
    eng.draft_block(k, 0.0, 0)
    eng.verify_block(k, 0.0, torch.zeros(B, k, device="cuda", dtype=torch.int32))
    st = eng.debug_gemm_stamps(0, -1)
    st = st[: len(st) // 2]
    return st[st[:, 0] > 0].astype("int64")


def test_every_workgroup_leaves_its_stamps():
    import torch
    from paper_2512_15176_amd import DeerEngine
    small = di.ModelShape(1, 128, 4, 2, 32, 512, 40960, rope_base=1e4)
    for ff, shares in ((8192, 4), (20544, 3), (65536, 1)):
        t = di.ModelShape(1, 1664, 8, 2, 64, ff, 40960, rope_base=1e4)
        eng = DeerEngine(t, small, 2, 128, 32, t.vocab - 1)
        gen = torch.Generator(device="cuda").manual_seed(ff)
        for m, s in enumerate((t, small)):
            d, q, kv, f = s.d_model, s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim, s.d_ff
            for name, r, c in (("embed", s.vocab, d), ("lm_head", d, s.vocab), ("wq", d, q), ("wk", d, kv), ("wv", d, kv), ("wo", q, d), ("wg", d, f), ("wu", d, f), ("wd", f, d)):
                eng.load_tensor(m, name, -1 if name in ("embed", "lm_head") else 0, -1, torch.randn(r, c, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(0.02))
        st = stamps(eng, 2, 2, torch)   # gate/up
        assert len(st) == -(-2 * ff // 256) * shares, (ff, len(st))
        assert (st[:, 1] >= st[:, 0]).all() and (st[:, 2] >= st[:, 1]).all()
        if shares > 1:
            assert (st[:, 3] >= st[:, 2]).all() and (st[:, 4] > 0).sum() == -(-2 * ff // 256) and (st[st[:, 4] > 0, 4] >= st[st[:, 4] > 0, 3]).all()
        for B in (1, 2):
            st = stamps(eng, 4, B, torch)   # LM head
            assert len(st) == 160 and (st[:, 1] >= st[:, 0]).all() and (st[:, 2] >= st[:, 1]).all(), (ff, B, len(st))
        eng.close()
