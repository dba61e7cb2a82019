"""The streaming GEMMs in small workgroups are no further off a 64-bit result than the wide ones, whose workgroups are fewer
and whose chains of sums are shorter.  Seen in the residual rows (fp32, in the workspace) behind one residual GEMM of a layer
whose other one adds nothing, with inputs that bf16 holds exactly: embeddings of +-1 (RMSNorm factors of 1); behind the O
projection blocks of one row over an empty cache (attention returns the row's own V); behind the down projection gates of 32
(their SiLU is 32) and one weight per up channel."""
import numpy as np
import pytest

import deer_inputs as di
from gpu_common import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# Error of all rows together, against that of the wide kernels.  A chain of n k-steps is off by about sqrt(n) of an addition's
# rounding, sums over 8 waves and S shares by sqrt(4 + S / 2): 24 k-steps and 4 shares against 12 and 8 make 1.17 (8B down)
# unless a wave's sums are cut; cut every 4 to 6 k-steps they make 0.8 to 1.0.  28672 values or more: 1 % of spread.
BOUND = 1.02


@pytest.mark.parametrize("which,d,heads,ff,rows", [
    ("down", 4096, 4, 12288, 32), ("down", 2560, 4, 9728, 32), ("down", 2048, 4, 5632, 64), ("down", 896, 4, 4864, 32),
    ("O", 4096, 32, 128, 32), ("O", 2560, 32, 128, 32), ("O", 4096, 32, 128, 64),
])
def test_sums_are_as_good_as_the_wide_kernels(which, d, heads, ff, rows):
    import torch
    from paper_2512_15176_amd import DeerEngine, binding
    hd, hkv, vocab = (64, 2, 1024) if d < 1024 else (128, heads // 4, 1024)
    t = di.ModelShape(1, d, heads, hkv, hd, ff, vocab, rope_base=1e4, rms_eps=0.0)
    small = di.ModelShape(1, 128, 4, 2, 32, 128, vocab, rope_base=1e4)
    gen = torch.Generator(device="cuda").manual_seed(d + rows)
    w = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(0.02)   # noqa: E731
    zero = lambda *s: torch.zeros(*s, device="cuda", dtype=torch.bfloat16)   # noqa: E731
    embed = torch.where(torch.rand(vocab, d, generator=gen, device="cuda") < 0.5, -1.0, 1.0).to(torch.bfloat16)
    embed[:, 0] = 1.0
    wg, wu = zero(d, ff), zero(d, ff)
    wg[0] = 32.0
    src = torch.randint(0, d, (ff,), generator=gen, device="cuda")
    wu[src, torch.arange(ff, device="cuda")] = torch.randn(ff, generator=gen, device="cuda").mul_(1 / 32).to(torch.bfloat16)
    wo, wd = (w(heads * hd, d) if which == "O" else zero(heads * hd, d)), (w(ff, d) if which == "down" else zero(ff, d))
    eng = DeerEngine(t, small, rows, 64, 1, vocab - 1, keep_logits=True)

    def load(model, s, tensors):
        for name, layer, x in tensors:
            eng.load_tensor(model, name, layer, -1, x)
    load(binding.DEER_TARGET, t, (("embed", -1, embed), ("lm_head", -1, w(d, vocab)), ("wq", 0, w(d, heads * hd)), ("wk", 0, w(d, hkv * hd)),
                                  ("wv", 0, w(d, hkv * hd)), ("wo", 0, zero(heads * hd, d)), ("wg", 0, wg), ("wu", 0, wu), ("wd", 0, zero(ff, d))))
    load(binding.DEER_DRAFTER, small, (("embed", -1, w(vocab, 128)), ("lm_head", -1, w(128, vocab)), ("wq", 0, w(128, 128)), ("wk", 0, w(128, 64)),
                                       ("wv", 0, w(128, 64)), ("wo", 0, w(128, 128)), ("wg", 0, w(128, 128)), ("wu", 0, w(128, 128)), ("wd", 0, w(128, 128))))
    last = [int(v) for v in np.random.default_rng(d).integers(0, vocab, rows)]
    x = embed[torch.tensor(last, device="cuda")]
    block = torch.zeros(rows, 1, device="cuda", dtype=torch.int32)

    def step():
        eng.set_prefilled([1] * rows, last)   # a block's row stands for the last token: it sees itself
        eng.draft_block(1, 0.0, 0)
        eng.verify_block(1, 0.0, block)
        torch.cuda.synchronize()
    step()   # both projections still add nothing: the residual rows are the embeddings
    words = eng._workspace[: eng._workspace.numel() // 4 * 4].view(torch.float32)
    n, first = words.numel() - rows * d, torch.ones(words.numel() - rows * d, device="cuda", dtype=torch.bool)
    for i in range(64):
        first &= words[i : i + n] == float(x[0, i])
    at = [i for i in first.nonzero().flatten().tolist() if torch.equal(words[i : i + rows * d].view(rows, d), x.float())]
    assert len(at) == 1, at
    h = words[at[0] : at[0] + rows * d].view(rows, d)
    load(binding.DEER_TARGET, t, (("wo", 0, wo), ("wd", 0, wd)))
    err = {}
    for mode in (0, 128):   # wide kernels, then the estimate's choice
        eng.debug_gemm_tiled(mode)
        step()
        if which == "O":
            lay = eng.get_kv_layout(binding.DEER_TARGET)   # V of slot 0: channel c of a head lies at 1024 (c / 32) + 8 (c % 32)
            c, v = torch.arange(hd, device="cuda"), eng._kv[0].view(torch.bfloat16)[lay.v_base :]
            v = v.as_strided((rows, hkv, lay.head_stride), (lay.seq_stride, lay.head_stride, 1))[..., c // 32 * 1024 + c % 32 * 8]
            y = v.double().repeat_interleave(heads // hkv, 1).reshape(rows, -1) @ wo.double()
        else:
            y = (32.0 * (x[:, src].double() * wu[src, torch.arange(ff, device="cuda")].double())) @ wd.double()
        err[mode] = float((h.double() - x.double() - y).norm() / y.norm())
    eng.close()
    print(f"\n[{which}, d {d}, ff {ff}, {rows} rows] wide {err[0]:.3e}, small {err[128]:.3e}, ratio {err[128] / err[0]:.3f}")
    assert err[0] < 1e-6 and err[128] < BOUND * err[0]
