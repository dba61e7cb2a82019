"""The blocked GEMM is no further off a 64-bit result than the weight-streaming kernel, for short and long contractions.
Seen through the LM head of a model whose layer adds nothing (zero output and down projections): its input is then the
embedding row itself, exact in bf16, and the logits' error is the GEMM's own sum (and the row's RMSNorm factor)."""
import numpy as np
import pytest

import deer_inputs as di
from gpu_common import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# Mean over 512 rows of a row's relative error: its spread between two sets of weights is below 1 %.  Shorter chains than
# the streaming kernel's leave 0.8 to 0.96 of its error, one chain over K 1.8 to 2.8 times it, a plain fold of short
# contractions 1.07 to 1.3 times.
BOUND = 1.03


@pytest.mark.parametrize("d,vocab", [
    (256, 2048), (512, 4096),      # 16 and 32 k-steps
    (896, 2048), (896, 16384),     # 56; 64 and 512 workgroups
    (1536, 16384), (1664, 2048),   # 96 and 104: either side of the two ways to fold (and, with 64 workgroups, of the ring of 8)
    (2560, 16384),                 # 160
    (4096, 2048), (4096, 16384),   # 256
])
def test_sums_are_as_good_as_the_streaming_kernels(d, vocab):
    import torch
    from paper_2512_15176_amd import DeerEngine, binding
    t, B, k = di.ModelShape(1, d, 4, 1, 64, 128, vocab, rope_base=1e4), 16, 32
    gen = torch.Generator(device="cuda").manual_seed(d + vocab)
    w = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(0.02)   # noqa: E731
    zero = lambda *s: torch.zeros(*s, device="cuda", dtype=torch.bfloat16)   # noqa: E731
    embed, head = w(vocab, d), w(d, vocab)
    eng = DeerEngine(t, t, B, 128, k, vocab - 1, keep_logits=True)
    for m in (binding.DEER_TARGET, binding.DEER_DRAFTER):
        for name, layer, x in (("embed", -1, embed), ("lm_head", -1, head), ("wq", 0, w(d, 256)), ("wk", 0, w(d, 64)), ("wv", 0, w(d, 64)),
                               ("wo", 0, zero(256, d)), ("wg", 0, w(d, 128)), ("wu", 0, w(d, 128)), ("wd", 0, zero(128, d))):
            eng.load_tensor(m, name, layer, -1, x)
    blocks = torch.randint(0, vocab, (B, k), generator=gen, device="cuda", dtype=torch.int32)
    last = [int(v) for v in np.random.default_rng(d).integers(0, vocab, B)]
    x = embed[torch.cat([torch.tensor(last, device="cuda")[:, None], blocks[:, :-1].long()], 1)].double()
    want = (x * torch.rsqrt(x.square().mean(-1, keepdim=True) + t.rms_eps)) @ head.double()
    err = {}
    for mode in (0, 1):   # streaming, blocked
        eng.debug_gemm_tiled(mode)
        eng.set_prefilled([40] * B, last)
        eng.draft_block(k, 0.0, 0)
        eng.verify_block(k, 0.0, blocks)
        z = torch.from_numpy(eng.debug_get_logits(0, k)).cuda().double()
        err[mode] = float(((z - want).norm(dim=-1) / want.norm(dim=-1)).mean())
    eng.close()
    print(f"\n[d {d}, vocab {vocab}] streaming {err[0]:.3e}, blocked {err[1]:.3e}, ratio {err[1] / err[0]:.3f}")
    assert err[1] < BOUND * err[0]
