"""GPU parity of the small-workgroup streaming GEMMs (one or two 32-column blocks per workgroup, K in up to eight shares),
which passes of one to four row tiles take by an estimate, against the wide streaming kernels: head dims 32, 64 and 128 (the
blocks of a rotation pair are neighbours or two apart), contractions that leave waves without k-steps, ragged last tiles;
and of passes of one row tile against the oracle.
test_host_routes.py checks that these shapes take them."""
import numpy as np
import pytest

import deer_inputs as di
from oracle import deer_oracle as O
from gpu_common import StoredWeights, fill_seeded_cache, gpu_available, make_engine, make_pair
from test_gpu_block_forms import _compare, _engine

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

SHAPES = {   # d, q heads, kv heads, head dim, d_ff
    "hd128": (1152, 9, 3, 128, 1216),    # 72, 72 and 76 k-steps
    "hd64": (2048, 16, 4, 64, 5632),     # 128, 64 and 352
    "hd32": (1280, 20, 4, 32, 1344),     # 80, 40 and 84
    "small": (384, 6, 3, 64, 2112),      # 24 and 132: one block per workgroup, beside the narrow QKV and O launches
}
BATCHES = [([70], 32), ([33], 5), ([40, 65, 8], 20), ([64, 31, 100], 31), ([50, 9, 128, 77], 32)]   # prefixes, k: 1, 1, 2, 3, 4 row tiles


@pytest.mark.parametrize("name", SHAPES)
def test_slim_launches_agree_with_the_wide_ones(name):
    import torch
    d, hq, hkv, hd, ff = SHAPES[name]
    t = di.ModelShape(2, d, hq, hkv, hd, ff, 1152, rope_base=1e4)
    eng = _engine(t, di.ModelShape(1, 384, 6, 3, 64, 2112, 1152, rope_base=1e4), 4, 256, torch)
    for x in eng._kv:   # stand-in keys and values everywhere: N(0, 1)
        v = x.view(torch.bfloat16)
        v.copy_(torch.randn(v.shape, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda", dtype=torch.bfloat16))
    for lens, k in BATCHES:
        blocks = torch.from_numpy(np.random.default_rng(k).integers(0, t.vocab, (2, len(lens), k)).astype(np.int32)).cuda()
        out = {}
        for mode in (0, 128):   # wide kernels, then the estimate's choice
            eng.debug_gemm_tiled(mode)
            eng.set_prefilled(lens, [5] * len(lens))
            res = []
            for block in blocks:   # the second iteration also takes in what the first committed
                eng.draft_block(k, 0.0, 0)
                zd = eng.debug_get_logits(1, k)
                eng.verify_block(k, 0.0, block)
                res += [zd, eng.debug_get_logits(0, k)]
                eng.debug_force_commit([[1, 2, 3]] * len(lens))
            out[mode] = ([x.view(torch.bfloat16).clone() for x in eng._kv], res)
        print(name, lens, k, flush=True)
        _compare(out[0], out[128])
    eng.close()


# Relative error of a row's logits.  One layer: activations enter as two bf16 planes (2^-17 = 7.6e-6 each time), four times
# that; a product without its second plane would be off by 2^-9 / sqrt(3) = 1e-3.  Two layers: one K or V value of a block's own
# rows that rounds the other way (2^-8 of it, one key of about 100) moves the rows above it by up to 1e-4 or so.
ORACLE = {1: 3e-5, 2: 3e-4}


@pytest.mark.parametrize("name", SHAPES)
@pytest.mark.parametrize("layers", [1, 2])
def test_slim_launches_against_the_oracle(name, layers):
    """One row tile, draft and verify, behind stand-in keys and values."""
    import torch
    d, hq, hkv, hd, ff = SHAPES[name]
    t, k, n = di.ModelShape(layers, d, hq, hkv, hd, ff, 1152, rope_base=1e4), 32, 70
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(t, di.DRAFTER_SEED, "bf16")
    eng = make_engine(t, t, wt, wd, 1, 192, k)
    block = [int(v) for v in np.random.default_rng(d).integers(0, t.vocab, k)]
    pair = make_pair(t, t, wt, wd, 192)
    pair.x = [0] * (n - 1) + [7]
    fill_seeded_cache(eng, torch, 0, t, 0, n - 1, pair.tc)
    fill_seeded_cache(eng, torch, 1, t, 0, n, pair.dc)
    eng.set_prefilled([n], [7])
    eng.draft_block(k, 0.0, 0)
    zd = pair.draft_logits(k)
    zt = O.deer_iteration(pair, k, 0.0, None, draft_override=block)["target_logits"]
    eng.verify_block(k, 0.0, torch.tensor([block], dtype=torch.int32, device="cuda"))
    for got, want in ((eng.debug_get_logits(1, k)[0], zd), (eng.debug_get_logits(0, k)[0], zt)):
        off = np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)
        print(f"[{name}, {layers} layers] rows off by {off.max():.2e}, mean {off.mean():.2e}")
        assert off.max() < ORACLE[layers], off.max()
    eng.close()
