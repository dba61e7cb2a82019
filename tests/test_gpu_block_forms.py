"""GPU parity of every form of the blocked GEMM (128- and 256-column workgroups, ring of 4 and 8 k-steps, K whole and in
shares, both ways to fold) in every dense GEMM of a pass, at ragged shapes, and of the 256-column form where the estimate
takes it, against the weight-streaming kernels: K,V rows of the prompts and logits of a block behind them."""
import numpy as np
import pytest

import deer_inputs as di
from gpu_common import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# Both kernels sum the same products in fp32.  What differs by more than rounding is a K or V value near the middle of two
# bf16 values: it is off by 2^-8 of itself, at most 2^-6 for the values up to 4 here, and moves later rows by less.  With
# every value off so the caches would differ by 2^-8 of their norm; a wrong fragment is off by the values' own size, about 1.
CACHE_REL, CACHE_MAX, LOGITS = 2e-3, 0.1, 2e-3


def _engine(t, d, batch, max_seq, torch):
    from paper_2512_15176_amd import DeerEngine
    eng = DeerEngine(t, d, batch, max_seq, 32, t.vocab - 1, keep_logits=True)
    gen = torch.Generator(device="cuda").manual_seed(11)
    w = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(0.02)   # noqa: E731
    for m, s in enumerate((t, d)):
        q, kv = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
        eng.load_tensor(m, "embed", -1, -1, w(s.vocab, s.d_model))
        eng.load_tensor(m, "lm_head", -1, -1, w(s.d_model, s.vocab))
        for layer in range(s.n_layers):
            for name, r, c in (("wq", s.d_model, q), ("wk", s.d_model, kv), ("wv", s.d_model, kv), ("wo", q, s.d_model),
                               ("wg", s.d_model, s.d_ff), ("wu", s.d_model, s.d_ff), ("wd", s.d_ff, s.d_model)):
                eng.load_tensor(m, name, layer, -1, w(r, c))
    return eng


def _outputs(eng, prompts, k, blocks, torch):
    """The caches after the prompts - behind these lie the block rows of the pass before - and the block's logits."""
    eng.prefill(prompts)
    kv = [x.view(torch.bfloat16).clone() for x in eng._kv]
    eng.draft_block(k, 0.0, 0)
    zd = eng.debug_get_logits(1, k)
    eng.verify_block(k, 0.0, blocks)
    zt = eng.debug_get_logits(0, k)
    eng.accept_and_commit(k, 0.0, 0)
    return kv, (zd, zt)


def _compare(want, got):
    for a, b in zip(want[0], got[0]):
        a, b = a.float(), b.float()
        off = (a - b).abs()
        assert float(off.norm() / a.norm()) < CACHE_REL and float(off.max()) < CACHE_MAX, (float(off.norm() / a.norm()), float(off.max()))
    for a, b in zip(want[1], got[1]):
        off = np.linalg.norm(a - b, axis=-1) / np.linalg.norm(a, axis=-1)
        assert np.isfinite(b).all() and float(off.max()) < LOGITS, float(off.max())


@pytest.mark.parametrize("shape", [
    # 24, 24 and 40 k-steps, 3, 6, 9 and 10 column groups (an odd number: half a 256-column block)
    dict(d_model=384, n_q_heads=6, n_kv_heads=3, d_ff=640, vocab=1152),
    # 176, 72 and 104 k-steps, 22, 15, 26 and 9 column groups
    dict(d_model=2816, n_q_heads=18, n_kv_heads=6, d_ff=1664, vocab=1152),
], ids=["short", "long"])
def test_every_form_agrees_with_the_streaming_kernels(shape):
    import torch
    t = di.ModelShape(2, shape["d_model"], shape["n_q_heads"], shape["n_kv_heads"], 64, shape["d_ff"], shape["vocab"], rope_base=1e4)
    d, k = di.ModelShape(1, 384, 6, 3, 64, 640, shape["vocab"], rope_base=1e4), 32
    lens = [290, 33, 1, 200]                          # 17 row tiles: a row block of one tile; 4 and more rows tiles of a block
    eng = _engine(t, d, len(lens), 384, torch)
    prompts = [di.prompt_ids(t.vocab, n, seq=b) for b, n in enumerate(lens)]
    blocks = torch.from_numpy(np.random.default_rng(1).integers(0, t.vocab, (len(lens), k)).astype(np.int32)).cuda()
    eng.debug_gemm_tiled(0)
    _outputs(eng, prompts, k, blocks, torch)
    want = _outputs(eng, prompts, k, blocks, torch)
    eng.debug_gemm_tiled(128)
    for form in ((2, 4, 1), (2, 4, 3), (2, 8, 1), (2, 8, 2), (4, 4, 1), (4, 4, 2), (4, 4, 5)):
        print("form", form, flush=True)
        eng.debug_gemm_block(*form)
        _compare(want, _outputs(eng, prompts, k, blocks, torch))
    eng.close()


@pytest.mark.parametrize("model,n", [("qwen3_8b", 2100), ("qwen3_4b", 3329)])
def test_wide_prompts_agree(model, n):
    """66 and 104 row tiles: the estimate takes the 256-column form for gate/up, the residual GEMMs and (8B) QKV, and shares
    of K for some; test_host_routes.py checks that it does."""
    import torch
    t, d = di.scaled(di.CONFIGS[model]["target"], n_layers=2, vocab=16384), di.scaled(di.DRAFTER_05B, n_layers=2, vocab=16384)
    eng = _engine(t, d, 1, 64 * (-(-(n + 32) // 64)), torch)
    prompts = [di.prompt_ids(t.vocab, n)]
    blocks = torch.from_numpy(np.random.default_rng(2).integers(0, t.vocab, (1, 32)).astype(np.int32)).cuda()
    eng.debug_gemm_tiled(0)
    _outputs(eng, prompts, 32, blocks, torch)
    want = _outputs(eng, prompts, 32, blocks, torch)
    eng.debug_gemm_tiled(128)
    _compare(want, _outputs(eng, prompts, 32, blocks, torch))
    eng.close()


def test_grouped_gemms_of_long_contractions():
    """Experts of 112 (gate/up) and 108 (down) k-steps, which fold the other way than the small ones of test_gpu_block_gemm.py:
    gathered rows and blocked gate/up, and the streaming gate/up, against the oracle."""
    import torch
    from gpu_common import StoredWeights, make_engine, make_pair
    t = di.ModelShape(1, 1792, 4, 2, 64, 0, 1024, n_experts=4, top_k=2, d_ff_expert=1728, rope_base=1e4)
    d, k, lens = di.CONFIGS["tiny"]["drafter"], 8, [190, 3]
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(d, di.DRAFTER_SEED, "bf16")
    eng = make_engine(t, d, wt, wd, len(lens), 256, k)
    prompts = [di.prompt_ids(t.vocab, n, seq=70 + b) for b, n in enumerate(lens)]
    blocks = np.random.default_rng(3).integers(0, t.vocab, (len(lens), k)).astype(np.int32)
    got = []
    for mode in (0, 128):
        eng.debug_gemm_tiled(mode)
        got.append(_outputs(eng, prompts, k, torch.from_numpy(blocks).cuda(), torch)[1][1])
    for b, prompt in enumerate(prompts):
        pair = make_pair(t, d, wt, wd, 256)
        pair.prefill(prompt)
        z = pair.verify_logits([int(v) for v in blocks[b]])
        for g in got:
            assert np.abs(g[b] - z).max() < 2e-3, (b, np.abs(g[b] - z).max())   # the small mixtures' bound
    eng.close()
