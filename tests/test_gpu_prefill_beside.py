"""A prefill whose drafter passes run beside the target's, on a second stream with buffers of their own, leaves the caches that
the same passes leave one after the other (which they do while launches are timed): bit for bit, pass after pass with new
prompts, for dense and mixture targets, from one row of the drafter to the 2048 that its second set of buffers holds (and one
more, which goes through the first set), and decoding from them agrees.  That they run on two streams is checked without a GPU
in test_host_prefill_beside.py."""
import numpy as np
import pytest

import deer_inputs as di
from gpu_common import gpu_available
from test_gpu_block_forms import _engine

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _mixture(t, d, batch, max_seq, torch):
    from paper_2512_15176_amd import DeerEngine
    eng = DeerEngine(t, d, batch, max_seq, 32, t.vocab - 1, keep_logits=True)
    gen = torch.Generator(device="cuda").manual_seed(11)
    w = lambda *s: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(0.02)   # noqa: E731
    for m, s in enumerate((t, d)):
        q, kv = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
        eng.load_tensor(m, "embed", -1, -1, w(s.vocab, s.d_model).mul_(50))   # N(0, 1): the router spreads the rows
        eng.load_tensor(m, "lm_head", -1, -1, w(s.d_model, s.vocab))
        for layer in range(s.n_layers):
            for name, r, c in (("wq", s.d_model, q), ("wk", s.d_model, kv), ("wv", s.d_model, kv), ("wo", q, s.d_model)):
                eng.load_tensor(m, name, layer, -1, w(r, c))
            f = s.d_ff_expert if s.n_experts else s.d_ff
            if s.n_experts:
                eng.load_tensor(m, "router", layer, -1, w(s.d_model, s.n_experts))
            for e in range(s.n_experts or 1):
                for name, r, c in (("wg", s.d_model, f), ("wu", s.d_model, f), ("wd", f, s.d_model)):
                    eng.load_tensor(m, name, layer, e if s.n_experts else -1, w(r, c))
    return eng


LONG = (6, 1024, ([5], [201], [60, 333, 7, 128, 64, 500], [2], [700, 31], [33] * 6, [960, 900], [700, 31, 640, 677], [700, 31, 640, 678]))
SHORT = (3, 64, ([32], [1, 32, 32], [32, 31, 32], [32] * 3))   # contexts whose second set has 6 row tiles and 6 attention tiles


@pytest.mark.parametrize("mixture,size", [(False, LONG), (True, LONG), (False, SHORT), (True, SHORT)], ids=["False", "True", "short", "short-mixture"])
def test_beside_is_the_same_as_one_after_the_other(mixture, size):
    import torch
    batch, max_seq, sets = size
    d = di.ModelShape(4, 896, 14, 2, 64, 2432, 2048, rope_base=1e4)
    t = di.ModelShape(3, 512, 8, 2, 64, 0, 2048, n_experts=16, top_k=4, d_ff_expert=256, rope_base=1e4) if mixture else \
        di.ModelShape(6, 1280, 10, 2, 128, 3456, 2048, rope_base=1e4)
    eng = (_mixture if mixture else _engine)(t, d, batch, max_seq, torch)
    for rep, lens in enumerate(sets):
        prompts = [di.prompt_ids(t.vocab, n, seq=100 * rep + b) for b, n in enumerate(lens)]
        block = torch.from_numpy(np.random.default_rng(rep).integers(0, t.vocab, (len(lens), 16)).astype(np.int32)).cuda()
        out = []
        for timed in (1, 0, 0):
            for x in eng._kv:
                x.zero_()
            eng.debug_profile(timed)
            eng.prefill(prompts)
            eng.debug_profile(0)
            kv = [x.view(torch.bfloat16).clone() for x in eng._kv]
            eng.draft_block(16, 0.0, 0)
            zd = eng.debug_get_logits(1, 16)
            eng.verify_block(16, 0.0, block)
            out.append((kv, zd, eng.debug_get_logits(0, 16)))
            eng.accept_and_commit(16, 0.0, 0)
        for kv, zd, zt in out[1:]:
            assert all(torch.equal(a, b) for a, b in zip(out[0][0], kv)), (mixture, lens)
            assert np.array_equal(out[0][1], zd) and np.array_equal(out[0][2], zt), (mixture, lens)
    eng.close()
