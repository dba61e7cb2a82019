"""GPU parity of a mixture's grouped GEMMs in passes with few rows per expert: contractions of one, three, five and many
stages of four k-steps, folded either way and summed in eighths, numbers of columns that leave waves without any, experts of one to 90 pairs (several
work items), against the oracle; and (on the CPU) that these passes take that kernel."""
import os
import sys

import numpy as np
import pytest

import deer_inputs as di
from gpu_common import StoredWeights, gpu_available, make_engine, make_pair

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub"))
from host_engine import run_script   # noqa: E402

TOL = 2e-3   # the small mixtures' bound elsewhere
SHAPES = {   # k-steps of gate/up and down, 64-column units of either
    "24, 12 k-steps, 6, 6 units": dict(d_model=384, n_experts=20, top_k=2, d_ff_expert=192),
    "8, 4 k-steps, 2, 2 units": dict(d_model=128, n_experts=12, top_k=1, d_ff_expert=64),
    "40, 20 k-steps, 10, 10 units": dict(d_model=640, n_experts=40, top_k=3, d_ff_expert=320),
    "112, 108 k-steps, 54, 28 units, folded plainly": dict(d_model=1792, n_experts=16, top_k=2, d_ff_expert=1728),
    "32, 8 k-steps, 4, 8 units, eighths of one stage": dict(d_model=512, n_experts=20, top_k=2, d_ff_expert=128),
    "128, 12 k-steps, 6, 32 units, eighths of four": dict(d_model=2048, n_experts=20, top_k=2, d_ff_expert=192),
}


def shape(name):
    s = SHAPES[name]
    return di.ModelShape(2, s["d_model"], 4, 2, 32, 0, 1024, n_experts=s["n_experts"], top_k=s["top_k"], d_ff_expert=s["d_ff_expert"], rope_base=1e4)


def prompts(vocab):
    """Few rows; a batch; one token again and again, whose rows all go to the same experts."""
    return [[di.prompt_ids(vocab, 4)], [di.prompt_ids(vocab, n, seq=9 + n) for n in (34, 20, 2)], [np.full(91, 7, np.int32)]]


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("name", SHAPES)
def test_few_rows_per_expert(name):
    import torch
    t, d, k = shape(name), di.CONFIGS["tiny"]["drafter"], 8
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(d, di.DRAFTER_SEED, "bf16")
    eng = make_engine(t, d, wt, wd, 3, 192, k)
    for ps in prompts(t.vocab):
        blocks = np.random.default_rng(6).integers(0, t.vocab, (len(ps), k)).astype(np.int32)
        eng.prefill(ps)
        eng.draft_block(k, 0.0, 0)
        eng.verify_block(k, 0.0, torch.from_numpy(blocks).cuda())
        zt = eng.debug_get_logits(0, k)
        for b, p in enumerate(ps):
            pair = make_pair(t, d, wt, wd, 192)
            pair.prefill(p)
            off = np.abs(zt[b] - pair.verify_logits([int(v) for v in blocks[b]])).max()
            assert off < TOL, (len(ps), b, off)
    eng.close()


def test_which_passes_take_it(tmp_path):
    """The shapes above up to their lines; 128 experts of 2048 x 768: gate/up up to 24, down up to 20 pairs per expert."""
    out = run_script(tmp_path, f"""
import deer_inputs as di
def kinds(e, call):
    e.stub.stub_reset()
    assert call() == 0
    names = [n for n, _ in e.launches()]
    return ["few" if "k_gemm_moe" in n else "block" for n in names if "k_gemm_moe" in n or "k_moe_block" in n][:2]
def grid(columns, rows, t, item):   # work items, at most, times blocks of 256 columns, the same for every XCD
    return -(-(min(t.n_experts, rows * t.top_k) + rows * t.top_k // item) * -(-columns // 256) // 8) * 8
for s in {list(SHAPES.values())!r}:
    t = di.ModelShape(2, s["d_model"], 4, 2, 32, 0, 1024, n_experts=s["n_experts"], top_k=s["top_k"], d_ff_expert=s["d_ff_expert"], rope_base=1e4)
    e = HostEngine(t, di.CONFIGS["tiny"]["drafter"], 3, 192)
    for lens in ([4], [34, 20, 2], [91]):
        rows = -(-sum(n - 1 for n in lens) // 32) * 32
        want = ["few" if rows * t.top_k < line * t.n_experts else "block" for line in ((14, 12) if t.d_model * t.d_ff_expert * 4 < 1 << 20 else (24, 20))]
        assert kinds(e, lambda: e.prefill([[3] * n for n in lens])) == want, (s, lens)
        assert want == ["few", "few"], (s, lens)
        got = [g[0] for n, g in e.launches() if "k_gemm_moe" in n][:2]   # items of 32 pairs
        assert got == [grid(2 * t.d_ff_expert, rows, t, 32), grid(t.d_model, rows, t, 32)], (s, lens, got)
t = di.scaled(di.CONFIGS["qwen3_30b_a3b"]["target"], n_layers=1, vocab=1024)
e = HostEngine(t, di.CONFIGS["tiny"]["drafter"], 1, 512)
out = []
for n in (1, 9, 10, 11, 12):   # the blocked kernel's items have 64
    out.append(kinds(e, lambda: e.prefill([[3] * (32 * n + 1)])))
    item = 32 if out[-1] == ["few", "few"] else 64
    got = [g[0] for n, g in e.launches() if "k_gemm_moe" in n or "k_moe_block" in n][:2]
    assert got == [grid(2 * t.d_ff_expert, 32 * n, t, item), grid(t.d_model, 32 * n, t, item)], (n, got)
print(out)
""")
    assert eval(out) == [["few", "few"], ["few", "few"], ["few", "block"], ["few", "block"], ["block", "block"]], out
