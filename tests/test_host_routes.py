"""Which GEMM kernels the host side launches for a prompt or a batch (a stand-in for the HIP runtime records them, no GPU):
that the forms the parity tests compare are the ones that run there, and that every form is reached by a test."""
import os
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub"))
from host_engine import run_script   # noqa: E402

SCRIPT = """
import re
import deer_inputs as di
def engine(t, d, batch, max_seq):
    return HostEngine(t, d, batch, max_seq)
def gemms(e, call):
    e.stub.stub_reset()
    assert call() == 0
    out = set()
    for name, grid in e.launches():
        m = re.search("k_gemm_blockILi(\\\\d)ELi(\\\\d)ELi(\\\\d)ELb(\\\\d)E", name)
        if m: out.add("block<%s,%s,%s,%s>" % m.groups())
        elif "k_moe_block" in name: out.add("moe_block")
        elif "k_gemm" in name: out.add(re.search("k_gemm(_rows|_narrow|_moe)?", name)[0])
    return out
"""
QKV, RESID, SWIGLU, LM = range(4)


def routes(tmp_path, body):
    return eval(run_script(tmp_path, SCRIPT + body))


def test_wide_prompts_reach_the_256_column_form(tmp_path):
    """The prompts of test_gpu_block_forms.py::test_wide_prompts_agree, with the estimate's own choice."""
    got = routes(tmp_path, """
t8, t4 = (di.scaled(di.CONFIGS[c]["target"], n_layers=2, vocab=16384) for c in ("qwen3_8b", "qwen3_4b"))
d = di.scaled(di.DRAFTER_05B, n_layers=2, vocab=16384)
print([gemms(e, lambda: e.prefill([[3] * n])) for e, n in ((engine(t8, d, 1, 2176), 2100), (engine(t4, d, 1, 3392), 3329))])
""")
    assert {f"block<4,4,{e},0>" for e in (QKV, RESID, SWIGLU)} <= got[0], got[0]
    assert {f"block<4,4,{e},0>" for e in (RESID, SWIGLU)} <= got[1], got[1]


@pytest.mark.parametrize("d,form,ring", [(384, (2, 4), 4), (384, (2, 8), 4), (384, (4, 4), 4), (1664, (2, 4), 4), (1664, (2, 8), 8)])
def test_the_forced_form_runs_in_every_dense_gemm(tmp_path, d, form, ring):
    """d = 1664: every contraction has 104 k-steps, the shortest that folds plainly and may have the ring of 8."""
    got = routes(tmp_path, f"""
t = di.ModelShape(1, {d}, {d // 64}, {d // 128}, 64, {d}, 1152, rope_base=1e4)
e = engine(t, t, 3, 512)
assert e.lib.deer_debug_gemm_block(e.ctx, {form[0]}, {form[1]}, 3) == 0
a = gemms(e, lambda: e.prefill([[3] * 290, [4] * 33, [5] * 200]))
b = gemms(e, lambda: e.draft_block(32))
assert e.lib.deer_debug_gemm_block(e.ctx, 0, 0, 0) == 0 and e.lib.deer_debug_gemm_tiled(e.ctx, 0) == 0
c = gemms(e, lambda: e.verify_block(32))
bad = [e.lib.deer_debug_gemm_block(e.ctx, *f) for f in ((4, 8, 1), (3, 4, 1), (2, 4, 0), (2, 4, 9), (2, 5, 1))]
print((a, b, c, bad))
""")
    name = lambda e: f"block<{form[0]},{ring},{e},{int(form[0] == 2 and d < 1664)}>"   # noqa: E731
    assert got[0] == {name(e) for e in (QKV, RESID, SWIGLU)}, got[0]
    assert got[1] == got[0] | {name(LM)}, got[1]
    assert not any("block" in n for n in got[2]), got[2]
    assert got[3] == [-1] * 5


def test_rows_of_the_block_gemm_tests_take_the_blocked_kernel(tmp_path):
    """The cases of test_gpu_block_gemm.py with the estimate's choice (its other two settings switch the kernel off and
    force it): from 5 row tiles on some GEMM of the prompt runs blocked."""
    got = routes(tmp_path, """
t = di.scaled(di.CONFIGS["qwen3_8b"]["target"], n_layers=2, vocab=16384)
d = di.scaled(di.DRAFTER_05B, n_layers=2, vocab=16384)
e = engine(t, d, 9, 1536)
out = []
for lens, k in (([97], 32), ([161, 33], 5), ([225], 1), ([511], 17), ([40, 300, 77, 129, 65, 31, 2, 1, 200], 32), ([1200], 32)):
    a = gemms(e, lambda: e.prefill([[3] * n for n in lens]))
    out.append((a, gemms(e, lambda: e.draft_block(k)) | gemms(e, lambda: e.verify_block(k))))
print(out)
""")
    for i, (prompt, block) in enumerate(got):
        print(i, sorted(prompt), sorted(block))
    assert all(any(n.startswith("block") for n in prompt) for prompt, _ in got)
    assert any(n.startswith("block<2") and n.split(",")[2] == str(LM) for n in got[4][1])


def test_small_models_take_the_kernel_that_is_faster_there(tmp_path):
    """Narrow workgroups against the blocked kernel, by the matrices' sizes.  Microseconds, narrow / blocked: O of d = 256 at 63
    row tiles 8.4 / 11.5, of d = 896 at 31 17.0 / 19.1 and at 63 41 / 20; QKV of d = 1024 with 16 kv heads at 31 40 / 26, of
    d = 512 with 2 at 31 10.8 / 19.0."""
    got = routes(tmp_path, """
out = []
for d, hq, hkv, tiles in ((256, 4, 2, 63), (896, 14, 2, 31), (896, 14, 2, 63), (1024, 16, 16, 31), (512, 8, 2, 31)):
    t = di.ModelShape(1, d, hq, hkv, 64, 2048, 1024, rope_base=1e4)
    e = engine(t, t, 1, 2112)
    e.stub.stub_reset()
    assert e.prefill([[3] * 32 * tiles]) == 0
    names = [n for n, _ in e.launches() if "k_gemm" in n]
    out.append(["block" in names[0], "block" in names[1]])   # QKV, O
print(out)
""")
    assert got[0][1] is False and got[1][1] is False and got[2][1] is True and got[3][0] is True and got[4][0] is False, got


def test_a_batch_of_64_blocks_runs_blocked_throughout(tmp_path):
    """The passes of test_gpu_tiled_gemm.py::test_batch_of_64_sequences_through_tiled_gemm: 64 row tiles, every GEMM blocked."""
    got = routes(tmp_path, """
t, d = di.CONFIGS["tiny"]["target"], di.CONFIGS["tiny"]["drafter"]
e = engine(t, d, 64, 128)
assert e.lib.deer_debug_gemm_tiled(e.ctx, 1) == 0
e.prefill([[3] * 40] * 64)
a = gemms(e, lambda: e.draft_block(32))
tiles = [g for n, g in e.launches() if "k_pass_begin" in n]
print((a, gemms(e, lambda: e.verify_block(32)), tiles))
""")
    assert all(n.startswith("block") for n in got[0] | got[1]) and len(got[0]) == 4, got
    assert got[2][0][1] == 64


def test_grouped_gate_up_runs_blocked_where_experts_have_rows_enough(tmp_path):
    """128 small experts, top 8: 12 pairs per expert at 6 row tiles, below the line of their gate/up projections (14) and at that
    of their down projections (12); 14 at 7."""
    got = routes(tmp_path, """
t = di.ModelShape(1, 256, 4, 2, 32, 0, 1024, n_experts=128, top_k=8, d_ff_expert=128, rope_base=1e4)
e = engine(t, di.CONFIGS["tiny"]["drafter"], 1, 512)
print([gemms(e, lambda: e.prefill([[3] * (32 * n + 1)])) for n in (6, 7)])
""")
    assert "k_gemm_moe" in got[0] and "k_gemm_moe" not in got[1] and "moe_block" in got[0] & got[1], got


def test_shapes_of_the_slim_gemm_tests_take_it(tmp_path):
    """The shapes and batches of test_gpu_slim_gemm.py: every form of the small-workgroup kernel runs in one of them, and none
    where it is switched off."""
    got = routes(tmp_path, """
def slim(e, call):
    e.stub.stub_reset()
    assert call() == 0
    return {re.search("k_gemm_slimILi(\\d)ELi(\\d)E", n).groups() for n, _ in e.launches() if "k_gemm_slim" in n}
out = []
for d, hq, hkv, hd, ff in ((1152, 9, 3, 128, 1216), (2048, 16, 4, 64, 5632), (1280, 20, 4, 32, 1344), (384, 6, 3, 64, 2112)):
    t = di.ModelShape(2, d, hq, hkv, hd, ff, 1152, rope_base=1e4)
    e = engine(t, di.ModelShape(1, 384, 6, 3, 64, 2112, 1152, rope_base=1e4), 4, 256)
    for lens, k in (([70], 32), ([33], 5), ([40, 65, 8], 20), ([64, 31, 100], 31), ([50, 9, 128, 77], 32)):
        for mode in (0, 128):
            e.lib.deer_debug_gemm_tiled(e.ctx, mode)
            e.set_prefilled(lens, [5] * len(lens))
            out.append((hd if d > 384 else 0, len(lens), mode, slim(e, lambda: e.draft_block(k)), slim(e, lambda: e.verify_block(k))))
print(out)
""")
    assert all(not d and not v for _, _, mode, d, v in got if mode == 0)
    on = [(hd, n, v) for hd, n, mode, _, v in got if mode]   # the target's passes
    for hd in (128, 64, 32):
        forms = set().union(*(f for h, _, f in on if h == hd))
        assert {("2", str(QKV)), ("2", str(RESID))} <= forms, (hd, forms)
    assert ("1", str(RESID)) in set().union(*(f for h, _, f in on if h == 0))
    assert ("2", str(SWIGLU)) in set().union(*(f for _, _, f in on)) and all(d for _, _, mode, d, _ in got if mode)
    assert all(any(f for h, n, f in on if n == m) for m in (1, 3, 4)), on


def test_shapes_of_the_pieces_tests_run_in_pieces(tmp_path):
    """The shape and prompts of test_gpu_block_pieces.py: launches of the blocked kernel whose grid is whole blocks for every
    compute unit and pieces of the rest."""
    got = routes(tmp_path, """
t = di.ModelShape(2, 1152, 18, 2, 64, 8384, 16512, rope_base=1e4)
def pieces(e, call):
    e.stub.stub_reset()
    assert call() == 0
    out = set()
    for name, grid in e.launches():
        m = re.search("k_gemm_blockILi(\\\\d)ELi4ELi(\\\\d)E", name)
        if m: out.add((int(m[1]), int(m[2]), grid[0]))
    return out
out = []
for lens, k in (([202], 5), ([130, 40, 33, 1, 60], 32), ([3840], 32)):
    e = engine(t, di.ModelShape(1, 384, 6, 3, 64, 640, 16512, rope_base=1e4), len(lens), -(-(max(lens) + 64) // 64) * 64)
    a = pieces(e, lambda: e.prefill([[3] * n for n in lens]))
    e.draft_block(k)
    out.append((a, pieces(e, lambda: e.verify_block(k))))
e = engine(di.scaled(di.CONFIGS["qwen3_4b"]["target"], n_layers=2, vocab=16384), di.scaled(di.DRAFTER_05B, n_layers=2, vocab=16384), 1, 3392)
out.append((pieces(e, lambda: e.prefill([[3] * 3329])), set()))
print(out)
""")
    print(got)
    blocks = lambda nb, cols, nrb: -(-cols // (64 * nb)) * nrb   # noqa: E731
    whole = lambda n: 8 * -(-n // 8)   # noqa: E731  (the grid without pieces)
    assert any(e == SWIGLU and g > whole(blocks(nb, 16768, 2)) for nb, e, g in got[0][0])
    assert any(e == LM and g > whole(blocks(nb, 16512, 2)) for nb, e, g in got[1][1])
    assert any(e == RESID and g > whole(blocks(nb, 1152, 30)) for nb, e, g in got[2][0])
    # and the 256-column form in the longer of the wide prompts of test_gpu_block_forms.py
    assert any((nb, e) == (4, RESID) and g > whole(blocks(4, 2560, 27)) for nb, e, g in got[3][0])


def test_no_share_of_a_slim_gemm_is_empty(tmp_path):
    """A share is a whole number of rounds of the eight waves: of 72 k-steps three shares have 24 each and a fourth none."""
    got = routes(tmp_path, """
out = []
for d, ff in ((1152, 1088), (1152, 1152), (1152, 2304), (2048, 2304), (2560, 1344), (2560, 9728), (4096, 12288)):
    t = di.ModelShape(1, d, 4, 2, 64, ff, 1152, rope_base=1e4)
    e = engine(t, di.ModelShape(1, 128, 4, 2, 32, 512, 1152, rope_base=1e4), 2, 256)
    for lens in ([70], [70, 33]):
        e.set_prefilled(lens, [5] * len(lens))
        assert e.draft_block(32) == 0
        e.stub.stub_reset()
        assert e.verify_block(32) == 0
        name, grid = [l for l in e.launches() if "k_gemm" in l[0]][3]   # down
        out.append((d, ff // 16, len(lens), grid[0] if "k_gemm_slim" in name else 0))
print(out)
""")
    seen = 0
    for d, ks, tiles, grid in got:
        if grid:
            S = next(s for s in range(1, 9) if (d // 64 * s + 7) // 8 * 8 * tiles == grid)
            assert (S - 1) * 8 * -(-ks // (8 * S)) < ks, (d, ks, tiles, S)
            seen += 1
    assert seen >= 10, got


def test_gate_up_of_four_row_tiles_takes_the_faster_kernel(tmp_path):
    """Microseconds streaming / blocked: 9728 columns of d = 896 18.1 / 19.1, 11264 of 1408 23.6 / 29.8, 24576 of 4096 81 / 73."""
    got = routes(tmp_path, """
out = []
for d, hq, hd, ff in ((896, 14, 64, 4864), (1408, 11, 128, 5632), (4096, 32, 128, 12288)):
    t = di.ModelShape(1, d, hq, 1 if hq % 2 else 2, hd, ff, 1152, rope_base=1e4)
    e = engine(t, di.ModelShape(1, 128, 4, 2, 32, 512, 1152, rope_base=1e4), 4, 256)
    e.set_prefilled([100] * 4, [5] * 4)
    assert e.draft_block(32) == 0
    e.stub.stub_reset()
    assert e.verify_block(32) == 0
    out.append("block" in [n for n, _ in e.launches() if "k_gemm" in n][2])
print(out)
""")
    assert got == [False, False, True], got


def test_down_projections_take_the_faster_streaming_kernel(tmp_path):
    """One row tile, microseconds wide / small workgroups: 12288 x 4096 in a pass 24.5 / 23.5, 9728 x 2560 19.8 / 16.1, 18944 x
    3584 31.9 / 33.3."""
    got = routes(tmp_path, """
out = []
for d, hq, ff in ((4096, 32, 12288), (2560, 32, 9728), (3584, 28, 18944)):
    t = di.ModelShape(1, d, hq, 4, 128, ff, 1152, rope_base=1e4)
    e = engine(t, di.ModelShape(1, 128, 4, 2, 32, 512, 1152, rope_base=1e4), 1, 256)
    e.set_prefilled([100], [5])
    assert e.draft_block(32) == 0
    e.stub.stub_reset()
    assert e.verify_block(32) == 0
    out.append("k_gemm_slim" in [n for n, _ in e.launches() if "k_gemm" in n][3])
print(out)
""")
    assert got == [True, True, False], got
