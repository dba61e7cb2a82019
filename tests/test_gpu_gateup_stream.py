"""GPU parity of gate/up over two row tiles of large matrices (columns streamed by one wave each, K in shares): one to four
shares, the last one shorter, waves without columns, against the weight-streaming kernels; and (on the CPU) which passes take it."""
import os
import sys

import numpy as np
import pytest

import deer_inputs as di
from gpu_common import gpu_available
from test_gpu_block_forms import _compare, _engine, _outputs

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub"))
from host_engine import run_script   # noqa: E402

# (d_model, d_ff, shares): 104, 112 and 160 k-steps; column blocks 64, 65 (the last with two waves of columns), 120 and 161
SHAPES = [(1664, 8192, 4), (1792, 8256, 3), (2560, 15360, 2), (1664, 20544, 3)]
LENS, K = [34, 31], 32
# not taken: below 51 MB, below 104 k-steps, columns so few that the streaming kernel has three shares of K or more, or small workgroups
NONE = [(1664, 4608), (1536, 9216), (4096, 4608), (5120, 4096), (4096, 4096), (8192, 2048)]


def shape(d, ff):
    return di.ModelShape(2, d, 8, 2, 64, ff, 1152, rope_base=1e4)


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("d,ff,shares", SHAPES)
def test_two_row_tiles_agree_with_the_streaming_kernels(d, ff, shares):
    import torch
    t, dr = shape(d, ff), di.ModelShape(1, 384, 6, 3, 64, 640, 1152, rope_base=1e4)
    eng = _engine(t, dr, len(LENS), 128, torch)
    prompts = [di.prompt_ids(t.vocab, n, seq=b) for b, n in enumerate(LENS)]
    blocks = torch.from_numpy(np.random.default_rng(1).integers(0, t.vocab, (len(LENS), K)).astype(np.int32)).cuda()
    out = {}
    for mode in (0, 128):
        eng.debug_gemm_tiled(mode)
        _outputs(eng, prompts, K, blocks, torch)
        out[mode] = _outputs(eng, prompts, K, blocks, torch)
    _compare(out[0], out[128])
    eng.close()


def test_which_passes_take_it(tmp_path):
    out = run_script(tmp_path, f"""
import deer_inputs as di
def grids(e, call):
    e.stub.stub_reset()
    assert call() == 0
    return [g[0] for n, g in e.launches() if "k_gemm_gateup" in n]
out = []
for d, ff in {[s[:2] for s in SHAPES] + [(4096, 5120)] + NONE!r}:
    t = di.ModelShape(2, d, 8, 2, 64, ff, 1152, rope_base=1e4)
    e = HostEngine(t, di.ModelShape(1, 384, 6, 3, 64, 640, 1152, rope_base=1e4), 3, 128)
    one = grids(e, lambda: e.prefill([[3] * 33]))
    two = grids(e, lambda: e.prefill([[3] * n for n in {LENS!r}]))
    three = grids(e, lambda: e.prefill([[3] * 33, [4] * 34, [5] * 32]))
    assert e.draft_block({K}) == 0
    e.set_prefilled([20, 30], [5, 5]); assert e.draft_block({K}) == 0
    verify = grids(e, lambda: e.verify_block({K}))
    e.lib.deer_debug_gemm_tiled(e.ctx, 0)
    off = grids(e, lambda: e.prefill([[3] * n for n in {LENS!r}]))
    assert one == three == off == [] and verify == two, (d, ff, one, two, three, verify, off)
    out.append(two)
print(out)
""")
    assert eval(out) == [[-(-ff * 2 // 256) * s] * 2 for _, ff, s in SHAPES] + [[40 * 6] * 2] + [[]] * len(NONE), out
