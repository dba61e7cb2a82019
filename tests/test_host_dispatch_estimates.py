"""Which kernel the dense GEMMs of a pass take where the streaming kernel and the blocked one are close (host side, no GPU):
launches that were measured on both sides, and the side that was faster there."""
import os
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub"))
from host_engine import run_script   # noqa: E402

SHAPES = {   # d_model, query heads, kv heads, head_dim, d_ff
    "d896": (896, 14, 2, 64, 4864), "d1024": (1024, 8, 4, 128, 3072), "d1536": (1536, 12, 4, 128, 8960), "d2048": (2048, 16, 8, 128, 6144),
    "d2560": (2560, 32, 8, 128, 9728), "d4096": (4096, 32, 8, 128, 12288),
}
SLOTS = ("QKV", "O", "gate/up", "down")


def launches(tmp_path, wanted):
    """(kernel, arguments' S) per (shape, row tiles, GEMM of the layer)."""
    return eval(run_script(tmp_path, f"""
import re
import deer_inputs as di
out = {{}}
for name, (d, hq, hkv, hd, ff) in {SHAPES!r}.items():
    tiles = sorted({{t for s, t, _ in {wanted!r} if s == name}})
    if not tiles: continue
    e = HostEngine(di.ModelShape(1, d, hq, hkv, hd, ff, 1152, rope_base=1e4), di.ModelShape(1, 128, 4, 2, 32, 512, 1152, rope_base=1e4), max(tiles), 64)
    for t in tiles:
        assert e.set_prefilled([20] * t, [5] * t) == 0 and e.draft_block(32) == 0
        e.stub.stub_reset()
        assert e.verify_block(32) == 0
        for slot, (n, g, a) in zip({SLOTS!r}, e.gemms()):
            m = re.search("k_gemm_blockILi(\\\\d)ELi(\\\\d)E", n)
            out[name, t, slot] = ("block, ring of " + m[2] if m else "streaming", a.S)
print(out)
"""))


# microseconds streaming / blocked
FASTER = [
    ("d2048", (3, 4, 6, 8), "gate/up", "block, ring of 8"),  # (rings of 4 / 8) 28.6 / 26.4, 29.8 / 28.4, 40.1 / 38.6, 40.8 / 39.0
    ("d2048", (18, 20, 28), "QKV", "block, ring of 8"),      # 42.0 / 40.8, 42.2 / 41.1, 45.4 / 43.5
]


def test_the_faster_kernel_runs(tmp_path):
    wanted = [(s, t, slot) for s, tiles, slot, _ in FASTER for t in tiles]
    got = launches(tmp_path, wanted)
    off = {(s, t, slot): got[s, t, slot] for s, tiles, slot, kernel in FASTER for t in tiles if got[s, t, slot][0] != kernel}
    assert not off, off
