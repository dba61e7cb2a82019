"""What a launch fetches ahead for the one behind it (host side, no GPU): the matrix, the column groups and the workgroups are those
of the launch that really follows, also where the last layer of a prompt ends with its K and V rows."""
import os
import sys

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub"))
from host_engine import run_script   # noqa: E402


def test_the_next_launch_is_the_one_planned_for(tmp_path):
    out = run_script(tmp_path, """
import re
import deer_inputs as di
def check(e, call):
    e.stub.stub_reset()
    assert call() == 0
    gemms, planned = e.gemms(), 0
    for (_, _, a), (name, grid, b) in zip(gemms, gemms[1:]):
        if not a.nx_base: continue
        planned += 1
        assert a.nx_base == b.W, (name, grid, b.N)
        if a.nx_narrow_nb:
            assert "k_gemm_narrow" in name and a.nx_ncg * 32 * a.nx_narrow_nb == b.N and a.nx_nwg == grid[0], (name, grid)
        else:
            slim = re.search("k_gemm_slimILi(\\d)", name)
            assert a.nx_ncg * 32 * a.nx_nblk == b.N and a.nx_nblk == (int(slim[1]) if slim else 4) and a.nx_nwg == a.nx_ncg * b.S, (name, grid, b.S)
    return planned
for d, hq, hkv, hd, ff in ((1152, 9, 3, 128, 1216), (2560, 32, 8, 128, 9728), (4096, 32, 8, 128, 12288), (896, 14, 2, 64, 4864), (384, 6, 3, 64, 2112), (256, 4, 2, 32, 512)):
    for layers in (4, 6):
        t = di.ModelShape(layers, d, hq, hkv, hd, ff, 1152, rope_base=1e4)
        e = HostEngine(t, di.ModelShape(1, 128, 4, 2, 32, 512, 1152, rope_base=1e4), 2, 256)
        got = [check(e, lambda: e.prefill([[3] * n])) for n in (20, 33, 60)]   # one row tile; two
        assert got[:2] == [layers - 1] * 2, (d, layers, got)
        e.set_prefilled([40], [3]); e.draft_block(8)
        assert check(e, lambda: e.verify_block(8)) == layers - 1, d
print("checked")
""")
    assert out == "checked\n"
