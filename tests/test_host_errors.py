"""What a HIP error in the middle of a call leaves behind, with a stand-in for the HIP runtime (no GPU): after a prefill or
set_prefilled that failed the context holds no sequences (the device state may be of the new ones, the host's mirror of the
old), nothing is in flight any more, and a repeated call works."""
import sys
import os

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub"))
from host_engine import run_script   # noqa: E402

SCRIPT = """
import deer_inputs as di
cfg = di.CONFIGS["tiny"]
e = HostEngine(cfg["target"], cfg["drafter"], 2, 256)
call = lambda: e.{call}
assert e.set_prefilled([200, 100], [1, 2]) == 0
e.stub.stub_reset()
assert call() == 0
launches, copies, syncs = e.stub.stub_launches(), e.stub.stub_copies(), e.stub.stub_syncs()
for kind, n in (("launch", launches), ("copy", copies), ("sync", syncs)):
    for at in range(n):
        assert e.set_prefilled([200, 100], [1, 2]) == 0
        e.stub.stub_reset()
        e.stub.stub_fail(*(at if k == kind else -1 for k in ("launch", "copy", "sync")))
        assert call() == -4, (kind, at)                     # DEER_EHIP
        assert e.stub.stub_syncs() >= 1, (kind, at)         # nothing is in flight: the next call may reuse the staging
        e.stub.stub_fail(-1, -1, -1)
        assert e.draft_block(8) == -2, (kind, at)           # DEER_ESTATE
        assert call() == 0 and e.draft_block(8) == 0
print("checked", launches, copies, syncs)
"""


@pytest.mark.parametrize("call", ["prefill([[3] * 40, [4] * 70])", "set_prefilled([40, 70], [3, 4])"])
def test_a_failed_call_leaves_no_sequences(tmp_path, call):
    out = run_script(tmp_path, SCRIPT.format(call=call))
    assert out.startswith("checked"), out


@pytest.mark.parametrize("layers", [4, 6])
def test_a_failed_prefill_of_both_models_at_once_leaves_no_sequences(tmp_path, layers):
    """The same where the drafter's passes run on a stream of their own (which stream is waited for, and failing events:
    test_host_prefill_beside.py)."""
    script = SCRIPT.replace('e = HostEngine(cfg["target"], cfg["drafter"], 2, 256)', f'e = HostEngine(cfg["target"], di.scaled(cfg["drafter"], n_layers={layers}), 2, 256)')
    out = run_script(tmp_path, script.format(call="prefill([[3] * 40, [4] * 70])"))
    assert out.startswith("checked"), out
