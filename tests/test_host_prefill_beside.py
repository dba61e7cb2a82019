"""The second stream of a prefill, with a stand-in for the HIP runtime (no GPU): which passes run on it, between which events,
what becomes of it where a call fails, and where there is none."""
import os
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub"))
from host_engine import run_script   # noqa: E402

HEAD = """
import deer_inputs as di
tiny = di.CONFIGS["tiny"]
def engine(layers=4, batch=2, max_seq=256):
    return HostEngine(tiny["target"], di.scaled(tiny["drafter"], n_layers=layers), batch, max_seq)
def streams(e, prompts):   # the streams of the passes, in the order of the calls
    e.stub.stub_reset()
    assert e.prefill(prompts) == 0
    return [s for k, s, h in e.ops() if k == "launch" and h]
"""


def test_the_drafters_passes_run_on_a_second_stream_between_two_events(tmp_path):
    out = run_script(tmp_path, HEAD + """
e = engine()
for prompts in ([[3] * 40, [4] * 70], [[5] * 33]):
    e.stub.stub_reset()
    assert e.prefill(prompts) == 0
    ops = e.ops()
    main = ops[0][1]                                       # the upload goes first, on the library's stream
    at = lambda kind, stream, what=None: [i for i, o in enumerate(ops) if o[0] == kind and o[1] == stream and (what is None or o[2] == what)]
    side = {s for k, s, w in ops} - {main}
    assert len(side) == 1
    side = side.pop()
    passes = [o for o in ops if o[0] == "launch" and o[2]]
    assert [o[1] for o in passes] == [main, side] and passes[0][2] != passes[1][2]   # target, drafter, each with its rows
    (fork,), (join,) = at("record", main), at("record", side)
    assert at("copy", main)[-1] < fork < at("launch", main)[0] and not at("copy", side)
    assert at("wait", side, ops[fork][2])[0] < at("launch", side)[0] and at("launch", side)[-1] < join
    assert join < at("wait", main, ops[join][2])[0] < at("sync", main)[-1] and at("launch", main)[-1] < at("sync", main)[-1]
    assert len(at("launch", side)) == 1 + 5 * 4            # all of the drafter's launches: the start of the pass, five per layer
    e.stub.stub_reset()                                    # what follows runs on the library's stream alone
    assert e.draft_block(8) == 0 and e.verify_block(8) == 0 and {s for k, s, w in e.ops()} == {main}
print("checked")
""")
    assert out == "checked\n"


def test_passes_that_run_one_after_the_other(tmp_path):
    """Drafters of few layers, passes of more than 64 row tiles (65 of the drafter; 64 run beside), prompts of one token (no pass
    of the target), launches that are timed or stamped, and a context that could make no second stream or no events."""
    out = run_script(tmp_path, HEAD + """
assert len(set(streams(engine(3), [[3] * 40]))) == 1
e = engine(4, 2, 2112)
assert len(set(streams(e, [[3] * 2048]))) == 2
assert len(set(streams(e, [[3] * 2049]))) == 1
assert len(set(streams(e, [[3] * 1000, [4] * 1048]))) == 2
assert len(set(streams(e, [[3] * 1000, [4] * 1049]))) == 1
assert len(streams(e, [[3], [4]])) == 1
assert e.lib.deer_debug_profile(e.ctx, 1) == 0
assert len(set(streams(e, [[3] * 40]))) == 1
assert e.lib.deer_debug_profile(e.ctx, 0) == 0 and len(set(streams(e, [[3] * 40]))) == 2
assert e.lib.deer_debug_gemm_stamps(e.ctx, 0, 1, None, 0, None) == 0
assert len(set(streams(e, [[3] * 40]))) == 1
assert e.lib.deer_debug_gemm_stamps(e.ctx, 0, -1, None, 0, None) == 0 and len(set(streams(e, [[3] * 40]))) == 2
for kind, n in (("stream_create", 0), ("event_create", 0), ("event_create", 1)):
    e.stub.stub_fail_op(OPS.index(kind), n)
    f = engine()
    assert len(set(streams(f, [[3] * 40]))) == 1 and f.draft_block(8) == 0
    assert f.lib.deer_destroy(f.ctx) == 0
print("checked")
""")
    assert out == "checked\n"


@pytest.mark.parametrize("prompts", ["[[3] * 40, [4] * 70]", "[[3] * 1]"])
def test_whatever_fails_both_streams_have_been_waited_for(tmp_path, prompts):
    """Every launch, copy, event and wait of a prefill fails in turn: behind the last launch on a stream the host waits for that
    stream before the call returns, no sequences are left, and the next call works."""
    out = run_script(tmp_path, HEAD + f"""
e = engine()
call = lambda: e.prefill({prompts})
e.stub.stub_reset()
assert call() == 0
ops, checked = e.ops(), 0
for kind in ("launch", "copy", "record", "wait"):
    for at in range(sum(k == kind for k, s, w in ops)):
        assert e.set_prefilled([200, 100], [1, 2]) == 0
        e.stub.stub_reset()
        if kind in ("launch", "copy"):
            e.stub.stub_fail(at if kind == "launch" else -1, at if kind == "copy" else -1, -1)
        else:
            e.stub.stub_fail_op(OPS.index(kind), at)
        assert call() == -4, (kind, at)                    # DEER_EHIP
        done = e.ops()
        for stream in {{s for k, s, w in done if k in ("launch", "copy")}}:
            last = max(i for i, o in enumerate(done) if o[1] == stream and o[0] in ("launch", "copy"))
            assert any(o[0] == "sync" and o[1] == stream for o in done[last:]), (kind, at, stream)
        e.stub.stub_reset()
        assert e.draft_block(8) == -2, (kind, at)          # DEER_ESTATE
        assert call() == 0 and e.draft_block(8) == 0
        checked += 1
print(checked)
""")
    assert int(out) >= (35 if "40" in prompts else 20), out


def test_the_second_set_of_buffers_is_no_larger_than_the_contexts_ask_for(tmp_path):
    """What the set adds to the workspace (drafters of 4 layers have it, of 3 not): for sequences of 64 slots less than a third of
    what 64 row tiles need, which is the most."""
    got = eval(run_script(tmp_path, """
import deer_inputs as di
def workspace(layers, batch, max_seq):
    d = di.scaled(di.DRAFTER_05B, n_layers=layers)
    return HostEngine.binding.query_sizes(HostEngine.binding.init_params(di.CONFIGS["qwen3_8b"]["target"], d, batch, max_seq, 32, 5)).workspace
print([workspace(4, b, s) - workspace(3, b, s) for b, s in ((1, 64), (1, 512), (1, 2048), (1, 8192), (16, 2048))])
"""))
    assert got[0] < got[1] < got[2] <= got[3] == got[4] and 3 * got[0] < got[3] < 160e6, got


def test_timed_passes_take_the_forms_of_the_others(tmp_path):
    """While launches are timed the drafter's passes use the target's buffers, which hold more partial sums: the same kernels and
    grids all the same, for drafters as wide as targets are."""
    out = run_script(tmp_path, """
import deer_inputs as di
t = di.CONFIGS["tiny"]["target"]
for d, hq, hkv, hd, ff in ((896, 14, 2, 64, 4864), (2560, 32, 8, 128, 9728), (4096, 32, 8, 128, 12288), (5120, 40, 8, 128, 25600), (8192, 64, 8, 128, 28672)):
    e = HostEngine(t, di.ModelShape(4, d, hq, hkv, hd, ff, t.vocab, rope_base=1e4), 1, 2112)
    for n in (20, 70, 130, 200, 400, 500, 900, 1024, 1500, 2048):
        runs = []
        for timed in (0, 1):
            assert e.lib.deer_debug_profile(e.ctx, timed) == 0
            e.stub.stub_reset()
            assert e.prefill([[3] * n]) == 0
            runs.append(e.launches())
        assert runs[0] == runs[1], (d, n)
print("checked")
""")
    assert out == "checked\n"
