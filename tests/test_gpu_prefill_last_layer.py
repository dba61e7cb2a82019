"""GPU parity of prompts through models of five layers, the shortest whose prefill ends with the K and V rows of the last
layer: every head width, numbers of K and V columns that are and are not whole column groups, passes of one to eleven row
tiles (narrow, small-workgroup, streaming and blocked QKV), a mixture, against the oracle; and (on the CPU) what is launched."""
import os
import sys

import numpy as np
import pytest

import deer_inputs as di
from gpu_common import StoredWeights, gpu_available, make_engine, make_pair

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub"))
from host_engine import run_script   # noqa: E402

TOL = 2e-3   # logits, as for the small shapes elsewhere
SHAPES = {
    "hd64": di.ModelShape(5, 384, 6, 3, 64, 640, 1024, rope_base=1e4),
    "hd128": di.ModelShape(5, 1152, 3, 1, 128, 640, 1024, rope_base=1e4),
    "hd32": di.ModelShape(5, 256, 4, 2, 32, 512, 1024, rope_base=1e4),
    "half a column group": di.ModelShape(5, 256, 2, 1, 32, 512, 1024, rope_base=1e4),   # runs whole
    "mixture": di.ModelShape(5, 256, 4, 2, 32, 0, 1024, n_experts=8, top_k=2, d_ff_expert=128, rope_base=1e4),
}


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("name", SHAPES)
def test_prompts_through_five_layers(name):
    import torch
    t, k = SHAPES[name], 8
    d = di.ModelShape(5, 256, 4, 2, 32, 512, 1024, rope_base=1e4)
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(d, di.DRAFTER_SEED, "bf16")
    eng = make_engine(t, d, wt, wd, 3, 384, k)
    for lens in ([6], [70], [300, 33, 1]):
        prompts = [di.prompt_ids(t.vocab, n, seq=300 + b) for b, n in enumerate(lens)]
        blocks = np.random.default_rng(4).integers(0, t.vocab, (len(lens), k)).astype(np.int32)
        eng.prefill(prompts)
        eng.draft_block(k, 0.0, 0)
        zd = eng.debug_get_logits(1, k)
        eng.verify_block(k, 0.0, torch.from_numpy(blocks).cuda())
        zt = eng.debug_get_logits(0, k)
        for b, prompt in enumerate(prompts):
            pair = make_pair(t, d, wt, wd, 384)
            pair.prefill(prompt)
            assert np.abs(zd[b] - pair.draft_logits(k)).max() < TOL, (lens, b)
            pair.dc.truncate(len(prompt))
            assert np.abs(zt[b] - pair.verify_logits([int(v) for v in blocks[b]])).max() < TOL, (lens, b)
    eng.close()


def test_the_last_layer_ends_with_its_kv_rows(tmp_path):
    """Five launches per layer, one for the last: over the columns of K and V alone.  A block's passes, which leave logits, and
    models of fewer layers run whole."""
    out = run_script(tmp_path, """
import deer_inputs as di
def names(t, call):
    e = HostEngine(t, t, 1, 256)
    assert e.set_prefilled([40], [3]) == 0
    e.stub.stub_reset()
    assert call(e) == 0
    return [(n, g) for n, g in e.launches() if "k_pass_begin" not in n and "k_rowstat" not in n and "k_draft" not in n]
for layers in (4, 5, 6):
    t = di.ModelShape(layers, 1152, 9, 3, 128, 640, 1024, rope_base=1e4)     # Q 9, K and V 6 column groups of 128
    a = names(t, lambda e: e.prefill([[3] * 70]))
    per = 5 * layers if layers < 5 else 5 * (layers - 1) + 1
    assert len(a) == 2 * per, (layers, len(a))
    if layers >= 5:
        for p in (a[:per], a[per:]):
            assert p[-1][1][0] < p[0][1][0], p    # fewer column groups than the first layer's QKV projection
    assert len(names(t, lambda e: e.draft_block(8))) == 5 * layers + 1
m = di.ModelShape(5, 256, 4, 2, 32, 0, 1024, n_experts=8, top_k=2, d_ff_expert=128, rope_base=1e4)
a = names(m, lambda e: e.prefill([[3] * 70]))
assert sum("k_moe_combine" in n for n, _ in a) == 8 and sum("k_attn" in n and "merge" not in n for n, _ in a) == 8, a
print("checked")
""")
    assert out == "checked\n"
