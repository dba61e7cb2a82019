"""GPU parity of the per-head block attention by the number of key ranges its heads are cut into: one (no merge), up to eight
(merged by the short code), up to sixteen (loads in one or two rounds) and more (eight at a time), per head dim, with ranges of unequal length and
waves without a key tile.  One layer behind seeded stand-in keys and values, against the oracle; the launches' grids say which
number of ranges ran (test below, without a GPU)."""
import os
import sys

import numpy as np
import pytest

import deer_inputs as di
from oracle import deer_oracle as O
from gpu_common import StoredWeights, fill_seeded_cache, gpu_available, make_engine, make_pair

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "hip_stub"))
from host_engine import run_script   # noqa: E402

# q heads, kv heads, head dim, prefix length, key ranges
CASES = [(4, 2, 32, 70, 1), (4, 2, 32, 2000, 5), (4, 2, 32, 16000, 14),
         (14, 2, 64, 470, 1), (14, 2, 64, 1023, 5), (14, 2, 64, 4096, 10),
         (8, 2, 128, 40, 1), (8, 2, 128, 900, 4), (8, 2, 128, 2500, 10), (8, 2, 128, 6000, 16), (32, 8, 128, 4096, 8),
         (4, 2, 32, 50000, 23), (14, 2, 64, 50000, 18), (8, 2, 128, 60000, 32)]


def _shape(hq, hkv, hd):
    return di.ModelShape(1, 256, hq, hkv, hd, 256, 1024, rope_base=1e4)


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("hq,hkv,hd,n,ranges", CASES)
def test_ranges_against_the_oracle(hq, hkv, hd, n, ranges):
    import torch
    t, k = _shape(hq, hkv, hd), 9
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(t, di.DRAFTER_SEED, "bf16")
    size = -(-(n + 64) // 64) * 64
    eng = make_engine(t, t, wt, wd, 1, size, k)
    pair = make_pair(t, t, wt, wd, size)
    pair.x = [0] * (n - 1) + [7]
    fill_seeded_cache(eng, torch, 0, t, 0, n - 1, pair.tc)
    fill_seeded_cache(eng, torch, 1, t, 0, n, pair.dc)
    eng.set_prefilled([n], [7])
    eng.draft_block(k, 0.0, 0)
    zd = pair.draft_logits(k)
    assert np.abs(eng.debug_get_logits(1, k)[0] - zd).max() < 2e-3   # as for the tiny shapes elsewhere
    block = [int(v) for v in np.random.default_rng(n).integers(0, t.vocab, k)]
    res = O.deer_iteration(pair, k, 0.0, None, draft_override=block)
    eng.verify_block(k, 0.0, torch.tensor([block], dtype=torch.int32, device="cuda"))
    assert np.abs(eng.debug_get_logits(0, k)[0] - res["target_logits"]).max() < 2e-3
    eng.close()


def test_the_cases_run_with_the_ranges_they_name(tmp_path):
    got = eval(run_script(tmp_path, f"""
import deer_inputs as di
out = []
for hq, hkv, hd, n, _ in {CASES}:
    t = di.ModelShape(1, 256, hq, hkv, hd, 256, 1024, rope_base=1e4)
    e = HostEngine(t, t, 1, -(-(n + 64) // 64) * 64)
    e.set_prefilled([n], [7])
    e.stub.stub_reset()
    assert e.draft_block(9) == 0
    out += [g[0] // hq for name, g in e.launches() if "k_attn_head" in name]
print(out)
"""))
    assert got == [c[4] for c in CASES], got


def test_few_heads_over_long_contexts_keep_a_workgroup_per_head(tmp_path):
    """As many ranges as a wave's share of 12 key tiles asks for, up to 32 and to one workgroup per compute unit."""
    got = eval(run_script(tmp_path, """
import deer_inputs as di
out = []
for hq, hkv, hd, n in ((4, 2, 32, 64000), (14, 2, 64, 32768), (14, 2, 64, 55200), (14, 2, 64, 55400), (8, 2, 128, 98200), (8, 2, 128, 98400)):
    t = di.ModelShape(1, 256, hq, hkv, hd, 256, 1024, rope_base=1e4)
    e = HostEngine(t, t, 1, -(-(n + 64) // 64) * 64)
    e.set_prefilled([n], [7])
    e.stub.stub_reset()
    assert e.draft_block(9) == 0
    out.append(sum(g[0] // hq for name, g in e.launches() if "k_attn_head" in name))
print(out)
"""))
    assert got == [26, 16, 18, 0, 32, 0], got
