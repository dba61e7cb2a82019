"""GPU parity of prompts that take several passes: sequences that continue in the next pass, passes that are full of tiles
long before they are full of rows, passes of more than 128 tiles (batches over 64), against the oracle; and the caches
against those of the same prompts one at a time (one pass each), also for a mixture."""
import numpy as np
import pytest

import deer_inputs as di
from gpu_common import StoredWeights, gpu_available, make_engine, make_pair

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

TOL = 2e-3         # logits, as for the tiny shapes elsewhere
CACHE_REL = 2e-3   # caches of two batches: the sums' order differs, and with it a bf16 value near the middle of two now and then


def n_tiles(lens):
    return sum(-(-n // 32) for n in lens)


MIX = di.ModelShape(2, 256, 4, 2, 32, 0, 1024, n_experts=8, top_k=2, d_ff_expert=128, rope_base=1e4)
rng = np.random.default_rng(8)
CASES = {
    # 4498 rows in 144 tiles: the third sequence goes on in the second pass, in the middle of a row tile of the GEMMs
    "long": (di.CONFIGS["tiny"]["target"], [1000, 37, 2500, 900, 61], 5, 2560, [1, 2, 4]),
    # two whole passes of 128 tiles and a third one
    "full": (di.CONFIGS["tiny"]["target"], [4096, 2049, 2048], 3, 4160, []),
    # 64 sequences of two and three tiles: passes of 128 tiles, about 2600 rows
    "short": (di.CONFIGS["tiny"]["target"], [33 + (11 * b) % 50 for b in range(64)], 64, 128, [0, 31, 50, 51, 63]),
    # passes of up to 180 tiles
    "wide": (di.CONFIGS["tiny"]["target"], [int(v) for v in rng.integers(1, 120, 90)], 90, 192, [0, 44, 71, 72, 89]),
    "mixture": (MIX, [2500, 3, 2100], 3, 2560, [1]),
}


@pytest.mark.parametrize("name", CASES)
def test_prompts_of_several_passes(name):
    import torch
    t, lens, max_batch, max_seq, check = CASES[name]
    assert n_tiles([n - 1 for n in lens]) > max(128, 2 * max_batch)
    d, k = di.CONFIGS["tiny"]["drafter"], 8
    wt, wd = StoredWeights(t, di.TARGET_SEED, "bf16"), StoredWeights(d, di.DRAFTER_SEED, "bf16")
    eng = make_engine(t, d, wt, wd, max_batch, max_seq, k)
    prompts = [di.prompt_ids(t.vocab, n, seq=200 + b) for b, n in enumerate(lens)]
    eng.prefill(prompts)
    caches = []
    for m, shape in enumerate((t, d)):   # [K, V][layer][sequence][head][32-slot block]...
        lay = eng.get_kv_layout(m)
        caches.append(eng._kv[m][: 4 * shape.n_layers * lay.layer_stride].view(torch.bfloat16).view(2, shape.n_layers, max_batch, shape.n_kv_heads, max_seq // 32, -1))
    got = [c.clone() for c in caches]
    eng.draft_block(k, 0.0, 0)
    zd = eng.debug_get_logits(1, k)
    blocks = np.random.default_rng(9).integers(0, t.vocab, (len(lens), k)).astype(np.int32)
    eng.verify_block(k, 0.0, torch.from_numpy(blocks).cuda())
    zt = eng.debug_get_logits(0, k)
    for b in check:
        pair = make_pair(t, d, wt, wd, max_seq)
        pair.prefill(prompts[b])
        assert np.abs(zd[b] - pair.draft_logits(k)).max() < TOL, b
        pair.dc.truncate(len(prompts[b]))
        assert np.abs(zt[b] - pair.verify_logits([int(v) for v in blocks[b]])).max() < TOL, b
    for b, prompt in enumerate(prompts):   # alone, in sequence slot 0: whole 32-slot blocks of rows that both have
        eng.prefill([prompt])
        for m, (c, g) in enumerate(zip(caches, got)):
            n = (len(prompt) - 1 + m) // 32
            if n:
                a, w = g[:, :, b, :, :n].float(), c[:, :, 0, :, :n].float()
                off = float((a - w).norm() / w.norm())
                assert off < CACHE_REL, (b, m, off)
    eng.close()
