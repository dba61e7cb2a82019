"""GPU parity of blocked GEMMs whose last blocks are cut into pieces of k-steps (more blocks than compute units, but not a
multiple): pieces that end inside a block, that span two, blocks of two to nine pieces, in gate/up, residual GEMMs
and the LM head, against the weight-streaming kernels.  test_host_routes.py checks that these shapes run so."""
import numpy as np
import pytest

import deer_inputs as di
from gpu_common import gpu_available
from test_gpu_block_forms import _compare, _engine, _outputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# d = 1152: 72 k-steps; gate/up has 131 column blocks of 128, QKV 11, the residual GEMMs 9, the LM head 129
SHAPE = dict(d_model=1152, n_q_heads=18, n_kv_heads=2, head_dim=64, d_ff=8384, vocab=16512)
PROMPTS = [([202], 5), ([130, 40, 33, 1, 60], 32), ([3840], 32)]   # row blocks: 2 (262 blocks of gate/up); 3, LM head 2 (258 blocks); 30


def shape():
    return di.ModelShape(2, rope_base=1e4, **SHAPE)


@pytest.mark.parametrize("lens,k", PROMPTS)
def test_pieces_agree_with_the_streaming_kernels(lens, k):
    import torch
    t, d = shape(), di.ModelShape(1, 384, 6, 3, 64, 640, SHAPE["vocab"], rope_base=1e4)
    eng = _engine(t, d, len(lens), -(-(max(lens) + 64) // 64) * 64, torch)
    prompts = [di.prompt_ids(t.vocab, n, seq=b) for b, n in enumerate(lens)]
    blocks = torch.from_numpy(np.random.default_rng(1).integers(0, t.vocab, (len(lens), k)).astype(np.int32)).cuda()
    out = {}
    for mode in (0, 128):
        eng.debug_gemm_tiled(mode)
        _outputs(eng, prompts, k, blocks, torch)
        out[mode] = _outputs(eng, prompts, k, blocks, torch)
    _compare(out[0], out[128])
    eng.close()
