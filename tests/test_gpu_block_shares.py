"""GPU parity of the sums of a blocked GEMM's K shares: two (only the other one is read), three and four at a time, whole
and with a remainder, for row blocks of four, three and one row tiles, against the weight-streaming kernels."""
import numpy as np
import pytest

import deer_inputs as di
from gpu_common import gpu_available
from test_gpu_block_forms import _compare, _engine, _outputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("lens", [[500], [450], [290, 33, 190]])   # 16, 15 and 17 row tiles
@pytest.mark.parametrize("k", [32, 31])
def test_shares_agree_with_the_streaming_kernels(lens, k):
    import torch
    t = di.ModelShape(2, 1408, 18, 6, 64, 1664, 1152, rope_base=1e4)   # 88, 72 and 104 k-steps
    d = di.ModelShape(1, 384, 6, 3, 64, 640, 1152, rope_base=1e4)      # 24, 24 and 40
    eng = _engine(t, d, len(lens), 576, torch)
    prompts = [di.prompt_ids(t.vocab, n, seq=b) for b, n in enumerate(lens)]
    blocks = torch.from_numpy(np.random.default_rng(1).integers(0, t.vocab, (len(lens), k)).astype(np.int32)).cuda()
    eng.debug_gemm_tiled(0)
    _outputs(eng, prompts, k, blocks, torch)
    want = _outputs(eng, prompts, k, blocks, torch)
    eng.debug_gemm_tiled(128)
    for shares in (2, 3, 4, 5, 6, 7, 8):
        print("shares", shares, flush=True)
        eng.debug_gemm_block(2, 4, shares)
        _compare(want, _outputs(eng, prompts, k, blocks, torch))
    eng.close()
