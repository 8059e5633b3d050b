"""RMSNorm, plain and quantized, at the lengths where a thread gets room for more vectors, one vector or one block either side; bits against
the oracle."""
import numpy as np
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, down_bf16, step, up_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [8, 64, 1984, 2040, 2048, 2056, 2112, 4032, 4088, 4096, 4104, 4160, 8128, 8192, 8200, 8256, 16320, 16376, 16384])
def test_bits_match_oracle(orc, H):
    import paper_2602_00182_amd as d
    M = 3
    x = ds.normal_bf16(ds.tensor_seed(3, 40) + H, (M, H))
    w = ds.normal_bf16(ds.tensor_seed(3, 41) + H, (H,), 0.1, 1.0)
    step(f"rmsnorm H={H}")
    y = torch.full((M + 1, H), 7.0, dtype=torch.bfloat16, device=DEV)
    d.det_rmsnorm(up_bf16(x), up_bf16(w), y[:M], 1e-5)
    torch.cuda.synchronize()
    want = orc.rmsnorm(x, w, 1e-5)
    assert np.array_equal(down_bf16(y[:M].contiguous()), want) and (y[M] == 7).all()
    if H % 64:
        return
    codes = torch.full((M + 1, H), 99, dtype=torch.int8, device=DEV)
    scales = torch.full((d.det_quant_act_scales_bytes(M, H) // 4,), 7.0, dtype=torch.float32, device=DEV)
    d.det_rmsnorm_quant_q8(up_bf16(x), up_bf16(w), codes[:M], scales, 1e-5)
    torch.cuda.synchronize()
    p, s = orc.quant_a8(want)
    assert np.array_equal(codes[:M].cpu().numpy(), p) and (codes[M] == 99).all()
    assert np.array_equal(scales.cpu().numpy().reshape(H // 64, -1)[:, :M].T, s)
