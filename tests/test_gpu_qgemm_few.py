"""The quantized GEMM of at most four rows on the GPU: blocks and batches of K that do not come out even, the longest rows whose
weights fit, every epilogue, and operands whose scale products are subnormal; bytes against the oracle or the unfused steps."""
import numpy as np
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, down_bf16, step, up_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    import paper_2602_00182_amd as d
    return d


def packed_and_codes(d, orc, M, K, N, scale_a=1.0, scale_w=0.02, seed=0):
    a = ds.normal_bf16(ds.tensor_seed(6, 700) + seed, (M, K), scale_a, 0.0)
    w = ds.normal_bf16(ds.tensor_seed(6, 701) + seed, (K, N), scale_w, 0.0)
    codes, scales = d.quant_activations(up_bf16(a))
    acc, out = orc.qgemm_w4a8(*orc.quant_a8(a), *orc.quant_w4(w))
    return d.quant_pack_weight(up_bf16(w)), codes, scales, acc, out


# K: one block; fewer blocks than a batch, than producers; a last batch and a last group of one to three blocks; the longest that fits
# for the row count in tiles of 16 columns (LDS: 560 + 64 M bytes a block of 158 KB), and one block more (the general kernel)
@pytest.mark.parametrize("M,K,N", [(1, 64, 16), (4, 64, 48), (2, 192, 16), (3, 320, 32), (1, 64 * 33, 16), (4, 64 * 31, 48), (2, 64 * 67, 2048), (3, 64 * 130, 16),
                                   (1, 64 * 259, 16), (1, 64 * 260, 16), (4, 64 * 198, 16), (4, 64 * 199, 16), (2, 64 * 235, 16), (3, 64 * 215, 16), (3, 64 * 216, 16),
                                   (1, 4096, 6144), (4, 64 * 70, 6144), (3, 2048, 11264), (4, 64 * 65, 11264), (2, 64 * 9, 11264)])
def test_bytes_match_oracle(d, orc, M, K, N):
    packed, codes, scales, acc, out = packed_and_codes(d, orc, M, K, N, seed=K + N)
    c = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    cf = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
    step(f"few rows M={M} K={K} N={N}")
    d.det_qgemm_w4a8(codes, scales, packed, c, N)
    d.det_qgemm_w4a8(codes, scales, packed, cf, N)
    torch.cuda.synchronize()
    assert np.array_equal(cf.cpu().numpy().view(np.uint32), acc.view(np.uint32))
    assert np.array_equal(down_bf16(c), out)


@pytest.mark.parametrize("M", [1, 4])
def test_subnormal_scale_products(d, orc, M):
    """d * s around and below the smallest normal number: products are rounded there as anywhere."""
    packed, codes, scales, acc, _ = packed_and_codes(d, orc, M, 640, 64, scale_a=2.0 ** -60, scale_w=2.0 ** -64, seed=M)
    cf = torch.full((M, 64), float("nan"), dtype=torch.float32, device=DEV)
    step(f"few rows, subnormal products M={M}")
    d.det_qgemm_w4a8(codes, scales, packed, cf, 64)
    torch.cuda.synchronize()
    assert np.array_equal(cf.cpu().numpy().view(np.uint32), acc.view(np.uint32)) and np.abs(acc).max() > 0


@pytest.mark.parametrize("M,K,N", [(1, 576, 2048), (3, 2112, 6144), (4, 320, 11264)])
def test_epilogues_equal_unfused_bytes(d, orc, M, K, N):
    packed, codes, scales, _, plain = packed_and_codes(d, orc, M, K, N, seed=N)
    r = ds.normal_bf16(ds.tensor_seed(6, 702) + N, (M, N), 1.0, 0.0)
    wide = torch.full((M, N + 8), float("nan"), dtype=torch.bfloat16, device=DEV)
    wide[:, :N] = up_bf16(r)
    step(f"few rows, residual in strided rows and in place M={M} K={K} N={N}")
    d.det_qgemm_w4a8_residual(codes, scales, packed, wide[:, :N], wide[:, :N], N)
    y = torch.full((M, N // 2), float("nan"), dtype=torch.bfloat16, device=DEV)
    w = ds.normal_bf16(ds.tensor_seed(6, 703) + N, (K, N), 0.02, 0.0)
    gu = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    d.det_qgemm_w4a8_swiglu(codes, scales, d.quant_pack_gate_up(up_bf16(w)), y, N // 2)
    d.det_qgemm_w4a8(codes, scales, d.quant_pack_weight(up_bf16(w)), gu, N)
    want = torch.empty_like(y)
    d.det_swiglu(gu[:, :N // 2].contiguous(), gu[:, N // 2:].contiguous(), want)
    torch.cuda.synchronize()
    assert np.array_equal(down_bf16(wide[:, :N].contiguous()), orc.residual(r, plain)) and torch.isnan(wide[:, N:]).all()
    assert np.array_equal(down_bf16(y), down_bf16(want))
