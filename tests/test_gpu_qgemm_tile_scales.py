"""Scale products of the quantized GEMM's tiles and of its kernel of fewer rows: subnormal, zero, infinite and NaN scales, odd and even counts of blocks.  A row's bits
are those of the row by itself, whose products are taken by vector multiplies: in the kernel of few rows, which packings of 128 columns
are too wide for, so that of those the single row's matrix is cut into narrower ones."""
import numpy as np
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    import paper_2602_00182_amd as d
    return d


# tiles of 32 x 64, 64 x 64 and 64 x 128; packings of 16, 32, 64 and 128 columns
@pytest.mark.parametrize("M,K,N", [(97, 64 * 9, 4096), (250, 64, 11264), (191, 64 * 8, 11264), (300, 64 * 3, 4096), (1000, 64 * 5, 6144), (131, 64 * 2, 28672),
                                   # fewer rows: one, two, three to four, eight and more row blocks of a wave, stages that do not come out even
                                   (13, 64 * 7, 28672), (30, 64 * 5, 28672), (61, 64 * 3, 28672), (80, 64 * 2, 28672), (14, 64 * 5, 11264), (41, 64 * 3, 11264),
                                   (70, 64 * 3, 4096), (300, 64 * 3, 5072)])
def test_rows_equal_single_rows(d, M, K, N):
    a = ds.normal_bf16_torch(ds.tensor_seed(6, 820) + K + N, (M, K), 1.0, 0.0, DEV)
    for i, factor in enumerate((2.0 ** -100, 2.0 ** -120, 0.0, float("inf"), float("nan"))):
        a[i, :64] *= factor
    a[5, 3] = float("inf")
    a[6, 63] = float("nan")
    a[7] = 3.0e38
    w = ds.normal_bf16_torch(ds.tensor_seed(6, 821) + K + N, (K, N), 0.02, 0.0, DEV)
    w[:, 1] *= 2.0 ** -30  # subnormal products with the rows that have small scales
    w[:, 2] = 0
    codes, scales = d.quant_activations(a)
    packed = d.quant_pack_weight(w)
    c = torch.full((M, N), 7.0, dtype=torch.float32, device=DEV)
    step(f"tile scales M={M} K={K} N={N}")
    d.det_qgemm_w4a8(codes, scales, packed, c, N)
    torch.cuda.synchronize()
    assert torch.isnan(c[3]).any() and (c[2, :].abs().sum() if K == 64 else torch.zeros(())) == 0
    parts = [(0, N)] if d.det_qgemm_tile(1, N, K)[1] < 128 else [(n, n + 4096) for n in range(0, N, 4096)]
    assert parts[-1][1] == N
    narrow = [(n0, n1, d.quant_pack_weight(w[:, n0:n1].contiguous())) for n0, n1 in parts]
    for i in (*range(8), *(i for i in (15, 16, 31, 32, 63, 64) if i < M), M - 1):
        codes1, scales1 = d.quant_activations(a[i:i + 1].contiguous())
        one = torch.full((1, N), 7.0, dtype=torch.float32, device=DEV)
        for n0, n1, part in narrow:
            assert d.det_qgemm_tile(1, n1 - n0, K)[1] <= 64
            d.det_qgemm_w4a8(codes1, scales1, part, one[:, n0:n1], n1 - n0)
        assert np.array_equal(one.cpu().numpy().view(np.uint32)[0], c[i].cpu().numpy().view(np.uint32)), i
