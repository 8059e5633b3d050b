"""Which launches of the bf16 GEMM take 256-column tiles (host arithmetic: this runs without a GPU)."""
import pytest

import paper_2602_00182_amd as d


@pytest.mark.parametrize("M,K,N,rows", [(3302, 4096, 6144, 160), (700, 4096, 6144, 128), (1500, 14336, 4096, 128), (2000, 1024, 11264, 192),
                                        (4096, 4096, 28672, 256), (300, 1088, 28672, 160), (351, 2048, 11264, 128),
                                        (552, 14336, 11264, 128)])
def test_taken(M, K, N, rows):
    assert d.det_gemm_wide_rows(M, N, K) == rows


# Measured faster in the other tilings, whose last row of tiles is nearly empty (42 against 62 us in the first).
@pytest.mark.parametrize("M,K,N", [(258, 4416, 11264), (267, 4096, 11264), (519, 2048, 6144), (541, 1152, 6144), (800, 2048, 4608),
                                   (1047, 2048, 3584), (1052, 4096, 28672), (514, 2048, 22528), (264, 14336, 22272)])
def test_left_where_few_rows_follow_whole_tiles(M, K, N):
    assert d.det_gemm_wide_rows(M, N, K) == 0


# 128-column packings, many rounds: measured 4 to 15 % faster there than in tiles of 128 rows
@pytest.mark.parametrize("M,K,N,rows", [(1590, 3328, 25088, 0), (1338, 1792, 29184, 0), (1398, 11648, 28928, 256), (1109, 13824, 27904, 160),
                                        (1102, 14336, 28672, 192)])
def test_few_rows_more_of_wide_packings(M, K, N, rows):
    assert d.det_gemm_wide_rows(M, N, K) == rows


def test_outside_its_range():
    for M, N, K in [(255, 28672, 4096), (4096, 28672 + 128, 4096), (4096, 28672, 960), (0, 256, 4096), (4096, 100, 4096), (4096, 256, 1000)]:
        assert d.det_gemm_wide_rows(M, N, K) == 0
