"""The tiles that launches of the quantized GEMM are cut into (host arithmetic: this runs without a GPU)."""
import pytest

import paper_2602_00182_amd as d


# The smallest tile of which the chip holds all, from the row counts where its chain over K is the shorter one
@pytest.mark.parametrize("M,K,N,tile", [(80, 4096, 4096, (256, 16)), (96, 4096, 4096, (32, 64)), (192, 4096, 4096, (32, 64)), (768, 4096, 4096, (64, 64)),
                                        (64, 2048, 11264, (32, 64)), (128, 2048, 11264, (32, 64)), (256, 2048, 11264, (64, 64)), (300, 2048, 11264, (64, 128)),
                                        (1536, 64, 2048, (64, 64)), (1537, 64, 2048, (64, 128)), (1962, 2048, 2048, (64, 128)), (700, 64, 3072, (64, 64)),
                                        (64, 4096, 28672, (256, 128)), (96, 4096, 28672, (64, 128))])
def test_choice(M, K, N, tile):
    assert d.det_qgemm_tile(M, N, K) == tile


# From one row more than the whole row blocks at which the tiles of 64 columns and the packing's own meet
@pytest.mark.parametrize("last,K,N,columns", [(89, 4096, 4096, 16), (64, 4096, 6144, 32), (64, 14336, 5120, 32), (64, 2048, 8192, 32), (48, 2048, 11264, 64),
                                              (48, 5632, 12800, 64)])
def test_lines_of_the_small_tiles(last, K, N, columns):
    assert d.det_qgemm_tile(last, N, K) == (256, columns) and d.det_qgemm_tile(last + 1, N, K) == (32, 64)


def test_every_launch_has_a_tile_of_whole_slabs():
    for N in list(range(16, 2049, 16)) + [3072, 4160, 4608, 5632, 6144, 8192, 11008, 11264, 20480, 22528, 28672, 32000]:
        for M in list(range(1, 300)) + [385, 500, 768, 1000, 1962, 3302, 4096, 70000, 65535 * 64 + 1]:
            rows, columns = d.det_qgemm_tile(M, N, 64)
            slab = d.det_qgemm_tile(1, N, 64)[1]
            assert rows >= 16 and N % columns == 0 and columns % slab == 0, (M, N, rows, columns)


def test_unsupported_shapes_have_no_tile():
    for M, N, K in [(0, 4096, 4096), (1, 100, 4096), (1, 4096, 1000), (-1, 4096, 4096)]:
        assert d.det_qgemm_tile(M, N, K)[0] == 0
