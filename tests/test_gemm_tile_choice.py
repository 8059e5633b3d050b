"""The tiles that launches of the bf16 GEMM are cut into (host arithmetic: this runs without a GPU)."""
import pytest

import paper_2602_00182_amd as d


# Rows dealt out in half blocks of 8 over as many tiles as fill the chip, where that does not make more XCDs read each weight.
@pytest.mark.parametrize("M,K,N,rows", [(130, 14336, 4096, 40), (201, 14336, 4096, 56), (400, 14336, 4096, 104), (173, 4224, 2816, 40),
                                        (335, 10368, 1792, 40), (255, 11392, 1216, 24)])
def test_half_blocks_fill_the_chip(M, K, N, rows):
    assert d.det_gemm_tile(M, N, K) == (rows, 64)


# Measured 10 to 28 % faster in the tiles of whole 16-row blocks: their columns are an odd number, or twice one, of 64, so that each
# tile of rows more has another XCD read the weights again.
@pytest.mark.parametrize("M,K,N,rows", [(123, 11904, 2624, 32), (98, 10496, 3008, 32), (203, 11904, 2624, 48), (202, 9728, 2368, 48),
                                        (147, 11136, 2112, 32), (139, 6400, 2624, 32), (93, 12800, 3200, 32)])
def test_half_blocks_do_not_add_reads_of_the_weights(M, K, N, rows):
    assert d.det_gemm_tile(M, N, K) == (rows, 64)


# Measured 6 to 45 % faster in tiles of the packing's width, which read the weights once: 64-column tiles of 16 or 32 rows would have
# three to six XCDs read them.  And the nearest that are faster in those.
@pytest.mark.parametrize("M,K,N,rows,columns", [(72, 8192, 3200, 256, 16), (88, 3584, 2624, 256, 16), (81, 11904, 2624, 256, 16), (68, 4864, 2496, 256, 16),
                                                (83, 3456, 3776, 256, 16), (72, 14080, 5440, 256, 32), (80, 7936, 5312, 256, 32),
                                                (72, 3072, 3072, 16, 64), (89, 7424, 2816, 24, 64), (85, 7040, 2432, 16, 64), (66, 2944, 4608, 24, 64),
                                                (120, 2816, 6848, 64, 64)])
def test_few_rows_take_tiles_that_read_the_weights_seldom(M, K, N, rows, columns):
    assert d.det_gemm_tile(M, N, K) == (rows, columns)


def test_tiles_hold_every_row_in_whole_half_blocks():
    for N in (16, 48, 64, 576, 2048, 2112, 2624, 3072, 4096, 6144, 8192, 11264, 28672):
        for M in list(range(1, 600)) + [1000, 1024, 4096, 4097]:
            rows, columns = d.det_gemm_tile(M, N, 2048)
            assert rows % 8 == 0 and 16 <= rows <= 256 and N % columns == 0


def test_unsupported_shapes_have_no_tile():
    for M, N, K in [(0, 4096, 4096), (1, 100, 4096), (1, 4096, 1000), (-1, 4096, 4096)]:
        assert d.det_gemm_tile(M, N, K)[0] == 0
