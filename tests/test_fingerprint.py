"""det_fingerprint() names the launch geometry that row counts select (host arithmetic: this runs without a GPU)."""
import hashlib
import re

import paper_2602_00182_amd as d


def tag():
    return re.search(r" (tiles-\d+)\((.*)\)$", d.det_fingerprint()).groups()


def geometry():
    """Digest of the tiles of both GEMMs over launches on every side of the rules."""
    h = hashlib.sha256()
    for N in (16, 48, 640, 1024, 1472, 2048, 2112, 2624, 3072, 3200, 4096, 4160, 5120, 5440, 6144, 6848, 8192, 11264, 12800, 20480, 28672, 32000):
        for K in (64, 2048, 4096, 14336):
            for M in list(range(1, 300)) + list(range(300, 1100, 25)) + [1962, 3302, 4096, 4939]:
                h.update(repr((d.det_gemm_tile(M, N, K), d.det_qgemm_tile(M, N, K))).encode())
    return h.hexdigest()[:16]


def test_a_changed_geometry_has_a_new_revision():
    """Two builds that cut launches differently must not name themselves alike: with a new digest goes a new revision."""
    assert (tag()[0], geometry()) == ("tiles-9", "d27915d872e373f5")


def test_changed_forms_have_a_new_revision():
    """The forms that no query names are stated in the tag, from the constants the code takes: with a new text goes a new revision."""
    assert (tag()[0], hashlib.sha256(tag()[1].encode()).hexdigest()[:16]) == ("tiles-9", "16f713d2eb7ab8ef")
    for form in ("few@4rows", "norm@3rows", "norm128@4rows", "mid@48rows|32rows", "rows8@16rows", "walk@256wg", "few@16pairs", "turn@32chunks"):
        assert form in re.split("[(,;:)]", tag()[1]), form


def test_the_tag_states_the_rules():
    rules = tag()[1]
    first = lambda N, K, columns, lo=1, hi=300: next(M for M in range(lo, hi) if d.det_gemm_tile(M, N, K)[1] == columns)
    assert "n64@m65|m64r64|m161" in rules
    assert first(3072, 2048, 64) == 65                  # 16-column packings
    assert first(8192, 4096, 64) == 113 and d.det_gemm_tile(113, 8192, 4096)[0] <= 64    # 32-column ones: where tiles of at most 64 rows pay
    assert first(6144, 4096, 64, 129) == 161                                            # and in higher tiles from here on
    assert "rowcut8" in rules and d.det_gemm_tile(130, 4096, 14336) == (40, 64)
    assert "reads@m96|m192" in rules and [d.det_gemm_tile(M, 2624, 11904)[1] for M in (95, 96)] == [16, 64]
    assert "32x64+64x64@768wg,64x128" in rules
    tiles = lambda M, N, rows, columns: -(-M // rows) * (N // columns)
    for M, N in [(1536, 2048), (192, 4096), (256, 11264), (500, 3072)]:
        rows, columns = d.det_qgemm_tile(M, N, 4096)
        assert columns == 64 and tiles(M, N, rows, columns) <= 768
    for M, N in [(1537, 2048), (300, 11264), (4096, 6144)]:
        assert d.det_qgemm_tile(M, N, 4096) == (64, 128) and tiles(M, N, 64, 64) > 768
