"""The bf16 GEMM's 256-column tiles: every row must have the bytes the one-tiling form (det_gemm_bf16_fixed_tile) gives it,
and each epilogue those of a call of few rows."""
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, step, up_bf16

pytestmark = pytest.mark.gpu

K = 1088  # the smallest multiple of 64 above the rule's bound that is no multiple of 128


@pytest.fixture(scope="module")
def d():
    import paper_2602_00182_amd as d
    return d


def bits(t):
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)


# every tile height, packings of 16, 32, 64 and 128 columns, tiles of one row, ragged and whole; K of 34, 32 and 64 steps
@pytest.mark.parametrize("M,N,K", [
    (2177, 3072, K),       # 128 rows, 32 columns a slab
    (3302, 2048, 1024),    # 128 rows, 16 columns
    (3303, 3072, K),       # 160 rows
    (300, 28672, K),       # 160 rows, 128 columns a slab
    (2000, 11264, 1024),   # 192 rows, 64 columns
    (3302, 28672, 1024),   # 256 rows, 128 columns
    (4097, 3072, 1024),    # 256 rows, 32 columns
    (1024, 11264, K),      # 256 rows, whole tiles
])
def test_bytes_equal_the_fixed_tiling(d, M, N, K):
    w = d.pack_weight(up_bf16(ds.normal_bf16(8000 + N, (K, N), 0.02)))
    a = up_bf16(ds.normal_bf16(8100 + M, (M, K)))
    got = torch.full((M, N), float("nan"), device=DEV)
    want = torch.full((M, N), 7.0, device=DEV)
    step(f"wide GEMM M={M} N={N} K={K}")
    d.det_gemm_bf16(a, w, got, N, K)
    d.det_gemm_bf16_fixed_tile(a, w, want, N, K)
    torch.cuda.synchronize()
    assert torch.equal(bits(got), bits(want))


@pytest.mark.parametrize("M,N", [(2177, 3072), (300, 28672)])
def test_residual_and_swiglu_equal_small_calls(d, M, N):
    w0 = up_bf16(ds.normal_bf16(8200 + N, (K, N), 0.02))
    w, gu = d.pack_weight(w0), d.pack_gate_up(w0)
    a = up_bf16(ds.normal_bf16(8300 + M, (M, K)))
    r = up_bf16(ds.normal_bf16(8400 + M, (M, N)))
    res = torch.full((M, N), 7.0, dtype=torch.bfloat16, device=DEV)
    swi = torch.full((M, N // 2), 7.0, dtype=torch.bfloat16, device=DEV)
    step(f"wide GEMM epilogues M={M} N={N}")
    d.det_gemm_bf16_residual(a, w, r, res, N, K)
    d.det_gemm_swiglu_bf16(a, gu, swi, N // 2, K)
    inplace = r.clone()
    d.det_gemm_bf16_residual(a, w, inplace, inplace, N, K)
    torch.cuda.synchronize()
    assert torch.equal(bits(inplace), bits(res))
    for i in range(0, M, 200):
        p = slice(i, min(i + 200, M))
        n = p.stop - p.start
        o1 = torch.empty((n, N), dtype=torch.bfloat16, device=DEV)
        o2 = torch.empty((n, N // 2), dtype=torch.bfloat16, device=DEV)
        d.det_gemm_bf16_residual(a[p].contiguous(), w, r[p].contiguous(), o1, N, K)
        d.det_gemm_swiglu_bf16(a[p].contiguous(), gu, o2, N // 2, K)
        assert torch.equal(bits(res[p]), bits(o1)) and torch.equal(bits(swi[p]), bits(o2))


def test_rope_append_equals_small_calls(d):
    Hq, Hkv, S, Lmax = 16, 4, 3, 1100
    N = (Hq + 2 * Hkv) * 128
    lens = [1100, 900, 177]
    M = sum(lens)
    w = d.pack_qkv(up_bf16(ds.normal_bf16(8500, (K, N), 0.02)), Hq, Hkv, 128)
    a = up_bf16(ds.normal_bf16(8501, (M, K)))
    pos = torch.tensor([p for n in lens for p in range(n)], dtype=torch.int32, device=DEV)
    slots = torch.tensor([s for s, n in enumerate(lens) for _ in range(n)], dtype=torch.int32, device=DEV)
    ang = torch.arange(Lmax, device=DEV, dtype=torch.float64)[:, None] * (0.9 ** torch.arange(64, device=DEV, dtype=torch.float64))
    cos, sin = ang.cos().float().contiguous(), ang.sin().float().contiguous()

    def run(n):
        q = torch.full((M, Hq, 128), 7.0, dtype=torch.bfloat16, device=DEV)
        k = torch.zeros((S, Hkv, Lmax, 128), dtype=torch.bfloat16, device=DEV)
        v = torch.zeros_like(k)
        for i in range(0, M, n):
            p = slice(i, min(i + n, M))
            d.det_gemm_qkv_rope_append(a[p], w, q[p], k, v, pos[p], slots[p], cos, sin)
        torch.cuda.synchronize()
        return q, k, v

    step("wide GEMM with rotation and append")
    for got, want in zip(run(M), run(200)):
        assert torch.equal(bits(got), bits(want))


def wide(shape, pad):
    """A [rows, columns] bf16 tensor whose rows are `pad` elements apart from one another, surrounded by NaN."""
    t = torch.full((shape[0], shape[1] + pad), float("nan"), dtype=torch.bfloat16, device=DEV)
    return t, t[:, :shape[1]]


# every tile height, packings of 16, 32, 64 and 128 columns; tiles of one row, ragged and whole
@pytest.mark.parametrize("M,N,K,rows", [(3302, 2048, 1024, 128), (3303, 3072, K, 160), (300, 28672, K, 160), (2000, 11264, 1024, 192),
                                        (1024, 11264, K, 256), (4097, 3072, 1024, 256)])
def test_every_tile_height_with_every_epilogue_and_strided_rows(d, M, N, K, rows):
    assert d.det_gemm_wide_rows(M, N, K) == rows
    w0 = up_bf16(ds.normal_bf16(8600 + N, (K, N), 0.02))
    w, gu = d.pack_weight(w0), d.pack_gate_up(w0)
    a = up_bf16(ds.normal_bf16(8601 + M, (M, K)))
    r = up_bf16(ds.normal_bf16(8602 + M, (M, N)))
    (_, a_s), (_, r_s) = wide((M, K), 24), wide((M, N), 12)
    a_s.copy_(a), r_s.copy_(r)
    (sto_all, sto), (res_all, res), (swi_all, swi) = wide((M, N), 8), wide((M, N), 4), wide((M, N // 2), 20)
    step(f"wide GEMM epilogues and strides M={M} N={N} K={K}")
    d.det_gemm_bf16(a_s, w, sto, N, K)
    d.det_gemm_bf16_residual(a_s, w, r_s, res, N, K)
    d.det_gemm_swiglu_bf16(a_s, gu, swi, N // 2, K)
    torch.cuda.synchronize()
    for whole, view in ((sto_all, sto), (res_all, res), (swi_all, swi)):
        assert torch.isnan(whole[:, view.shape[1]:]).all(), "written between the rows"
    for i in range(0, M, 200):
        p = slice(i, min(i + 200, M))
        n = p.stop - p.start
        o0, o1 = torch.empty((n, N), dtype=torch.bfloat16, device=DEV), torch.empty((n, N), dtype=torch.bfloat16, device=DEV)
        o2 = torch.empty((n, N // 2), dtype=torch.bfloat16, device=DEV)
        assert d.det_gemm_wide_rows(n, N, K) == 0
        d.det_gemm_bf16(a[p].contiguous(), w, o0, N, K)
        d.det_gemm_bf16_residual(a[p].contiguous(), w, r[p].contiguous(), o1, N, K)
        d.det_gemm_swiglu_bf16(a[p].contiguous(), gu, o2, N // 2, K)
        assert torch.equal(bits(sto[p].contiguous()), bits(o0)) and torch.equal(bits(res[p].contiguous()), bits(o1))
        assert torch.equal(bits(swi[p].contiguous()), bits(o2))


@pytest.mark.parametrize("Hq,Hkv,lens,rows", [(16, 4, [1100, 1000, 77], 128), (32, 8, [1100, 1100, 1000, 102], 160), (16, 4, [1100] * 3 + [797], 256),
                                              (32, 28, [1100, 900], 192)])
def test_rope_append_at_every_tile_height(d, Hq, Hkv, lens, rows):
    N, M, S, Lmax = (Hq + 2 * Hkv) * 128, sum(lens), len(lens), 1100
    assert d.det_gemm_wide_rows(M, N, K) == rows
    w = d.pack_qkv(up_bf16(ds.normal_bf16(8700 + N, (K, N), 0.02)), Hq, Hkv, 128)
    a = up_bf16(ds.normal_bf16(8701 + M, (M, K)))
    _, a_s = wide((M, K), 8)
    a_s.copy_(a)
    pos = torch.tensor([p for n in lens for p in range(n)], dtype=torch.int32, device=DEV)
    slots = torch.tensor([s for s, n in enumerate(lens) for _ in range(n)], dtype=torch.int32, device=DEV)
    ang = torch.arange(Lmax, device=DEV, dtype=torch.float64)[:, None] * (0.9 ** torch.arange(64, device=DEV, dtype=torch.float64))
    cos, sin = ang.cos().float().contiguous(), ang.sin().float().contiguous()

    def run(x, n):
        q = torch.full((M, Hq, 128), 7.0, dtype=torch.bfloat16, device=DEV)
        k = torch.zeros((S, Hkv, Lmax, 128), dtype=torch.bfloat16, device=DEV)
        v = torch.zeros_like(k)
        for i in range(0, M, n):
            p = slice(i, min(i + n, M))
            d.det_gemm_qkv_rope_append(x[p], w, q[p], k, v, pos[p], slots[p], cos, sin)
        torch.cuda.synchronize()
        return q, k, v

    step(f"wide GEMM with rotation and append M={M} heads {Hq}/{Hkv}")
    for got, want in zip(run(a_s, M), run(a, 200)):
        assert torch.equal(bits(got), bits(want))
