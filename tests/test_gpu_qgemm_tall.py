"""The quantized GEMM's tiles of 32 or 64 rows for launches of many rows: every row must have the bytes it has in calls of
fewer rows, down to the 48 that take the kernel test_gpu_qgemm.py holds to the bit-exact oracle."""
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, step, up_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    import paper_2602_00182_amd as d
    return d


def parts(M, n=48):
    return [slice(i, min(i + n, M)) for i in range(0, M, n)]


# packings of 16, 32, 64 and 128 columns; one block of K, odd and even numbers of them; a tile of one row, whole tiles
@pytest.mark.parametrize("M,K,N", [(385, 64, 2048), (450, 192, 2048), (449, 1088, 3072), (225, 64, 5120), (257, 320, 5248),
                                   (129, 192, 11008), (256, 128, 11264), (129, 64, 20480), (200, 704, 28672)])
def test_rows_equal_small_calls(d, M, K, N):
    assert d.det_qgemm_tile(M, N, K) == ((64, 128) if N >= 20480 else (64, 64) if N >= 11008 else (32, 64))
    rows_equal_small_calls(d, M, K, N)


# 64 x 128 tiles of every packing: a tile of one row, nearly whole ones, odd and even numbers of blocks
@pytest.mark.parametrize("M,K,N", [(1601, 64, 2048), (1540, 192, 2048), (1087, 128, 3072), (900, 320, 5120), (300, 192, 11264), (321, 64, 11264)])
def test_rows_of_tall_tiles_equal_small_calls(d, M, K, N):
    assert d.det_qgemm_tile(M, N, K) == (64, 128)
    rows_equal_small_calls(d, M, K, N)


# 32 x 64 tiles of packings of 16, 32 and 64 columns, the last row in a tile of its own, at its end and before it; 64 x 64 tiles, also of
# a width that is no multiple of 128; 64 x 128 of the first row count that takes them with 128-column packings
@pytest.mark.parametrize("M,K,N", [(97, 64, 4096), (96, 192, 3072), (161, 320, 2048), (129, 128, 6144), (65, 64, 11264),
                                   (257, 192, 8192), (700, 64, 3072), (1000, 64, 4160), (96, 192, 20480),
                                   # where the tiles of 32- and 64-column packings begin
                                   (65, 64 * 7, 6144), (79, 64 * 20, 5120), (66, 64, 10112), (49, 64 * 7, 11264), (59, 64 * 20, 12800), (50, 128, 19968)])
def test_rows_of_small_tiles_equal_small_calls(d, M, K, N):
    rows_equal_small_calls(d, M, K, N)


def rows_equal_small_calls(d, M, K, N):
    for n in {48, M % 48 or 48}:  # the calls compared with take the kernel that is held to the oracle: columns and rows of no tile above
        rows, columns = d.det_qgemm_tile(n, N, K)
        assert columns == d.det_qgemm_tile(1, N, K)[1] and (columns != 64 or rows == 256)
    w = up_bf16(ds.normal_bf16(7000 + N, (K, N), 0.02))
    a = up_bf16(ds.normal_bf16(7100 + M, (M, K)))
    r = up_bf16(ds.normal_bf16(7200 + M, (M, N)))
    wp, gu = d.quant_pack_weight(w), d.quant_pack_gate_up(w)
    out = torch.full((M, N), float("nan"), device=DEV)
    res = torch.full((M, N), 7.0, dtype=torch.bfloat16, device=DEV)
    swi = torch.full((M, N // 2), 7.0, dtype=torch.bfloat16, device=DEV)
    codes, scales = d.quant_activations(a)
    step(f"tall quantized GEMM M={M} K={K} N={N}")
    d.det_qgemm_w4a8(codes, scales, wp, out, N)
    d.det_qgemm_w4a8_residual(codes, scales, wp, r, res, N)
    d.det_qgemm_w4a8_swiglu(codes, scales, gu, swi, N // 2)
    torch.cuda.synchronize()
    for p in parts(M):
        c, s = d.quant_activations(a[p].contiguous())
        n = p.stop - p.start
        o1 = torch.empty((n, N), device=DEV)
        o2 = torch.empty((n, N), dtype=torch.bfloat16, device=DEV)
        o3 = torch.empty((n, N // 2), dtype=torch.bfloat16, device=DEV)
        d.det_qgemm_w4a8(c, s, wp, o1, N)
        d.det_qgemm_w4a8_residual(c, s, wp, r[p].contiguous(), o2, N)
        d.det_qgemm_w4a8_swiglu(c, s, gu, o3, N // 2)
        assert torch.equal(out[p].view(torch.int32), o1.view(torch.int32))
        assert torch.equal(res[p].view(torch.int16), o2.view(torch.int16))
        assert torch.equal(swi[p].view(torch.int16), o3.view(torch.int16))


# a fused SwiGLU quantizer where the packing has 64 columns (no other kernel's tile holds a block there) and where it has 128, and a
# launch too small for it, which takes the two steps
@pytest.mark.parametrize("R,H,Hq,Hkv,F", [(390, 256, 2, 1, 5632), (241, 128, 2, 2, 10240), (420, 128, 4, 2, 64), (131, 2048, 16, 4, 512)])
def test_quantized_layer_rows_equal_small_calls(d, R, H, Hq, Hkv, F):
    D, Lmax = 128, 420
    g = lambda s, shape, std=0.05, mean=0.0: up_bf16(ds.normal_bf16(s, shape, std, mean))
    w = d.layer_weights(g(1, (H,), 0.1, 1.0), d.quant_pack_qkv(g(2, (H, (Hq + 2 * Hkv) * D)), Hq, Hkv, D),
                        d.quant_pack_weight(g(3, (Hq * D, H))), g(4, (H,), 0.1, 1.0), d.quant_pack_gate_up(g(5, (H, 2 * F))),
                        d.quant_pack_weight(g(6, (F, H))))
    cfg = d.layer_cfg(H, Hq, Hkv, D, F, Lmax, 1e-5, 0.08838834764831845)
    pos = torch.arange(R, dtype=torch.int32, device=DEV)
    slots = torch.zeros(R, dtype=torch.int32, device=DEV)
    ang = torch.arange(Lmax, device=DEV, dtype=torch.float64)[:, None] * (0.9 ** torch.arange(64, device=DEV, dtype=torch.float64))
    cos, sin = ang.cos().float().contiguous(), ang.sin().float().contiguous()
    x0 = g(7, (R, H), 1.0)

    def run(cuts):
        x = x0.clone()
        k = torch.zeros((1, Hkv, Lmax, D), dtype=torch.bfloat16, device=DEV)
        v = torch.zeros_like(k)
        for p in cuts:
            xp = x[p].contiguous()
            ws = torch.full((d.det_qdecoder_layer_workspace_bytes(cfg, xp.shape[0]),), 0xFF, dtype=torch.uint8, device=DEV)
            d.det_qdecoder_layer(w, cfg, xp, k, v, pos[p].contiguous(), slots[p].contiguous(), cos, sin, ws)
            x[p] = xp
        torch.cuda.synchronize()
        return x.view(torch.int16), k.view(torch.int16), v.view(torch.int16)

    step(f"quantized layer R={R} H={H} heads {Hq}/{Hkv} F={F}")
    for got, want in zip(run([slice(0, R)]), run(parts(R))):
        assert torch.equal(got, want)


def test_quantized_layer_refuses_misaligned_gate_up_weights(d):
    """Whichever kernel quantizes the SwiGLU output: 390 rows of F = 5632 take the tall tiles, 5 rows the two steps."""
    H, Hq, Hkv, D, F, Lmax = 256, 2, 1, 128, 5632, 390
    g = lambda s, shape, std=0.05, mean=0.0: up_bf16(ds.normal_bf16(s, shape, std, mean))
    gu = d.quant_pack_gate_up(g(5, (H, 2 * F)))
    shifted = torch.zeros(gu.numel() * gu.element_size() + 16, dtype=torch.uint8, device=DEV)
    w = d.layer_weights(g(1, (H,), 0.1, 1.0), d.quant_pack_qkv(g(2, (H, (Hq + 2 * Hkv) * D)), Hq, Hkv, D),
                        d.quant_pack_weight(g(3, (Hq * D, H))), g(4, (H,), 0.1, 1.0), gu, d.quant_pack_weight(g(6, (F, H))))
    cfg = d.layer_cfg(H, Hq, Hkv, D, F, Lmax, 1e-5, 0.08838834764831845)
    cos = sin = torch.zeros((Lmax, 64), device=DEV)
    k = torch.zeros((1, Hkv, Lmax, D), dtype=torch.bfloat16, device=DEV)
    v = torch.zeros_like(k)

    def run(R):
        ws = torch.empty((d.det_qdecoder_layer_workspace_bytes(cfg, R),), dtype=torch.uint8, device=DEV)
        pos = torch.arange(R, dtype=torch.int32, device=DEV)
        d.det_qdecoder_layer(w, cfg, g(7, (R, H), 1.0), k, v, pos, torch.zeros_like(pos), cos, sin, ws)
        torch.cuda.synchronize()

    for R in (390, 5):
        step(f"misaligned gate/up weights R={R}")
        w.wgu = gu.data_ptr()
        run(R)
        w.wgu = shifted.data_ptr() + 8
        with pytest.raises(d.DetError) as e:
            run(R)
        assert e.value.code == 3


# 2F of 2048 and 5120 columns: packings of 16 and 32, whose SwiGLU output only the tall tiles quantize (112 and 280 workgroups)
@pytest.mark.parametrize("R,H,Hq,Hkv,F", [(400, 256, 2, 1, 1024), (390, 128, 2, 2, 2560)])
def test_quantized_layer_of_narrow_packings(d, R, H, Hq, Hkv, F):
    test_quantized_layer_rows_equal_small_calls(d, R, H, Hq, Hkv, F)


@pytest.mark.parametrize("M,K,N", [(385, 64, 2048), (450, 192, 2048), (225, 64, 5120), (129, 192, 11008), (200, 704, 28672)])
def test_strided_rows(d, M, K, N):
    """Outputs and residuals whose rows lie apart: nothing is written between them."""
    w = up_bf16(ds.normal_bf16(7300 + N, (K, N), 0.02))
    wp, gu = d.quant_pack_weight(w), d.quant_pack_gate_up(w)
    codes, scales = d.quant_activations(up_bf16(ds.normal_bf16(7400 + M, (M, K))))
    r = up_bf16(ds.normal_bf16(7500 + M, (M, N + 12)))[:, :N]
    nan = lambda cols: torch.full((M, cols), float("nan"), dtype=torch.bfloat16, device=DEV)
    out, res, swi = nan(N + 8), nan(N + 4), nan(N // 2 + 20)
    o1, o2, o3 = nan(N), nan(N), nan(N // 2)
    step(f"tall quantized GEMM, strided M={M} K={K} N={N}")
    d.det_qgemm_w4a8(codes, scales, wp, out[:, :N], N)
    d.det_qgemm_w4a8_residual(codes, scales, wp, r, res[:, :N], N)
    d.det_qgemm_w4a8_swiglu(codes, scales, gu, swi[:, :N // 2], N // 2)
    d.det_qgemm_w4a8(codes, scales, wp, o1, N)
    d.det_qgemm_w4a8_residual(codes, scales, wp, r.contiguous(), o2, N)
    d.det_qgemm_w4a8_swiglu(codes, scales, gu, o3, N // 2)
    torch.cuda.synchronize()
    for got, want in ((out, o1), (res, o2), (swi, o3)):
        cols = want.shape[1]
        assert torch.isnan(got[:, cols:]).all(), "written between the rows"
        assert torch.equal(got[:, :cols].contiguous().view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("M,K,N", [(1601, 64, 2048), (900, 64, 5120), (300, 192, 11264)])
def test_strided_rows_of_tall_tiles(d, M, K, N):
    assert d.det_qgemm_tile(M, N, K) == (64, 128)
    test_strided_rows(d, M, K, N)
