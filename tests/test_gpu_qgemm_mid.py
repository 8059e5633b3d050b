"""The quantized GEMM of up to 48 rows on packings of 16 and 32 columns on the GPU: row counts around the tiles' edges, blocks of K that
do not come out even over the producing waves and the groups of results, every epilogue; and the short last tiles of higher ones; bytes against the oracle or the unfused steps."""
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


def operands(d, orc, M, K, N):
    a = ds.normal_bf16(ds.tensor_seed(6, 800) + K + N, (M, K), 1.0, 0.0)
    w = ds.normal_bf16(ds.tensor_seed(6, 801) + K + N, (K, N), 0.02, 0.0)
    codes, scales = d.quant_activations(up_bf16(a))
    return w, codes, scales, *orc.qgemm_w4a8(*orc.quant_a8(a), *orc.quant_w4(w))


# one block of K; fewer than producers; one group and a block; a group more than LDS holds; the last of a tile's rows and one more, in one
# tile (3072 and 4096 columns), in several (2048, 1024 and 16), and past the form's largest; 32-column packings (5120 and 6144)
@pytest.mark.parametrize("M,K,N", [(5, 64, 16), (8, 448, 48), (16, 512, 2048), (17, 576, 3072), (32, 64 * 33, 4096), (33, 64 * 41, 3072), (48, 64 * 16, 4096),
                                   (49, 64 * 9, 4096), (64, 64 * 25, 2048), (101, 320, 1024), (77, 128, 16), (48, 64 * 224, 16), (5, 64 * 8, 6144), (16, 64 * 17, 5120),
                                   (31, 64 * 50, 5120), (33, 64 * 9, 6144)])
def test_bytes_match_oracle(d, orc, M, K, N):
    w, codes, scales, acc, out = operands(d, orc, M, K, N)
    packed = d.quant_pack_weight(up_bf16(w))
    c = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    cf = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
    step(f"some rows M={M} K={K} N={N}")
    d.det_qgemm_w4a8(codes, scales, packed, c, N)
    d.det_qgemm_w4a8(codes, scales, packed, cf, N)
    torch.cuda.synchronize()
    assert np.array_equal(cf.cpu().numpy().view(np.uint32), acc.view(np.uint32))
    assert np.array_equal(down_bf16(c), out)


# Higher tiles, which the general kernel has: a last one of one to eight rows, whose one or two computing waves are fed by ten or eleven
# in long chunks; tiles of 64 rows (1024 and 512 columns) and of 256 (widths that no 64-column tile fits), the last chunk a part of one
@pytest.mark.parametrize("M,K,N", [(196, 64 * 130, 1024), (193, 64 * 3, 1024), (200, 64 * 130, 1024), (387, 320, 512), (257, 64 * 70, 5072), (261, 64 * 30, 5152),
                                   (264, 64 * 77, 5152)])
def test_short_last_tiles(d, orc, M, K, N):
    rows, columns = d.det_qgemm_tile(M, N, K)
    assert columns < 64 and rows > 48 and 0 < M % rows <= 8
    test_bytes_match_oracle(d, orc, M, K, N)


@pytest.mark.parametrize("M,K,N", [(7, 576, 2048), (45, 320, 3072), (19, 2112, 6144)])
def test_epilogues_equal_unfused_bytes(d, orc, M, K, N):
    w, codes, scales, _, plain = operands(d, orc, M, K, N)
    r = ds.normal_bf16(ds.tensor_seed(6, 802) + N, (M, N), 1.0, 0.0)
    wide = torch.full((M + 1, N + 8), float("nan"), dtype=torch.bfloat16, device=DEV)
    wide[:M, :N] = up_bf16(r)
    y = torch.full((M + 1, N // 2), float("nan"), dtype=torch.bfloat16, device=DEV)
    step(f"some rows, residual in strided rows and in place, swiglu M={M} K={K} N={N}")
    d.det_qgemm_w4a8_residual(codes, scales, d.quant_pack_weight(up_bf16(w)), wide[:M, :N], wide[:M, :N], N)
    d.det_qgemm_w4a8_swiglu(codes, scales, d.quant_pack_gate_up(up_bf16(w)), y[:M], N // 2)
    torch.cuda.synchronize()
    assert np.array_equal(down_bf16(wide[:M, :N].contiguous()), orc.residual(r, plain))
    assert torch.isnan(wide[:, N:]).all() and torch.isnan(wide[M]).all() and torch.isnan(y[M]).all()
    assert np.array_equal(down_bf16(y[:M].contiguous()), orc.swiglu(plain[:, :N // 2], plain[:, N // 2:]))


# 50 and 66 rows: the gate/up and the fused projection in the smallest tiles of 64 columns
@pytest.mark.parametrize("H,F,Hq,Hkv,R", [(2048, 5632, 16, 4, 43), (4096, 1408, 32, 8, 43), (2048, 5632, 16, 4, 50), (4096, 1408, 32, 8, 66)])
def test_layer_rows_equal_single_rows(d, H, F, Hq, Hkv, R):
    """The rotation and cache append among the epilogues: each row's bytes are those of the row by itself."""
    Lmax, D, s = 300, 128, ds.tensor_seed(6, 810) + H
    n = lambda i, shape, std, mean=0.0: ds.normal_bf16_torch(s + i, shape, std, mean, DEV)
    w = d.layer_weights(n(0, (H,), 0.1, 1.0), d.quant_pack_qkv(n(1, (H, (Hq + 2 * Hkv) * D), 0.02), Hq, Hkv, D), d.quant_pack_weight(n(2, (Hq * D, H), 0.02)),
                        n(3, (H,), 0.1, 1.0), d.quant_pack_gate_up(n(4, (H, 2 * F), 0.02)), d.quant_pack_weight(n(5, (F, H), 0.02)))
    cfg = d.layer_cfg(H, Hq, Hkv, D, F, Lmax, 1e-5, float(np.float32(D ** -0.5)))
    cos, sin = (torch.from_numpy(t).to(DEV) for t in ds.rope_tables(Lmax, D))
    pos = torch.arange(0, 7 * R, 7, dtype=torch.int32, device=DEV).clamp_(max=Lmax - 1)
    x, k, v = n(6, (R, H), 1.0), n(7, (R, Hkv, Lmax, D), 1.0), n(8, (R, Hkv, Lmax, D), 1.0)

    def run(rows, slots=None):
        xr, kr, vr = x[rows].clone(), k[rows].clone(), v[rows].clone()
        if slots is not None:
            kr[slots.long()], vr[slots.long()] = k[rows], v[rows]
        ws = torch.full((d.det_qdecoder_layer_workspace_bytes(cfg, len(rows)),), 0xFF, dtype=torch.uint8, device=DEV)
        step(f"quantized layer H={H} F={F} rows={len(rows)}")
        d.det_qdecoder_layer(w, cfg, xr, kr, vr, pos[rows].contiguous(), slots, cos, sin, ws)
        torch.cuda.synchronize()
        return [down_bf16(t) for t in (xr, kr if slots is None else kr[slots.long()], vr if slots is None else vr[slots.long()])]

    single = [run([i]) for i in (0, 15, 16, 30, 42)]
    for rows, at in (((0, 15, 16, 30, 42), (0, 1, 2, 3, 4)), (tuple(range(R)), (0, 15, 16, 30, 42))):
        rows = list(rows)
        for slots in (None, torch.arange(len(rows) - 1, -1, -1, dtype=torch.int32, device=DEV)):
            got = run(rows, slots)
            for i, want in zip(at, single):
                for g_, w_ in zip(got, want):
                    assert np.array_equal(g_[i], w_[0])
