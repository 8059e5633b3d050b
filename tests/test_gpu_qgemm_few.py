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


# hidden and inner sizes: rows of less than one and of two vectors a thread, and one too long to be normalized in the projection;
# gate/up packings of 16, 64 and 128 columns (the last with its output quantized in the projection), down projections that fit or not
@pytest.mark.parametrize("H,F,Hq,Hkv", [(192, 10240, 2, 1), (1984, 704, 4, 2), (2048, 5632, 16, 4), (4096, 14336, 32, 8), (4160, 1088, 8, 8)])
def test_layer_of_few_rows_equals_the_larger_batch(d, H, F, Hq, Hkv):
    """Up to four rows the layer normalizes and quantizes inside the projections; six rows take launches of their own for it."""
    Lmax, D, s = 300, 128, ds.tensor_seed(6, 710) + H
    n = lambda i, shape, std, mean=0.0: ds.normal_bf16_torch(s + i, shape, std, mean, DEV)
    w = d.layer_weights(n(0, (H,), 0.1, 1.0), d.quant_pack_qkv(n(1, (H, (Hq + 2 * Hkv) * D), 0.02), Hq, Hkv, D), d.quant_pack_weight(n(2, (Hq * D, H), 0.02)),
                        n(3, (H,), 0.1, 1.0), d.quant_pack_gate_up(n(4, (H, 2 * F), 0.02)), d.quant_pack_weight(n(5, (F, H), 0.02)))
    cfg = d.layer_cfg(H, Hq, Hkv, D, F, Lmax, 1e-5, float(np.float32(D ** -0.5)))
    cos, sin = (torch.from_numpy(t).to(DEV) for t in ds.rope_tables(Lmax, D))
    pos = torch.tensor([299, 0, 130, 255, 256, 7], dtype=torch.int32, device=DEV)
    x, k, v = n(6, (6, H), 1.0), n(7, (6, Hkv, Lmax, D), 1.0), n(8, (6, Hkv, Lmax, D), 1.0)
    x[1] = 0  # scales that are zero

    def run(R):
        xr, kr, vr = x[:R].clone(), k[:R].clone(), v[:R].clone()
        ws = torch.full((d.det_qdecoder_layer_workspace_bytes(cfg, R),), 0xFF, dtype=torch.uint8, device=DEV)
        step(f"quantized layer H={H} F={F} rows={R}")
        d.det_qdecoder_layer(w, cfg, xr, kr, vr, pos[:R].contiguous(), None, cos, sin, ws)
        torch.cuda.synchronize()
        return [down_bf16(t) for t in (xr, kr, vr)]

    full = run(6)
    for R in (1, 2, 3, 4):
        for got, want in zip(run(R), full):
            assert np.array_equal(got, want[:R]), R
