"""det_gemm_bf16 on the GPU against the fp64 oracle, and its determinism / batch-invariance
contract (byte equality, never allclose).  Bound for floating point, from the benchmark spec:
|err| <= 2^-8 |ref| + 2^-20 sum_k |a_ik b_kj|."""
import numpy as np
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, bits_to_f64, down_bf16, step, up_bf16, within_bound

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    import paper_2602_00182_amd as d
    return d


def run_gemm(d, A_bits, B_bits, out_f32=False, lda=None):
    """Packs B, runs the GEMM, returns bf16 bits (or fp32) as numpy."""
    M, K = A_bits.shape
    N = B_bits.shape[1]
    Bp = d.pack_weight(up_bf16(B_bits))
    if lda is None:
        A = up_bf16(A_bits)
    else:
        buf = torch.zeros((M, lda), dtype=torch.bfloat16, device=DEV)
        buf[:, :K] = up_bf16(A_bits)
        A = buf[:, :K]
    C = torch.empty((M, N), dtype=torch.float32 if out_f32 else torch.bfloat16, device=DEV)
    d.det_gemm_bf16(A, Bp, C, N, K)
    torch.cuda.synchronize()
    return C.cpu().numpy() if out_f32 else down_bf16(C)


def test_config1_tolerance_and_row_bytes(d, orc):
    """A [16,512], B [512,512] ~ N(0,1)/sqrt(512); rerun at M=1 and M=64: shared rows keep their bytes."""
    K = N = 512
    s = 1.0 / np.sqrt(K)
    A = ds.normal_bf16(ds.tensor_seed(1, 0), (16, K), s)
    Bm = ds.normal_bf16(ds.tensor_seed(1, 1), (K, N), s)
    step("gemm config 1 M=16")
    C16 = run_gemm(d, A, Bm)
    ref, refabs = orc.gemm_f64(A, Bm)
    assert within_bound(bits_to_f64(C16), ref, refabs).all()
    step("gemm config 1 M=1")
    C1 = run_gemm(d, A[:1], Bm)
    assert np.array_equal(C1[0], C16[0])
    extra = ds.normal_bf16(ds.tensor_seed(1, 2), (48, K), s)
    A64 = np.concatenate([A, extra], axis=0)
    step("gemm config 1 M=64")
    C64 = run_gemm(d, A64, Bm)
    assert np.array_equal(C64[:16], C16)
    ref, refabs = orc.gemm_f64(A64, Bm)
    assert within_bound(bits_to_f64(C64), ref, refabs).all()


@pytest.mark.parametrize("M,N,K", [
    (1, 16, 64), (5, 48, 64), (16, 512, 512), (17, 4096, 128), (100, 7680, 192), (33, 28672, 64),
    (257, 64, 1088), (300, 3840 * 2, 64), (64, 32000, 128), (256, 4096, 2048 + 64),
    (20, 11520, 64), (20, 16000, 128), (35, 20000, 64), (70, 24000, 192),
])
def test_integer_matrices_are_exact(d, orc, M, N, K):
    """Entries in -4..4: every summation order gives the exact integer (|sum| < 2^24), so the GPU
    bytes must equal bf16_rne(exact).  Pins layout, packing, K coverage, masking of ragged M and
    round-to-nearest-even of the output."""
    A = ds.small_int_bf16(100 + M, (M, K))
    Bm = ds.small_int_bf16(200 + N, (K, N))
    exact = ds.bf16_bits_to_f32(A).astype(np.int64) @ ds.bf16_bits_to_f32(Bm).astype(np.int64)
    want = orc.bf16_rne(exact.astype(np.float32))
    step(f"gemm integer exact M={M} N={N} K={K}")
    got = run_gemm(d, A, Bm)
    assert np.array_equal(got, want)
    got32 = run_gemm(d, A, Bm, out_f32=True)
    assert np.array_equal(got32, exact.astype(np.float32))


@pytest.mark.parametrize("M,N", [(M, N) for N in (2048, 6224, 11264) for M in (7, 9, 23, 33, 35, 45, 57, 65, 95, 121, 129, 250, 256)] +
                         [(M, 4096) for M in (66, 95, 97, 129, 131, 201, 300, 393, 420, 500, 601, 999)] + [(M, 6144) for M in (161, 193, 290, 401)] + [(M, 3072) for M in (65, 81)] + [(M, 8192) for M in (97, 128, 129, 163)])
def test_ragged_rows_whatever_the_split_of_the_loads(d, orc, M, N):
    """Row counts around every split of a tile's half blocks over the loading waves, in the row-cut (N = 2048), two-workgroups-a-
    compute-unit (6224) and wide (11264) forms, and every pipeline of the 64-column tiles (4096 and 6144: tiles of 32 to 256
    rows), the rows behind the last one NaN: small integers, so exact."""
    check_small_integers(d, orc, M, N, 64 * 11)


def check_small_integers(d, orc, M, N, K):
    A = ds.small_int_bf16(500 + M, (M, K))
    Bm = ds.small_int_bf16(600 + N, (K, N))
    want = orc.bf16_rne((ds.bf16_bits_to_f32(A) @ ds.bf16_bits_to_f32(Bm)).astype(np.float32))  # |sum| < 2^24: exact in fp32
    buf = torch.full((M + 16, K), float("nan"), dtype=torch.bfloat16, device=DEV)
    buf[:M] = up_bf16(A)
    C = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    step(f"gemm ragged M={M} N={N} K={K}")
    d.det_gemm_bf16(buf[:M], d.pack_weight(up_bf16(Bm)), C, N, K)
    torch.cuda.synchronize()
    assert np.array_equal(down_bf16(C), want)


# Tiles of 48 to 112 columns whose rows are loaded in front of the weights or spaced out, and the heights and depths beside those
@pytest.mark.parametrize("M,N,K", [(M, N, 704) for N in (10752, 12800, 15360, 17920) for M in (16, 17, 56, 57, 64, 75, 96, 97)] +
                         [(M, 9984, 704) for M in (16, 23, 24, 25, 33, 48, 49)] +
                         [(M, 10752, K) for M in (32, 33, 40, 47, 49) for K in (5056, 5120)] + [(49, 16384, 704), (49, 16448, 704)] +
                         [(M, 10752, 11520) for M in (64, 65)] + [(96, 10752, 11456)])
def test_rows_loaded_in_front_of_the_weights(d, orc, M, N, K):
    check_small_integers(d, orc, M, N, K)


def test_rne_ties_and_identity(d, orc):
    """Identity weights copy A; a product of 257 must round to 256 (tie to even)."""
    K = N = 256
    A = ds.normal_bf16(301, (40, K))
    eye = ds.f32_to_bf16_bits(np.eye(K, dtype=np.float32))
    step("gemm identity")
    assert np.array_equal(run_gemm(d, A, eye), A)
    a = np.zeros((1, K), dtype=np.float32)
    a[0, :257 - 1] = 1.0  # 256 ones ...
    b = np.zeros((K, N), dtype=np.float32)
    b[:, 0] = 1.0
    b[0, 0] = 2.0        # ... one of them weighted 2 -> sum 257
    b[:, 1] = 1.0
    b[0, 1] = 4.0        # 259 -> tie between 258 and 260 -> 260
    got = run_gemm(d, ds.f32_to_bf16_bits(a), ds.f32_to_bf16_bits(b))
    assert ds.bf16_bits_to_f32(got[0, :2]).tolist() == [256.0, 260.0]


def test_strided_a_and_lda(d, orc):
    K, N, M = 512, 4096, 37
    A = ds.normal_bf16(311, (M, K))
    Bm = ds.normal_bf16(312, (K, N), 0.02)
    step("gemm strided A")
    assert np.array_equal(run_gemm(d, A, Bm), run_gemm(d, A, Bm, lda=K + 64))


def _llama_case(K, N, Mmax=256):
    W = ds.normal_bf16(ds.tensor_seed(2, K // 64 + N), (K, N), 0.02)
    X = ds.normal_bf16(ds.tensor_seed(2, 7), (Mmax, K))
    return X, W


@pytest.mark.parametrize("K,N", [(4096, 4096), (4096, 6144), (4096, 28672), (14336, 4096)])
def test_llama_shapes_sampled_vs_oracle_and_batch_invariance(d, orc, K, N):
    """Full-size projection GEMMs: M swept over 1..256 with the first M rows of one X, every row's
    bytes identical at every M; a seeded sample of outputs against the fp64 oracle."""
    X, W = _llama_case(K, N)
    Wp = d.pack_weight(up_bf16(W))
    Xd = up_bf16(X)
    outs = {}
    for M in [1, 2, 4, 8, 16, 32, 64, 128, 256]:
        step(f"gemm llama K={K} N={N} M={M}")
        C = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
        d.det_gemm_bf16(Xd[:M], Wp, C, N, K)
        torch.cuda.synchronize()
        outs[M] = down_bf16(C)
    full = outs[256]
    for M, c in outs.items():
        assert np.array_equal(c, full[:M]), f"rows changed between M={M} and M=256"
    rng = np.random.default_rng(K + N)
    rows = rng.integers(0, 256, 4096).astype(np.int32)
    cols = rng.integers(0, N, 4096).astype(np.int32)
    rows[:64] = np.arange(64) * 4
    cols[:64] = N - 1 - np.arange(64)
    ref, refabs = orc.gemm_f64_sample(X, W, rows, cols)
    got = bits_to_f64(full[rows, cols])
    assert within_bound(got, ref, refabs).all()


@pytest.mark.parametrize("K,N", [(4096, 4096), (1024, 6144), (512, 1024), (14336, 4096)])
def test_tile_shape_switch_points_keep_bytes(d, orc, K, N):
    """Narrow matrices change tile shape with M (16- or 32-column tiles of up to 256 rows up to 64, 80, 112 or 160
    rows, 64-column tiles of fewer rows from there on; M = 1100 is more rows than one round of tiles
    holds, with a ragged last tile): every row's bytes are those of the M = 1 launch that computes it
    alone, and a sample agrees with fp64."""
    X = ds.normal_bf16(ds.tensor_seed(3, K), (1100, K))
    W = ds.normal_bf16(ds.tensor_seed(3, N), (K, N), 0.02)
    Wp = d.pack_weight(up_bf16(W))
    Xd = up_bf16(X)

    def gemm(lo, hi):
        C = torch.empty((hi - lo, N), dtype=torch.bfloat16, device=DEV)
        d.det_gemm_bf16(Xd[lo:hi], Wp, C, N, K)
        torch.cuda.synchronize()
        return down_bf16(C)

    step(f"gemm tile switch K={K} N={N} M=1100")
    full = gemm(0, 1100)
    for M in [1, 17, 64, 65, 66, 80, 81, 95, 96, 97, 111, 112, 113, 129, 160, 161, 177, 191, 192, 193, 255, 256, 257, 513, 1025]:
        step(f"gemm tile switch K={K} N={N} M={M}")
        assert np.array_equal(gemm(0, M), full[:M]), f"rows changed between M={M} and M=1100"
    for r in [0, 95, 96, 200, 255, 256, 512, 1099]:
        assert np.array_equal(gemm(r, r + 1)[0], full[r]), f"row {r} alone differs"
    rng = np.random.default_rng(K * 3 + N)
    rows = rng.integers(0, 1100, 2048).astype(np.int32)
    cols = rng.integers(0, N, 2048).astype(np.int32)
    rows[:16] = 1099
    cols[:16] = N - 1 - np.arange(16) * 5
    ref, refabs = orc.gemm_f64_sample(X, W, rows, cols)
    assert within_bound(bits_to_f64(full[rows, cols]), ref, refabs).all()


@pytest.mark.parametrize("K,N", [(512, 1024), (256, 2048), (128, 6144), (128, 12288)])
def test_prefill_sized_launch_keeps_bytes(d, orc, K, N):
    """Launches with thousands of rows use 128-column tiles whatever the packing (16-, 32- or 64-column
    slabs): rows keep the bytes of the launches that compute them in small groups, and a sample agrees
    with fp64."""
    tiles = -(-256 // (N // 128))          # row tiles that make 256 workgroups of 128 columns
    M = 256 * (tiles - 1) + 77
    X = ds.normal_bf16(ds.tensor_seed(3, K + 1), (M, K))
    W = ds.normal_bf16(ds.tensor_seed(3, N + 1), (K, N), 0.05)
    Wp = d.pack_weight(up_bf16(W))
    Xd = up_bf16(X)

    def gemm(lo, hi):
        C = torch.empty((hi - lo, N), dtype=torch.bfloat16, device=DEV)
        d.det_gemm_bf16(Xd[lo:hi], Wp, C, N, K)
        torch.cuda.synchronize()
        return down_bf16(C)

    step(f"gemm prefill-sized K={K} N={N} M={M}")
    full = gemm(0, M)
    for lo, hi in [(0, 1), (0, 64), (255, 300), (M - 100, M), (M - 1, M), (M // 2, M // 2 + 256)]:
        assert np.array_equal(gemm(lo, hi), full[lo:hi]), (lo, hi)
    rng = np.random.default_rng(K + N)
    rows = rng.integers(0, M, 2048).astype(np.int32)
    cols = rng.integers(0, N, 2048).astype(np.int32)
    rows[:8] = M - 1
    ref, refabs = orc.gemm_f64_sample(X, W, rows, cols)
    assert within_bound(bits_to_f64(full[rows, cols]), ref, refabs).all()


def test_rows_do_not_see_each_other(d, orc):
    """Row i's bytes are unchanged when the other rows are replaced, when row i moves to another
    slot, and when M is not a multiple of the row block."""
    K, N = 4096, 4096
    X, W = _llama_case(K, N)
    Wp = d.pack_weight(up_bf16(W))

    def gemm(Xb):
        C = torch.empty((Xb.shape[0], N), dtype=torch.bfloat16, device=DEV)
        d.det_gemm_bf16(up_bf16(Xb), Wp, C, N, K)
        torch.cuda.synchronize()
        return down_bf16(C)

    step("gemm row isolation")
    base = gemm(X[:200])
    other = ds.normal_bf16(999, (200, K), 3.0)
    other[57] = X[57]
    assert np.array_equal(gemm(other)[57], base[57])
    nanrows = X[:200].copy()
    nanrows[:] = 0x7FC0
    nanrows[130] = X[130]
    assert np.array_equal(gemm(nanrows)[130], base[130])
    perm = np.random.default_rng(5).permutation(200)
    assert np.array_equal(gemm(X[:200][perm]), base[perm])
    assert np.array_equal(gemm(X[:93]), base[:93])
    big = np.concatenate([X, X[:77]], axis=0)  # M = 333 > 256: second row tile
    out = gemm(big)
    assert np.array_equal(out[:200], base) and np.array_equal(out[256:], base[:77])


def test_repeat_streams_launch_order_and_background_load(d, orc):
    """100 repeats, three streams, shuffled launch order and a bandwidth hog on another stream:
    every result byte-identical (the paper's same-host, batch and stress conditions, section 6.7,
    10.1 and 10.2)."""
    K, N = 4096, 6144
    X, W = _llama_case(K, N)
    Wp = d.pack_weight(up_bf16(W))
    Xd = up_bf16(X)
    Ms = [1, 8, 64, 256]
    want = {}
    for M in Ms:
        C = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
        d.det_gemm_bf16(Xd[:M], Wp, C, N, K)
        want[M] = C.clone()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(device=DEV) for _ in range(3)]
    hog_stream = torch.cuda.Stream(device=DEV)
    hog = torch.empty(256 << 20, dtype=torch.uint8, device=DEV)
    rng = np.random.default_rng(9)
    mismatches = 0
    step("gemm 100 repeats over 3 streams with background copies")
    for rep in range(100):
        with torch.cuda.stream(hog_stream):
            hog.copy_(hog.flip(0) if rep % 10 == 0 else hog)
        order = rng.permutation(len(Ms))
        outs = []
        for j in order:
            M = Ms[j]
            st = streams[(rep + j) % 3]
            C = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
            with torch.cuda.stream(st):
                d.det_gemm_bf16(Xd[:M], Wp, C, N, K)
            outs.append((M, C))
        torch.cuda.synchronize()
        for M, C in outs:
            mismatches += int(not torch.equal(C.view(torch.int16), want[M].view(torch.int16)))
    assert mismatches == 0


def test_error_codes(d):
    A = torch.zeros((4, 64), dtype=torch.bfloat16, device=DEV)
    Bp = torch.zeros(64 * 16, dtype=torch.bfloat16, device=DEV)
    C = torch.zeros((4, 16), dtype=torch.bfloat16, device=DEV)
    lib = d.api.lib()
    s = torch.cuda.current_stream().cuda_stream
    assert lib.det_gemm_bf16(A.data_ptr(), 64, Bp.data_ptr(), C.data_ptr(), 16, 4, 16, 64, 0, s) == 0
    assert lib.det_gemm_bf16(A.data_ptr(), 64, Bp.data_ptr(), C.data_ptr(), 16, 4, 24, 64, 0, s) == 2
    assert lib.det_gemm_bf16(A.data_ptr(), 64, Bp.data_ptr(), C.data_ptr(), 16, 4, 16, 96, 0, s) == 2
    assert lib.det_gemm_bf16(A.data_ptr() + 2, 64, Bp.data_ptr(), C.data_ptr(), 16, 4, 16, 64, 0, s) == 3
    assert lib.det_gemm_bf16(None, 64, Bp.data_ptr(), C.data_ptr(), 16, 4, 16, 64, 0, s) == 1
    assert lib.det_gemm_bf16(A.data_ptr(), 64, Bp.data_ptr(), C.data_ptr(), 16, 0, 16, 64, 0, s) == 1
    assert lib.det_gemm_bf16(A.data_ptr(), 64, Bp.data_ptr(), C.data_ptr(), 16, 4, 16, 64, 7, s) == 1
    # the fused projections: argument errors launch nothing
    buf = torch.zeros(1 << 20, dtype=torch.uint8, device=DEV)
    p = buf.data_ptr()
    qkv = lib.det_gemm_qkv_rope_append
    assert qkv(p, 64, p, p, p, p, p, None, p, p, 2, 1, 1, 128, 8, 64, s) == 0          # N = 384, K = 64: fine
    assert qkv(p, 64, p, p, p, p, p, None, p, p, 2, 1, 1, 64, 8, 64, s) == 2           # head size
    assert qkv(p, 64, p, p, p, p, p, None, p, p, 2, 0, 1, 128, 8, 64, s) == 2          # no query heads
    assert qkv(p, 64, p, p, p, p, None, None, p, p, 2, 1, 1, 128, 8, 64, s) == 1       # no positions
    assert qkv(p, 64, p, p, p + 4, p, p, None, p, p, 2, 1, 1, 128, 8, 64, s) == 3      # cache alignment
    assert qkv(p, 32, p, p, p, p, p, None, p, p, 2, 1, 1, 128, 8, 64, s) == 1          # lda < K
    assert lib.det_gemm_pack_qkv(p, p, 1, 1, 96, 64, s) == 2
    nq = lib.det_rmsnorm_gemm_qkv_rope_append
    assert nq(p, 64, p, 1e-5, p, p, p, p, p, p, None, p, p, 2, 1, 1, 128, 8, 64, s) == 0
    assert nq(p, 64, None, 1e-5, p, p, p, p, p, p, None, p, p, 2, 1, 1, 128, 8, 64, s) == 1    # no norm weight
    assert nq(p, 64, p, 1e-5, p, None, p, p, p, p, None, p, p, 2, 1, 1, 128, 8, 64, s) == 1    # no scratch
    assert nq(p, 128, p, 1e-5, p, p, p, p, p, p, None, p, p, 9, 1, 1, 128, 16, 64, s) == 1     # two launches need ldx == K
    ns = lib.det_rmsnorm_gemm_swiglu_bf16
    assert ns(p, 64, p, 1e-5, p, p, p, 8, 2, 8, 64, s) == 0
    assert ns(p, 64, p, 1e-5, p, p, p, 4, 2, 8, 64, s) == 1                              # ldy < F
    assert ns(p, 64, p, 1e-5, p, p, p, 12, 2, 12, 64, s) == 2                            # F % 8
    torch.cuda.synchronize()


@pytest.mark.parametrize("M,K,N", [(1, 512, 4096), (19, 4096, 4096), (130, 1024, 28672), (64, 5632, 2048), (200, 1024, 4096),
                                   (250, 512, 6144)])
def test_fused_residual_epilogue_equals_unfused_bytes(d, orc, M, K, N):
    """det_gemm_bf16_residual = det_gemm_bf16 then det_residual_add, byte for byte (and the oracle's
    residual of the GPU's own GEMM output), also in place (C is R)."""
    A = ds.normal_bf16(700 + M, (M, K))
    W = ds.normal_bf16(701 + N, (K, N), 0.02)
    R = ds.normal_bf16(702 + M, (M, N))
    Wp = d.pack_weight(up_bf16(W))
    Ad, Rd = up_bf16(A), up_bf16(R)
    plain = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    step(f"gemm residual epilogue M={M} K={K} N={N}")
    d.det_gemm_bf16(Ad, Wp, plain, N, K)
    unfused = torch.empty_like(plain)
    d.det_residual_add(Rd, plain, unfused)
    fused = torch.empty_like(plain)
    d.det_gemm_bf16_residual(Ad, Wp, Rd, fused, N, K)
    inplace = Rd.clone()
    d.det_gemm_bf16_residual(Ad, Wp, inplace, inplace, N, K)
    torch.cuda.synchronize()
    assert torch.equal(fused.view(torch.int16), unfused.view(torch.int16))
    assert torch.equal(inplace.view(torch.int16), unfused.view(torch.int16))
    assert np.array_equal(down_bf16(fused), orc.residual(R, down_bf16(plain)))


@pytest.mark.parametrize("M,K,F", [(1, 512, 2048), (33, 4096, 14336), (7, 2048, 5632), (200, 256, 1000 * 8),
                                   (130, 512, 2048)])
def test_fused_swiglu_epilogue_equals_unfused_bytes(d, orc, M, K, F):
    """det_gemm_swiglu_bf16 on the gate/up-interleaved packing = det_gemm_bf16 on the plain packing
    then det_swiglu, byte for byte."""
    A = ds.normal_bf16(710 + M, (M, K))
    W = ds.normal_bf16(711 + F, (K, 2 * F), 0.03)
    Ad, Wd = up_bf16(A), up_bf16(W)
    gu = torch.empty((M, 2 * F), dtype=torch.bfloat16, device=DEV)
    step(f"gemm swiglu epilogue M={M} K={K} F={F}")
    d.det_gemm_bf16(Ad, d.pack_weight(Wd), gu, 2 * F, K)
    unfused = torch.empty((M, F), dtype=torch.bfloat16, device=DEV)
    d.det_swiglu(gu[:, :F], gu[:, F:], unfused)
    fused = torch.empty((M, F), dtype=torch.bfloat16, device=DEV)
    d.det_gemm_swiglu_bf16(Ad, d.pack_gate_up(Wd), fused, F, K)
    torch.cuda.synchronize()
    assert torch.equal(fused.view(torch.int16), unfused.view(torch.int16))
    guh = down_bf16(gu)
    assert np.array_equal(down_bf16(fused), orc.swiglu(np.ascontiguousarray(guh[:, :F]), np.ascontiguousarray(guh[:, F:])))


# 64-column tiles of more than 64 rows, which four waves compute, of 16- and 32-column packings: heights around whole numbers of blocks
@pytest.mark.parametrize("M,K,N,rows", [(300, 512, 4096, 80), (520, 256, 4096, 136), (700, 256, 3072, 144), (1000, 256, 4096, 256),
                                        (176, 256, 6144, 88), (300, 512, 6144, 152)])
def test_epilogues_of_tiles_that_four_waves_compute(d, orc, M, K, N, rows):
    assert d.det_gemm_tile(M, N, K) == (rows, 64)
    test_fused_residual_epilogue_equals_unfused_bytes(d, orc, M, K, N)
    test_fused_swiglu_epilogue_equals_unfused_bytes(d, orc, M, K, N // 2)


@pytest.mark.parametrize("M,Hq,Hkv,K,Lmax,use_slots", [(1, 32, 8, 4096, 64, False), (7, 4, 2, 256, 40, True),
                                                       (33, 8, 2, 1024, 96, True), (300, 32, 8, 4096, 320, False),
                                                       (1300, 32, 8, 512, 700, True), (130, 2, 1, 512, 130, True)])
def test_fused_rope_append_epilogue_equals_unfused_bytes(d, M, Hq, Hkv, K, Lmax, use_slots):
    """det_gemm_qkv_rope_append on the pair-interleaved packing = det_gemm_bf16 on the plain packing, then
    det_rope on the query and key heads and a copy of the key and value heads into the caches, byte for
    byte; every other cache row keeps its bytes."""
    D = 128
    N = (Hq + 2 * Hkv) * D
    A = up_bf16(ds.normal_bf16(720 + M, (M, K)))
    W = up_bf16(ds.normal_bf16(721 + Hq, (K, N), 0.05))
    cos_h, sin_h = ds.rope_tables(Lmax, D, 5.0e5)
    cos_t, sin_t = torch.from_numpy(cos_h).to(DEV), torch.from_numpy(sin_h).to(DEV)
    rng = np.random.default_rng(722 + M)
    if use_slots:  # a few slots, several rows each, distinct (slot, position) pairs, out-of-range positions clamped
        S = max(2, (M + Lmax - 1) // Lmax + 1)
        cells = rng.permutation(S * Lmax)[:M]
        slots_h, pos_h = (cells // Lmax).astype(np.int32), (cells % Lmax).astype(np.int32)
    else:
        S = M
        slots_h, pos_h = np.arange(M, dtype=np.int32), rng.integers(0, Lmax, M).astype(np.int32)
        pos_h[0] = Lmax + 5  # clamped to Lmax - 1
    pos = torch.from_numpy(pos_h).to(DEV)
    slots = torch.from_numpy(slots_h).to(DEV) if use_slots else None
    kc0 = up_bf16(ds.normal_bf16(723, (S, Hkv, Lmax, D)))
    vc0 = up_bf16(ds.normal_bf16(724, (S, Hkv, Lmax, D)))
    step(f"gemm rope/append epilogue M={M} Hq={Hq} Hkv={Hkv} K={K}")
    qkv = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    d.det_gemm_bf16(A, d.pack_weight(W), qkv, N, K)
    qk = qkv[:, :(Hq + Hkv) * D].contiguous().view(M, Hq + Hkv, D)
    qk_rot = torch.empty_like(qk)
    d.det_rope(qk, qk_rot, pos, cos_t, sin_t)
    torch.cuda.synchronize()
    pc = torch.from_numpy(np.clip(pos_h, 0, Lmax - 1).astype(np.int64)).to(DEV)
    sl = torch.from_numpy(slots_h.astype(np.int64)).to(DEV)
    k_ref, v_ref = kc0.clone(), vc0.clone()
    k_ref[sl, :, pc, :] = qk_rot[:, Hq:, :]
    v_ref[sl, :, pc, :] = qkv[:, (Hq + Hkv) * D:].view(M, Hkv, D)
    qbuf = torch.zeros((M, Hq, D), dtype=torch.bfloat16, device=DEV)
    kc, vc = kc0.clone(), vc0.clone()
    d.det_gemm_qkv_rope_append(A, d.pack_qkv(W, Hq, Hkv, D), qbuf, kc, vc, pos, slots, cos_t, sin_t)
    torch.cuda.synchronize()
    assert torch.equal(qbuf.view(torch.int16), qk_rot[:, :Hq, :].contiguous().view(torch.int16))
    assert torch.equal(kc.view(torch.int16), k_ref.view(torch.int16))
    assert torch.equal(vc.view(torch.int16), v_ref.view(torch.int16))


@pytest.mark.parametrize("K,Hq,Hkv,F", [(4096, 32, 8, 14336), (2048, 16, 4, 5632), (1024, 4, 2, 2048), (256, 2, 1, 8000),
                                        (4096, 8, 8, 24000), (3072, 24, 8, 8192), (1024, 4, 2, 3112)])
def test_gemm_that_normalizes_its_rows_equals_rmsnorm_then_gemm(d, K, Hq, Hkv, F):
    """det_rmsnorm_gemm_qkv_rope_append / det_rmsnorm_gemm_swiglu_bf16 / det_rmsnorm_gemm_bf16 (bf16 and fp32
    out) = det_rmsnorm, then the GEMM, byte for byte, for every M in 1..6 (1..4: the workgroups normalize the rows themselves; 5, 6: two launches)."""
    D, Lmax = 128, 48
    N = (Hq + 2 * Hkv) * D
    Wq = d.pack_qkv(up_bf16(ds.normal_bf16(731 + K, (K, N), 0.05)), Hq, Hkv, D)
    Wg_logical = up_bf16(ds.normal_bf16(732 + F, (K, 2 * F), 0.05))
    Wg, Wplain = d.pack_gate_up(Wg_logical), d.pack_weight(Wg_logical)
    wn = up_bf16(ds.normal_bf16(733 + K, (K,), 0.3, 1.0))
    cos_h, sin_h = ds.rope_tables(Lmax, D, 5.0e5)
    cos_t, sin_t = torch.from_numpy(cos_h).to(DEV), torch.from_numpy(sin_h).to(DEV)
    eps = 1e-5
    for M in range(1, 7):
        step(f"norm-fused gemm K={K} N={N} F={F} M={M}")
        lda = K + 64 if M % 2 == 0 else K  # strided rows on the fused path
        xbuf = up_bf16(ds.normal_bf16(734 + M, (M, lda), 1.5, 0.25))
        x = xbuf[:, :K] if M < 5 else xbuf[:, :K].contiguous()
        pos = torch.from_numpy(np.random.default_rng(735 + M).permutation(Lmax)[:M].astype(np.int32)).to(DEV)
        h = torch.empty((M, K), dtype=torch.bfloat16, device=DEV)
        d.det_rmsnorm(x.contiguous(), wn, h, eps)
        q_ref = torch.zeros((M, Hq, D), dtype=torch.bfloat16, device=DEV)
        kc_ref = up_bf16(ds.normal_bf16(736, (M, Hkv, Lmax, D)))
        vc_ref = up_bf16(ds.normal_bf16(737, (M, Hkv, Lmax, D)))
        kc, vc, q = kc_ref.clone(), vc_ref.clone(), torch.zeros_like(q_ref)
        d.det_gemm_qkv_rope_append(h, Wq, q_ref, kc_ref, vc_ref, pos, None, cos_t, sin_t)
        y_ref = torch.empty((M, F), dtype=torch.bfloat16, device=DEV)
        d.det_gemm_swiglu_bf16(h, Wg, y_ref, F, K)
        h2 = torch.zeros_like(h)
        d.det_rmsnorm_gemm_qkv_rope_append(x, wn, eps, Wq, h2, q, kc, vc, pos, None, cos_t, sin_t)
        y = torch.empty_like(y_ref)
        d.det_rmsnorm_gemm_swiglu_bf16(x, wn, eps, Wg, h2, y, F)
        plain = {}
        for dt in (torch.bfloat16, torch.float32):
            want_c = torch.empty((M, 2 * F), dtype=dt, device=DEV)
            d.det_gemm_bf16(h, Wplain, want_c, 2 * F, K)
            got_c = torch.zeros_like(want_c)
            d.det_rmsnorm_gemm_bf16(x, wn, eps, Wplain, h2, got_c, 2 * F)
            plain[dt] = (got_c, want_c)
        torch.cuda.synchronize()
        for got, want in plain.values():
            assert torch.equal(got.view(torch.uint8), want.view(torch.uint8)), (K, M, got.dtype)
        for got, want in ((q, q_ref), (kc, kc_ref), (vc, vc_ref), (y, y_ref)):
            assert torch.equal(got.view(torch.int16), want.view(torch.int16)), (K, M)


def test_seeded_shape_sweep_both_gemms(d, orc):
    """Thirty seeded (M, N, K) drawn across every tiling rule (narrow and wide packings, row-cut, 64- and
    128-column tiles, several row tiles, ragged M): a sample of each product within the fp64 bound, one
    row equal to its M = 1 launch, and the quantized GEMM of the same operands equal to the oracle's."""
    rng = np.random.default_rng(20260200182)
    widths = [16, 48, 64, 128, 320, 1024, 1536, 2048, 2560, 3072, 4096, 5120, 6144, 7168, 9216, 11264, 12288, 16384]
    heights = [1, 3, 8, 9, 16, 17, 40, 64, 95, 96, 130, 191, 192, 255, 256, 257, 300, 700, 1500, 4500]
    for it in range(30):
        N, K, M = int(rng.choice(widths)), 64 * int(rng.integers(1, 40)), int(rng.choice(heights))
        if M * N * K > 2e10:
            M = max(1, int(2e10 / (N * K)))
        step(f"sweep gemm M={M} N={N} K={K}")
        X = ds.normal_bf16(ds.tensor_seed(3, 100 + it), (M, K))
        W = ds.normal_bf16(ds.tensor_seed(3, 200 + it), (K, N), 0.05)
        Wp, Xd = d.pack_weight(up_bf16(W)), up_bf16(X)
        C = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
        d.det_gemm_bf16(Xd, Wp, C, N, K)
        r = int(rng.integers(0, M))
        C1 = torch.empty((1, N), dtype=torch.bfloat16, device=DEV)
        d.det_gemm_bf16(Xd[r:r + 1], Wp, C1, N, K)
        torch.cuda.synchronize()
        full = down_bf16(C)
        assert np.array_equal(down_bf16(C1)[0], full[r]), (M, N, K, r)
        rows = rng.integers(0, M, 512).astype(np.int32)
        cols = rng.integers(0, N, 512).astype(np.int32)
        ref, refabs = orc.gemm_f64_sample(X, W, rows, cols)
        assert within_bound(bits_to_f64(full[rows, cols]), ref, refabs).all(), (M, N, K)
        if M <= 600 and M * N * K < 3e9:
            step(f"sweep qgemm M={M} N={N} K={K}")
            codes, scales = d.quant_activations(Xd)
            c = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
            d.det_qgemm_w4a8(codes, scales, d.quant_pack_weight(up_bf16(W)), c, N)
            torch.cuda.synchronize()
            assert np.array_equal(down_bf16(c), orc.qlinear(X, *orc.quant_w4(W))), (M, N, K)


@pytest.mark.parametrize("K,N", [(4096, 4096), (4096, 6144), (4096, 28672), (14336, 4096), (2048, 32000), (5632, 2048)])
def test_every_m_from_1_to_256_keeps_row_bytes(d, orc, K, N):
    """Exhaustive over the batch sizes of the contract: for every M in 1..256 the launch on the first M rows
    gives rows 0..M-1 of the M = 256 launch byte for byte, for the bf16 GEMM and the quantized GEMM (whose
    tile shape, loader split and stage schedule are all picked from M).  Compared on the device."""
    X = ds.normal_bf16_torch(ds.tensor_seed(2, 7) + K, (256, K), 1.0, 0.0, DEV)
    W = ds.normal_bf16_torch(ds.tensor_seed(2, 900) + K // 64 + N, (K, N), 0.02, 0.0, DEV)
    Wp, Wq = d.pack_weight(W), d.quant_pack_weight(W)
    del W
    step(f"gemm every M, K={K} N={N}: M=256 reference launches")
    full = torch.empty((256, N), dtype=torch.bfloat16, device=DEV)
    d.det_gemm_bf16(X, Wp, full, N, K)
    codes, scales = d.quant_activations(X)
    qfull = torch.empty((256, N), dtype=torch.bfloat16, device=DEV)
    d.det_qgemm_w4a8(codes, scales, Wq, qfull, N)
    torch.cuda.synchronize()
    bad = []
    for M in range(1, 257):
        if M % 32 == 1:
            step(f"gemm every M, K={K} N={N}: M={M}..")
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
        d.det_gemm_bf16(X[:M], Wp, C, N, K)
        cm, sm = d.quant_activations(X[:M])
        Cq = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
        d.det_qgemm_w4a8(cm, sm, Wq, Cq, N)
        if not torch.equal(C.view(torch.int16), full[:M].view(torch.int16)):
            bad.append(("bf16", M))
        # the tiling that never looks at M gives the same bytes as the one keyed on M
        C.fill_(float("nan"))
        d.det_gemm_bf16_fixed_tile(X[:M], Wp, C, N, K)
        if not torch.equal(C.view(torch.int16), full[:M].view(torch.int16)):
            bad.append(("bf16 fixed tile", M))
        if not torch.equal(Cq.view(torch.int16), qfull[:M].view(torch.int16)):
            bad.append(("w4a8", M))
    assert not bad, bad[:10]
