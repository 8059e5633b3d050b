"""Decode attention (a workgroup for one row's chunk and KV head), alone, in a small and in a large batch: the bytes of the same sequences
in the form that takes eight rows a workgroup, at lengths around the steps, subtiles and chunks, with cache tails that are not
finite, and with the output quantized; and every chunk wherever the grid has it."""
import math

import numpy as np
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, step, up, up_bf16

pytestmark = pytest.mark.gpu

SCALE = float(np.float32(1.0 / math.sqrt(128.0)))
LENS = [700, 1, 31, 32, 33, 63, 64, 65, 0, -3, 127, 224, 225, 255, 256, 257, 288, 300, 511, 512, 513, 699]


@pytest.fixture(scope="module")
def d():
    import paper_2602_00182_amd as d
    return d


@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (16, 2), (8, 4)])
@pytest.mark.parametrize("quant", [False, True])
def test_small_launch_equals_large_launch(d, Hq, Hkv, quant):
    Lmax = 700
    B = 3 * 512 // (3 * Hkv) + len(LENS)          # several rounds of workgroups
    lens = LENS + [1] * (B - len(LENS))
    q = up_bf16(ds.normal_bf16(9500 + Hq, (B, Hq, 128)))
    k = up_bf16(ds.normal_bf16(9501 + Hq, (B, Hkv, Lmax, 128)))
    v = up_bf16(ds.normal_bf16(9502 + Hq, (B, Hkv, Lmax, 128)))
    for b, n in enumerate(lens):
        k[b, :, max(n, 0):] = float("inf")
        v[b, :, max(n, 0):] = float("nan")
    lens_t = up(np.asarray(lens, dtype=np.int32))

    def run(p, slots=None):
        n = p.stop - p.start
        ws = torch.full((d.det_attn_decode_workspace_bytes(n, Hq, 128, Lmax),), 0xFF, dtype=torch.uint8, device=DEV)
        if not quant:
            out = torch.full((n, Hq, 128), 7.0, dtype=torch.bfloat16, device=DEV)
            if slots is None:
                d.det_attn_decode(q[p], k[p], v[p], lens_t[p], out, ws, SCALE)
            else:
                d.det_attn_decode_rows(q[p], k[p], v[p], lens_t[p], slots, out, ws, SCALE)
            return out.view(torch.int16)
        codes = torch.full((n, Hq * 128), 99, dtype=torch.int8, device=DEV)
        scales = torch.full((Hq * 2, (n + 3) & ~3), 7.0, dtype=torch.float32, device=DEV)
        d.det_attn_decode_quant_q8(q[p], k[p], v[p], lens_t[p], slots, codes, scales.view(-1), ws, SCALE)
        return torch.cat([codes.view(torch.int32), scales[:, :n].t().contiguous().view(torch.int32)], 1)

    # rows that name their slots, too few to walk their chunks: eight a workgroup
    n = len(LENS)
    assert n >= 16 and -(-n // (64 // (Hq // Hkv))) * Hkv < 256
    step(f"attention by chunk, heads {Hq}/{Hkv} quant={quant}")
    want = run(slice(0, n), torch.arange(n, dtype=torch.int32, device=DEV))
    large = run(slice(0, B))
    torch.cuda.synchronize()
    assert torch.equal(large[:n], want)
    for i in range(0, n, 5):
        p = slice(i, min(i + 5, n))
        assert torch.equal(run(p), want[p]), LENS[p]


# KV heads that do and do not spread over eight XCDs by themselves, caches of odd and even numbers of chunks on both sides of the
# largest whose heads come first in the grid
@pytest.mark.parametrize("Hq,Hkv,Lmax,B", [(8, 1, 2100, 60), (4, 2, 1300, 45), (3, 3, 2048, 70), (8, 4, 1025, 30), (16, 16, 600, 12),
                                           (4, 2, 8192, 9), (4, 2, 8200, 9)])
def test_every_chunk_is_computed_whatever_the_order_of_the_grid(d, Hq, Hkv, Lmax, B):
    lens = [Lmax, 1, Lmax - 255, 256, 257, 0] + [(37 * i * i) % Lmax + 1 for i in range(B - 6)]
    q = up_bf16(ds.normal_bf16(9600 + Hq, (B, Hq, 128)))
    k = up_bf16(ds.normal_bf16(9601 + Hq, (B, Hkv, Lmax, 128)))
    v = up_bf16(ds.normal_bf16(9602 + Hq, (B, Hkv, Lmax, 128)))
    lens_t = up(np.asarray(lens, dtype=np.int32))

    def run(p):
        n = p.stop - p.start
        ws = torch.full((d.det_attn_decode_workspace_bytes(n, Hq, 128, Lmax),), 0xFF, dtype=torch.uint8, device=DEV)
        out = torch.full((n, Hq, 128), 7.0, dtype=torch.bfloat16, device=DEV)
        d.det_attn_decode(q[p], k[p], v[p], lens_t[p], out, ws, SCALE)
        return out.view(torch.int16)

    step(f"attention of {B} rows, heads {Hq}/{Hkv}, cache of {Lmax}")
    want = run(slice(0, B))
    for b in range(B):
        assert torch.equal(run(slice(b, b + 1)), want[b:b + 1]), lens[b]
    torch.cuda.synchronize()


# numbers of chunks with every power of two in them that the chunks' places turn by, up to the whole number, and the smallest
@pytest.mark.parametrize("Hq,Hkv,Lmax,B", [(16, 16, 200, 40), (16, 16, 512, 40), (8, 4, 1024, 64), (4, 2, 3072, 45), (8, 2, 4096, 33),
                                           (4, 2, 6144, 22), (4, 4, 16384, 9)])
def test_every_chunk_is_computed_wherever_it_is_placed(d, Hq, Hkv, Lmax, B):
    test_every_chunk_is_computed_whatever_the_order_of_the_grid(d, Hq, Hkv, Lmax, B)
