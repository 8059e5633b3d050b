"""Decode attention (a workgroup for one row's chunk) against the same rows in the form that takes eight of them a workgroup:
every number of query heads a KV head, lengths around the steps, waves and chunks, cache tails that are not finite, scores of either sign
of scale, outputs plain and quantized."""
import numpy as np
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, step, up, up_bf16

pytestmark = pytest.mark.gpu

LENS = [600, -3, 1, 15, 16, 31, 32, 33, 63, 64, 65, 0, 127, 129, 191, 193, 223, 224, 225, 255, 256, 257, 287, 289, 511, 512, 513, 599]


@pytest.fixture(scope="module")
def d():
    import paper_2602_00182_amd as d
    return d


# three chunks, and four and eight, whose places in the grid change from stream to stream
@pytest.mark.parametrize("Lmax,longest", [(600, []), (1024, [1024, 767, 768, 769, 1023]), (2048, [2048, 1025, 1791, 1793])])
@pytest.mark.parametrize("Hq,Hkv", [(4, 4), (8, 4), (16, 4), (16, 2)])
@pytest.mark.parametrize("quant", [False, True])
@pytest.mark.parametrize("scale", [0.088, -0.3])
def test_one_row_a_workgroup_equals_eight(d, Lmax, longest, Hq, Hkv, quant, scale):
    lengths = LENS + longest
    B = len(lengths)
    assert B >= 16 and -(-B // (64 // (Hq // Hkv))) * Hkv < 256   # rows that name their slots: eight a workgroup, not the walk
    q = up_bf16(ds.normal_bf16(9700 + Hq, (B, Hq, 128)))
    k = up_bf16(ds.normal_bf16(9701 + Hq, (B, Hkv, Lmax, 128)))
    v = up_bf16(ds.normal_bf16(9702 + Hq, (B, Hkv, Lmax, 128)))
    for b, n in enumerate(lengths):
        k[b, :, max(n, 0):] = float("nan")
        v[b, :, max(n, 0):] = float("inf")
    lens = up(np.asarray(lengths, dtype=np.int32))
    slots = torch.arange(B, dtype=torch.int32, device=DEV)

    def run(named):
        ws = torch.full((d.det_attn_decode_workspace_bytes(B, Hq, 128, Lmax),), 0xFF, dtype=torch.uint8, device=DEV)
        if quant:
            codes = torch.full((B, Hq * 128), 99, dtype=torch.int8, device=DEV)
            scales = torch.full((Hq * 2, (B + 3) & ~3), 7.0, dtype=torch.float32, device=DEV)
            d.det_attn_decode_quant_q8(q, k, v, lens, slots if named else None, codes, scales.view(-1), ws, scale)
            return codes, scales[:, :B].clone().view(torch.int32)
        out = torch.full((B, Hq, 128), 7.0, dtype=torch.bfloat16, device=DEV)
        if named:
            d.det_attn_decode_rows(q, k, v, lens, slots, out, ws, scale)
        else:
            d.det_attn_decode(q, k, v, lens, out, ws, scale)
        return (out.view(torch.int16),)

    step(f"decode attention against eight rows a workgroup, cache of {Lmax}, heads {Hq}/{Hkv} quant={quant} scale={scale}")
    got, want = run(False), run(True)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
