"""The second pass of decode attention against the fold it stands for, computed here from the chunk partials the first pass left in the
workspace: counts of chunks around the groups whose sums are asked for together (8) and the lanes that hold their statistics (64), mixed
in one call, workspace beyond a row's chunks not finite; plain and quantized."""
import numpy as np
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, down_bf16, step, up, up_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunks", [(1, 2, 7, 8, 9), (16, 15, 17, 3), (64, 63, 56, 57), (65, 64, 66), (129, 72, 73, 128)])
def test_fold_of_the_partials(orc, chunks):
    import paper_2602_00182_amd as d
    B, Hq, Hkv, NC = len(chunks), 4, 1, max(chunks)
    Lmax, s = 256 * NC, ds.tensor_seed(6, 830) + NC
    lens = [256 * c - (5 * i) % 256 for i, c in enumerate(chunks)]
    q = ds.normal_bf16_torch(s, (B, Hq, 128), 1.0, 0.0, DEV)
    k = ds.normal_bf16_torch(s + 1, (B, Hkv, Lmax, 128), 1.0, 0.0, DEV)
    v = ds.normal_bf16_torch(s + 2, (B, Hkv, Lmax, 128), 1.0, 0.0, DEV)
    n = up(np.asarray(lens, dtype=np.int32))
    ws = torch.full((d.det_attn_decode_workspace_bytes(B, Hq, 128, Lmax),), 0xFF, dtype=torch.uint8, device=DEV)
    out = torch.full((B, Hq, 128), 7.0, dtype=torch.bfloat16, device=DEV)
    codes = torch.full((B, Hq * 128), 99, dtype=torch.int8, device=DEV)
    scales = torch.full((Hq * 2, (B + 3) & ~3), 7.0, dtype=torch.float32, device=DEV)
    step(f"decode attention, chunks {chunks}")
    d.det_attn_decode_quant_q8(q, k, v, n, None, codes, scales.view(-1), ws, 0.088)  # (keeps the partials of rows of one chunk as well)
    torch.cuda.synchronize()
    parts = ws.cpu().numpy()[:B * Hq * NC * 130 * 4].view(np.float32)
    m, l, o = (parts[a * B * Hq * NC:b * B * Hq * NC].reshape(B, Hq, NC, -1) for a, b in ((0, 1), (1, 2), (2, 130)))
    want = np.empty((B, Hq, 128), np.float32)
    for b, c in enumerate(chunks):
        for h in range(Hq):
            w = orc.expf(m[b, h, :c, 0] - m[b, h, :c, 0].max())
            L, O = np.float32(0), np.zeros(128, np.float32)
            for i in range(c):
                L, O = L + w[i] * l[b, h, i, 0], O + w[i] * o[b, h, i]
            want[b, h] = O / L
    want = orc.bf16_rne(want)
    d.det_attn_decode(q, k, v, n, out, ws, 0.088)
    wc, wscales = d.quant_activations(up_bf16(want.reshape(B, Hq * 128)))
    torch.cuda.synchronize()
    assert np.array_equal(down_bf16(out), want)
    assert torch.equal(codes, wc)
    assert torch.equal(scales[:, :B].contiguous().view(torch.int32), wscales.view(Hq * 2, -1)[:, :B].contiguous().view(torch.int32))
