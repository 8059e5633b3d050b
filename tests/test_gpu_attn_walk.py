"""Attention of many slot-named rows: from 256 (row tile, KV head) pairs on, a workgroup walks its rows' chunks
itself.  Every row must have the bytes it has in a call of at most 15 rows, which takes the per-chunk form that
test_gpu_attn.py holds to the fp64 definition."""
import math

import numpy as np
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, step, up, up_bf16

pytestmark = pytest.mark.gpu

SCALE = float(np.float32(1.0 / math.sqrt(128.0)))


@pytest.fixture(scope="module")
def d():
    import paper_2602_00182_amd as d
    return d


def prompts(lens):
    """Lengths and slots of the rows of whole prompts, one slot each."""
    return [p + 1 for n in lens for p in range(n)], [s for s, n in enumerate(lens) for _ in range(n)]


def scattered(R, S, longest, seed):
    """Rows in any order: lengths 0 (no tokens) .. longest, any slot."""
    r = np.random.default_rng(seed)
    return list(r.integers(0, longest + 1, R)), list(r.integers(0, S, R))


def inputs(seed, R, Hq, S, Hkv, Lmax):
    return up_bf16(ds.normal_bf16(seed, (R, Hq, 128))), up_bf16(ds.normal_bf16(seed + 1, (S, Hkv, Lmax, 128))), up_bf16(
        ds.normal_bf16(seed + 2, (S, Hkv, Lmax, 128)))


def rows_call(d, q, k, v, lens, slots, scale, quant):
    R, Hq, _ = q.shape
    Lmax = k.shape[2]
    ws = torch.full((d.det_attn_decode_workspace_bytes(R, Hq, 128, Lmax),), 0xFF, dtype=torch.uint8, device=DEV)
    lens, slots = up(np.asarray(lens, dtype=np.int32)), up(np.asarray(slots, dtype=np.int32))
    if not quant:
        out = torch.full((R, Hq, 128), 7.0, dtype=torch.bfloat16, device=DEV)
        d.det_attn_decode_rows(q, k, v, lens, slots, out, ws, scale)
        return out.view(torch.int16)
    codes = torch.full((R, Hq * 128), 99, dtype=torch.int8, device=DEV)
    scales = torch.full((Hq * 2, (R + 3) & ~3), 7.0, dtype=torch.float32, device=DEV)
    d.det_attn_decode_quant_q8(q, k, v, lens, slots, codes, scales.view(-1), ws, scale)
    return torch.cat([codes.view(torch.int32), scales[:, :R].t().contiguous().view(torch.int32)], 1)


def check(d, name, q, k, v, lens, slots, quant=False, scale=SCALE, pick=None):
    R, Hq, _ = q.shape
    Hkv = k.shape[1]
    G = Hq // Hkv
    assert -(-R * G // 64) * Hkv >= 256, "the case must reach the walking form"
    step(f"{name}: R={R} heads {Hq}/{Hkv} quant={quant}")
    got = rows_call(d, q, k, v, lens, slots, scale, quant)
    torch.cuda.synchronize()
    pick = list(range(R)) if pick is None else pick
    for at in range(0, len(pick), 15):
        p = pick[at:at + 15]
        want = rows_call(d, q[p].contiguous(), k, v, [lens[i] for i in p], [slots[i] for i in p], scale, quant)
        assert torch.equal(got[p], want), (name, p)


@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (32, 16), (32, 32), (64, 8)])
@pytest.mark.parametrize("quant", [False, True])
def test_rows_equal_small_calls(d, Hq, Hkv, quant):
    Lmax = 583  # not whole subtiles of 64 nor chunks of 256
    lens, slots = prompts([583, 1, 2, 63, 64, 65, 7, 3, 1, 1, 1])  # tiles of one, two and many prompts
    q, k, v = inputs(4100 + Hq + Hkv, len(lens), Hq, 11, Hkv, Lmax)
    check(d, "prompts", q, k, v, lens, slots, quant)
    lens, slots = scattered(530, 6, Lmax, 5)
    q, k, v = inputs(4200 + Hq + Hkv, 530, Hq, 6, Hkv, Lmax)
    check(d, "scattered", q, k, v, lens, slots, quant)


def test_chunk_boundaries_and_long_contexts(d):
    """Lengths on both sides of the subtile and chunk boundaries, and past the chunks whose maxima are kept."""
    Lmax = 49 * 256 + 70
    r = np.random.default_rng(8)
    edges = [64, 65, 255, 256, 257, 319, 320, 321, 511, 512, 513, 48 * 256 - 1, 48 * 256, 48 * 256 + 1, 49 * 256, 49 * 256 + 1, Lmax]
    lens = list(r.integers(1, Lmax + 1, 512))
    for i, n in enumerate(edges):
        lens[30 * i] = n
    q, k, v = inputs(4300, 512, 32, 1, 8, Lmax)
    pick = [30 * i for i in range(len(edges))] + list(range(1, 512, 17))
    check(d, "long", q, k, v, lens, [0] * 512, pick=pick)
    check(d, "long, negative scale", q, k, v, lens, [0] * 512, scale=-0.11, pick=pick[:30])


def test_infinite_and_nan_cache_rows(d):
    """A V row that is not finite reaches the rows that read it and no other; K rows likewise; cache tails reach nobody."""
    lens, slots = prompts([300, 229])
    q, k, v = inputs(4400, len(lens), 32, 2, 8, 310)
    v[0, 1, 100, 5] = float("inf")
    v[0, 2, 299, :] = float("nan")
    v[1, 3, 40, 7] = float("-inf")
    k[1, 0, 63, 3] = float("nan")
    k[0, 4, 256, :] = float("inf")
    v[0, :, 300:] = float("nan")
    k[0, :, 300:] = float("nan")
    v[1, :, 229:] = float("inf")
    check(d, "not finite", q, k, v, lens, slots)


@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (32, 16), (64, 8), (32, 32)])
@pytest.mark.parametrize("quant", [False, True])
def test_few_long_rows_among_short_ones(d, Hq, Hkv, quant):
    """Rows many times longer than the call's others are left to the per-chunk kernels, inside a tile of short rows too."""
    Lmax = 5120
    lens, slots = prompts([600])
    for at, n in ((0, 5000), (17, 4097), (18, 2049), (300, 5120), (599, 4864)):
        lens.insert(at, n)
        slots.insert(at, 1 + at % 2)
    q, k, v = inputs(4500 + Hq + Hkv, len(lens), Hq, 3, Hkv, Lmax)
    pick = [i for i, n in enumerate(lens) if n > 600] + list(range(0, len(lens), 41))
    check(d, "few long rows", q, k, v, lens, slots, quant, pick=pick)


@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (32, 16), (64, 8), (32, 32)])
@pytest.mark.parametrize("per", [2, 9, 24])
def test_slots_at_regular_intervals(d, Hq, Hkv, per):
    """Tiles of several slots, in runs of equal size that begin anywhere in a tile, with rows of no tokens among them."""
    R, S, Lmax = 541, 11, 300
    lens = [0 if i % 31 == 5 else 300 - 7 * (i % per) for i in range(R)]
    slots = [(i // per) % S for i in range(R)]
    q, k, v = inputs(4600 + Hq + Hkv + per, R, Hq, S, Hkv, Lmax)
    check(d, f"runs of {per}", q, k, v, lens, slots, pick=range(0, R, 4))
