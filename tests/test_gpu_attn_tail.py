"""What a cache slot holds at and past a row's length reaches no output of that row, whichever form of the attention runs it:
rows of one slot and many lengths share a workgroup, V rows between those lengths are not finite, and every row must have
the bytes it has in a call of its own, which never reads past it."""
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


def rows_call(d, q, k, v, lens, slots, quant):
    R, Hq, _ = q.shape
    ws = torch.full((d.det_attn_decode_workspace_bytes(R, Hq, 128, k.shape[2]),), 0xFF, dtype=torch.uint8, device=DEV)
    lens, slots = up(np.asarray(lens, dtype=np.int32)), up(np.asarray(slots, dtype=np.int32))
    if not quant:
        out = torch.full((R, Hq, 128), 7.0, dtype=torch.bfloat16, device=DEV)
        d.det_attn_decode_rows(q, k, v, lens, slots, out, ws, SCALE)
        return out.view(torch.int16)
    codes = torch.full((R, Hq * 128), 99, dtype=torch.int8, device=DEV)
    scales = torch.full((Hq * 2, (R + 3) & ~3), 7.0, dtype=torch.float32, device=DEV)
    d.det_attn_decode_quant_q8(q, k, v, lens, slots, codes, scales.view(-1), ws, SCALE)
    return torch.cat([codes.view(torch.int32), scales[:, :R].t().contiguous().view(torch.int32)], 1)


def check(d, name, seed, Hq, Hkv, S, Lmax, lens, slots, poison, quant, pick):
    q = up_bf16(ds.normal_bf16(seed, (len(lens), Hq, 128)))
    k, v = (up_bf16(ds.normal_bf16(seed + i, (S, Hkv, Lmax, 128))) for i in (1, 2))
    for slot, token, value in poison:
        v[slot, :, token, 3::17] = value
        k[slot, 0, token, 5] = value
    step(f"{name}: R={len(lens)} heads {Hq}/{Hkv} quant={quant}")
    got = rows_call(d, q, k, v, lens, slots, quant)
    torch.cuda.synchronize()
    for i in pick:
        want = rows_call(d, q[i:i + 1].contiguous(), k, v, lens[i:i + 1], slots[i:i + 1], quant)
        assert torch.equal(got[i:i + 1], want), (name, i, lens[i])


@pytest.mark.parametrize("Hq,Hkv", [(16, 16), (32, 16), (32, 8), (64, 8)])
@pytest.mark.parametrize("quant", [False, True])
def test_eight_rows_a_workgroup(d, Hq, Hkv, quant):
    """Calls of sixteen to a hundred rows: lengths ascending, mixed, and two slots in one workgroup."""
    lens = list(range(250, 290)) + [700, 3, 130, 129, 700, 256, 512, 1] + [300, 290, 300, 290, 0, 300, 290, 2]
    slots = [0] * 48 + [0, 1, 0, 1, 0, 1, 0, 1]
    poison = [(0, 254, float("inf")), (0, 258, float("nan")), (0, 285, float("-inf")), (0, 130, float("nan")), (0, 600, float("inf")),
              (1, 295, float("nan"))]
    check(d, "rows of eight", 6100 + Hq + Hkv, Hq, Hkv, 2, 700, lens, slots, poison, quant, range(len(lens)))


@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (32, 32)])
@pytest.mark.parametrize("quant", [False, True])
def test_long_rows_among_short_ones(d, Hq, Hkv, quant):
    """Rows that a call of many rows leaves to the per-chunk kernels: five of one slot, many times longer than the others."""
    lens, slots = [p + 1 for p in range(600)], [0] * 600
    for at, n in ((0, 5000), (1, 4097), (2, 2049), (3, 4990), (4, 4870)):
        lens.insert(at, n)
        slots.insert(at, 1)
    poison = [(1, 4995, float("nan")), (1, 2100, float("inf")), (1, 4880, float("inf")), (0, 300, float("nan"))]
    check(d, "long rows", 6200 + Hq + Hkv, Hq, Hkv, 2, 5120, lens, slots, poison, quant, list(range(5)) + [305, 306, 420, 604])


@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (32, 16), (64, 8), (32, 32)])
@pytest.mark.parametrize("quant", [False, True])
def test_many_slots_a_tile(d, Hq, Hkv, quant):
    """Rows of a call of many rows whose neighbours name other slots."""
    r = np.random.default_rng(61)
    lens, slots = [int(x) for x in r.integers(0, 584, 530)], [int(x) for x in r.integers(0, 6, 530)]
    poison = [(s, t, float(x)) for s, t, x in ((0, 500, "nan"), (1, 250, "inf"), (2, 80, "-inf"), (3, 580, "nan"), (4, 3, "inf"))]
    check(d, "many slots", 6300 + Hq + Hkv, Hq, Hkv, 6, 583, lens, slots, poison, quant, range(0, 530, 9))


@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (32, 16), (64, 8), (32, 32)])
@pytest.mark.parametrize("quant", [False, True])
def test_long_rows_all_over_a_call(d, Hq, Hkv, quant):
    """Seventy long rows of three slots scattered over seven hundred short ones."""
    r = np.random.default_rng(62)
    lens, slots = [int(x) for x in r.integers(0, 50, 700)], [0] * 700
    at = sorted(int(x) for x in r.choice(700, 70, replace=False))
    for i in at:
        lens[i], slots[i] = int(r.integers(2049, 2900)), int(r.integers(1, 4))
    check(d, "long rows all over", 6400 + Hq + Hkv, Hq, Hkv, 4, 2900, lens, slots, [(1, 2500, float("inf"))], quant, at + list(range(0, 700, 37)))
