"""Calls of many slot-named rows with few rows a slot: groups of at most sixteen (row, head) pairs in tiles that name several
slots, taken a chunk at a time with K and V read once.  Every row must have the bytes it has in a call of at most 15 rows."""
import numpy as np
import pytest

from test_gpu_attn_walk import check, d, inputs, pytestmark  # noqa: F401

HEADS = [(32, 8), (32, 16), (64, 8), (32, 32)]


def runs(R, S, sizes, lens_of):
    """R rows in runs of the given sizes in turn, run i on slot i % S; lens_of(i, j): length of row j of run i."""
    lens, slots, i = [], [], 0
    while len(lens) < R:
        for j in range(sizes[i % len(sizes)]):
            lens.append(lens_of(i, j))
            slots.append(i % S)
        i += 1
    return lens[:R], slots[:R]


@pytest.mark.parametrize("Hq,Hkv", HEADS)
@pytest.mark.parametrize("quant", [False, True])
def test_rows_a_slot(d, Hq, Hkv, quant):
    """One row a slot, and runs on both sides of sixteen pairs, lengths around the subtiles and chunks."""
    edges = [1, 63, 64, 65, 127, 192, 193, 255, 256, 257, 319, 511, 512, 513, 700]
    R, Lmax = 530, 700
    q, k, v = inputs(7100 + Hq + Hkv, R, Hq, 40, Hkv, Lmax)
    lens, slots = runs(R, 40, [1], lambda i, j: edges[i % len(edges)])
    check(d, "a row a slot", q, k, v, lens, slots, quant, pick=range(0, R, 5))
    lens, slots = runs(R, 40, [2, 16 * Hkv // Hq, 1, 16 * Hkv // Hq + 1, 3], lambda i, j: max(0, edges[i % len(edges)] - j))
    check(d, "runs", q, k, v, lens, slots, quant, pick=range(0, R, 5))


@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (32, 32)])
@pytest.mark.parametrize("quant", [False, True])
def test_chunks_kept_in_registers_and_in_the_workspace(d, Hq, Hkv, quant):
    """Eight chunks and nine, the last lengths that do not walk and the first that do, rows of one group chunks apart."""
    Lmax = 81 * 256 + 3
    edges = [8 * 256, 8 * 256 + 1, 9 * 256 - 1, 16 * 256 + 130, 80 * 256, 80 * 256 + 1, Lmax, 300]
    R = 512
    q, k, v = inputs(7200 + Hkv, R, Hq, 2, Hkv, Lmax)
    lens, slots = runs(R, 2, [2], lambda i, j: edges[i % len(edges)] - 1500 * j if edges[i % len(edges)] > 2000 else edges[i % len(edges)])
    check(d, "chunks", q, k, v, lens, slots, quant, pick=range(0, 48))


def test_scale_of_either_sign_and_values_that_are_not_finite(d):
    R, Lmax = 512, 600
    q, k, v = inputs(7300, R, 32, 30, 8, Lmax)
    r = np.random.default_rng(3)
    lens, slots = runs(R, 30, [1, 3, 2], lambda i, j: int(r.integers(0, Lmax + 1)))
    check(d, "negative scale", q, k, v, lens, slots, scale=-0.11, pick=range(0, R, 5))
    v[3, 1, 100, 5] = float("inf")
    v[4, :, 300:] = float("nan")
    v[7, 2, 40, :] = float("-inf")
    k[9, 3, 63, 3] = float("nan")
    k[12, :, 256, :] = float("inf")
    for quant in (False, True):
        check(d, "not finite", q, k, v, lens, slots, quant, pick=range(0, R, 2))
