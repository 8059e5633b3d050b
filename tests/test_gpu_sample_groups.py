"""Seeded sampling where the candidates come from group maxima: top-k on both sides of every group size, rows of every number of logits
a thread, whole and broken into 16-byte pieces, and temperatures whose quotients tie, vanish or overflow; against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    import paper_2602_00182_amd as d
    return d


def rows(V, seed):
    r = np.random.default_rng(seed)
    x = (r.standard_normal((6, V)) * 2.5).astype(np.float32)
    x[1] = np.round(x[1] * 2) / 2                      # ties
    x[2, V // 3:] = -np.inf                            # fewer candidates than k in some groups
    x[3] *= np.float32(1e-30)                          # quotients that lose digits at large temperatures
    x[4, ::2] = 0.0
    x[4, 1::4] = -0.0                                  # zeros of either sign at the bound
    x[4, 3::4] = -1.0
    x[5, r.integers(0, V, 5)] = np.nan
    return x


def check(d, orc, x, k, T):
    B = len(x)
    ids, steps = np.arange(B, dtype=np.int32), np.full(B, 17, np.int32)
    out = torch.full((B,), -1, dtype=torch.int32, device=DEV)
    step(f"sampling V={x.shape[1]} top-k {k} temperature {T}")
    d.det_sample(torch.from_numpy(x).to(DEV), T, k, 0.95, 99, torch.from_numpy(ids).to(DEV), torch.from_numpy(steps).to(DEV), out)
    assert np.array_equal(out.cpu().numpy(), orc.sample(x, T, k, 0.95, 99, ids, steps))


@pytest.mark.parametrize("V", [513, 4095, 4096, 8192, 8196, 32768, 32772])
@pytest.mark.parametrize("k", [1, 64, 65, 128, 129, 256, 257])
def test_sizes(d, orc, V, k):
    check(d, orc, rows(V, V + k), k, 0.8)


@pytest.mark.parametrize("T", [1e-38, 1e-3, 1.0, 3.7, 1e10, 1e38])
@pytest.mark.parametrize("k", [50, 100])
def test_temperatures(d, orc, T, k):
    check(d, orc, rows(5000, k), k, T)


# Divided by an infinite temperature, +inf is no number and comes behind the finite logits, which are all zeros.  Rows where groups of
# either kind are fewer than k, both together more.  A call before it leaves sorted lists of its own in every compute unit's LDS.
@pytest.mark.parametrize("V", [513, 5000, 8201, 40000])
@pytest.mark.parametrize("k", [2, 50, 100, 200, 300])
def test_infinite_temperature(d, orc, V, k):
    x = np.full((8, V), -np.inf, np.float32)
    x[0, 0], x[0, 8 * (V // 16)] = np.inf, 5.0
    for row, apart in zip(x[1:4], (4, 16, 64)):
        row[::apart], row[apart // 2::apart] = np.inf, 5.0
    x[4:6] = rows(V, V + k)[[0, 5]]
    x[5, ::7] = np.inf
    x[6] = np.inf
    before = np.random.default_rng(V).standard_normal((1024, V)).astype(np.float32) + 60
    n = torch.zeros(1024, dtype=torch.int32, device=DEV)
    d.det_sample(torch.from_numpy(before).to(DEV), 1.0, 1000, 0.95, 99, n, n, torch.empty_like(n))
    check(d, orc, x, k, float("inf"))
