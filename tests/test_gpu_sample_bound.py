"""det_sample where its candidates come from the threads' maxima (top-k up to 256): the oracle's tokens on both sides of
that limit, with rows shorter than the workgroup, with ties at the bound, and with more keys at the bound than are ranked."""
import numpy as np
import pytest
import torch

import detsynth as ds
from gpu_util import DEV, step, up

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def d():
    import paper_2602_00182_amd as d
    return d


@pytest.mark.parametrize("V", [1, 255, 1023, 1024, 1025, 8003, 40000])
@pytest.mark.parametrize("k", [1, 2, 17, 255, 256, 257])
def test_tokens_match_oracle(d, orc, V, k):
    B = 12
    x = (ds.bf16_bits_to_f32(ds.normal_bf16(9000 + V + k, (B, V))) * np.float32(2.0)).astype(np.float32)
    x[1] = np.round(x[1])                              # a few dozen values: every bound is tied
    x[2] = 0.25                                        # one value: more ties than are ranked
    x[3, : V // 2] = 1.0e30                            # half the row above the rest, all tied
    x[4, ::3] = -np.inf
    x[5, ::2] = np.nan
    x[6] = -np.inf
    x[7] = x[7] * np.float32(1e-42)                    # denormal and equal scaled logits
    x[8, :: max(1, V // 5)] = np.inf
    x[9] = np.sort(x[9])                               # the candidates all with the last threads
    x[10] = np.sort(x[10])[::-1]
    ids = np.arange(B, dtype=np.int32) * 3
    steps = np.arange(B, dtype=np.int32)
    step(f"sample bound V={V} k={k}")
    tok = torch.full((B,), -1, dtype=torch.int32, device=DEV)
    d.det_sample(up(x), 0.8, k, 0.97, 77, up(ids), up(steps), tok)
    torch.cuda.synchronize()
    assert np.array_equal(tok.cpu().numpy(), orc.sample(x, 0.8, k, 0.97, 77, ids, steps))
