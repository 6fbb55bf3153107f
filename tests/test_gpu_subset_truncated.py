"""The truncated upward transform skips rows without inputs: what lies in the
entries with more than d ones must not matter, and every output must be written.
Sizes at each split of the high bits into passes (one pass of 1..9 bits, two
passes whose first takes 1..9), d from 0 to nbits - 1; integer inputs, compared
bit for bit with the dense definition computed by untruncated steps."""
import numpy as np
import pytest
import torch

import paper_1408_1664_amd as bn


def _dense(x, nbits, d):
    pop = np.array([bin(i).count("1") for i in range(1 << 12)], dtype=np.int8)
    idx = np.arange(1 << nbits)
    ones = pop[idx & 0xfff] + pop[idx >> 12 & 0xfff] + pop[idx >> 24]
    y = np.where(ones <= d, x, 0.0)
    for b in range(nbits):
        v = y.reshape(-1, 2, 1 << b)
        v[:, 1] += v[:, 0]
    return y


@pytest.mark.gpu
@pytest.mark.parametrize("nbits,d", [(12, 3), (13, 0), (13, 2), (15, 14), (16, 3), (17, 1), (19, 5),
                                     (20, 4), (21, 3), (22, 0), (22, 2), (22, 21), (23, 3), (24, 4)])
def test_truncated_transform(nbits, d):
    print(f"truncated transform nbits={nbits} d={d}", flush=True)
    rng = np.random.default_rng(nbits * 32 + d)
    x = rng.integers(-1000, 1001, 1 << nbits).astype(np.float64)
    want = _dense(x, nbits, d)
    y = torch.from_numpy(x).cuda()
    bn.subset_transform(y, "zeta_up", d)
    assert np.array_equal(y.cpu().numpy(), want)
    # entries that are no inputs may hold anything
    pop = np.array([bin(i).count("1") for i in range(1 << 12)], dtype=np.int8)
    idx = np.arange(1 << nbits)
    z = np.where(pop[idx & 0xfff] + pop[idx >> 12 & 0xfff] > d, np.nan, x)
    y = torch.from_numpy(z).cuda()
    bn.subset_transform(y, "zeta_up", d)
    assert np.array_equal(y.cpu().numpy(), want)
