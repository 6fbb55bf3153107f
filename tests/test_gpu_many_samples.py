"""Bit planes of many binary samples: more 64-sample groups than one launch has
waves for, and more than 2^32 samples in all variables together (4.4 GB of data).
Without parents a score is a function of one count: BDeu with ess = 1,
lgamma(1/2 + c) + lgamma(1/2 + m - c) - 2 lgamma(1/2) - lgamma(1 + m)."""
from math import lgamma

import numpy as np
import pytest

import paper_1408_1664_amd as bn


@pytest.mark.gpu
@pytest.mark.parametrize("n,m", [(18, 300_000), (22, 200_000_000)])
def test_counts_of_many_samples(n, m):
    print(f"many samples n={n} m={m}", flush=True)
    data = np.zeros((n, m), np.uint8)
    ones = [1 + m // 7 + 1009 * j for j in range(n)]
    for j, c in enumerate(ones):
        data[j, m - c:] = 1
        data[j, :j] = 1
    got = bn.local_scores(data, np.full(n, 2, np.uint8), 0)
    bn.release_idle()
    want = [lgamma(0.5 + c + j) + lgamma(0.5 + m - c - j) - 2 * lgamma(0.5) - lgamma(1.0 + m)
            for j, c in enumerate(ones)]
    np.testing.assert_allclose(got[:, 0], want, rtol=1e-12)
