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


@pytest.mark.gpu
@pytest.mark.parametrize("nbits,d", [(12, 5), (16, 2), (16, 3), (17, 2), (17, 3), (18, 6), (18, 12), (20, 3),
                                     (20, 7), (22, 3), (22, 5), (22, 9), (23, 12), (24, 4)])
def test_truncated_equals_dense_of_cleared(nbits, d):
    """On both sides of the rule that chooses the split of the bits and whether
    rows are skipped, in both storages: the truncated transform of an array whose
    other entries hold anything is, bit for bit, the untruncated one of the array
    with those entries cleared."""
    print(f"truncated against dense nbits={nbits} d={d}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(nbits * 32 + d)
    idx = torch.arange(1 << nbits, device="cuda")
    ones = sum((idx >> b) & 1 for b in range(nbits))
    x = torch.rand(1 << nbits, dtype=torch.float64, device="cuda", generator=gen) - 0.5
    clear = torch.where(ones <= d, x, torch.zeros_like(x))
    x = torch.where(ones <= d, x, torch.full_like(x, float("nan")))
    bn.subset_transform(x, "zeta_up", d)
    bn.subset_transform(clear, "zeta_up", -1)
    assert torch.equal(x, clear)
    f = torch.rand(1 << nbits, device="cuda", generator=gen) + 0.5
    b = torch.randint(190, 211, (1 << nbits,), device="cuda", generator=gen).to(torch.uint8)
    f0 = torch.where(ones <= d, f, torch.zeros_like(f))
    b0 = torch.where(ones <= d, b, torch.zeros_like(b))
    f = torch.where(ones <= d, f, torch.full_like(f, float("inf")))
    bn.subset_transform_x32(f, b, "zeta_up", d)
    bn.subset_transform_x32(f0, b0, "zeta_up", -1)
    assert torch.equal(f, f0) and torch.equal(b, b0)
