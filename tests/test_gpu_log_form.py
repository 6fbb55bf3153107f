"""Rounding of the FP64 log form where logarithms are small. Without data every
parent set weighs rho(|G|) = 1, so the posterior of an edge is the rational
    P(u -> v) = 1/n sum_s s/(n-1) K(s-1, d-1) / K(s, d),  K(s, d) = sum_k<=d C(s, k),
for every u, v and whatever q is; q(s) = 1 / ((s + 1) K(s, d)) makes every
forward and backward sum a power of 2 at most, F(V) = 1.

Tolerance: no logarithm on the way is larger than A = n ln 2 + ln n, and about
2 n sums and products of such logarithms lie between the scores and a
posterior, each rounded to half a spacing of A."""
from fractions import Fraction
from math import comb, fsum, log

import numpy as np
import pytest

import paper_1408_1664_amd as bn


@pytest.mark.gpu
@pytest.mark.parametrize("n", [2, 3, 6, 9, 10, 11, 12, 13, 14, 16, 20])
def test_small_logarithms(n):
    d = min(3, n - 1)
    K = lambda s, t: sum(comb(s, k) for k in range(t + 1))
    log_q = np.array([-log((s + 1) * K(s, d)) for s in range(n)])
    want = float(sum(Fraction(s, n - 1) * Fraction(K(s - 1, d - 1), K(s, d))
                     for s in range(1, n)) / n)
    log_lv = fsum(list(log_q) + [log((s + 1) * K(s, d)) for s in range(n)])
    print(f"small logarithms n={n}", flush=True)
    post, rep = bn.edge_posteriors(np.zeros((n, 0), np.uint8), np.full(n, 2, np.uint8), d,
                                   precision="fp64", log_rho=np.zeros(d + 1), log_q=log_q)
    tol = n * np.spacing(n * log(2) + log(n))
    off = post[~np.eye(n, dtype=bool)]
    print(f"  max error {np.abs(off / want - 1).max():.2e} of {tol:.2e}", flush=True)
    assert np.abs(off / want - 1).max() <= tol
    assert abs(rep["log_LV"] - log_lv) <= tol
    assert rep["max_invariant_residual"] <= tol


@pytest.mark.gpu
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-5)])
@pytest.mark.parametrize("n,d", [(10, 3), (11, 4), (12, 3), (13, 3)])
def test_wide_ranges_of_small_lattices(n, d, precision, tol):
    """Near-copies over 3000 samples: nodes of a small lattice beyond the range
    of one FP64 scale beside nodes within it, and Gamma outputs below 2^-1000 of
    the largest product, which rerun in the number system. Against the oracle."""
    from oracle import oracle as O
    rng = np.random.default_rng(11)
    data = rng.integers(0, 2, (n, 3000)).astype(np.uint8)
    for j in range(1, 4):
        data[j] = data[0] ^ (rng.random(3000) < 0.01)
    arity = np.full(n, 2, np.uint8)
    print(f"wide ranges n={n} d={d} {precision}", flush=True)
    post, rep = bn.edge_posteriors(data, arity, d, precision=precision)
    ref = O.edge_posteriors(data, arity, d, ess=1.0)
    assert np.abs(post - ref["post"]).max() <= tol
    assert abs(rep["log_LV"] - ref["log_LV"]) <= 1e-9 * abs(ref["log_LV"])
