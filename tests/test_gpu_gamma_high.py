"""Gamma's one-level high-bit pass, 2^(12 - hv) ranks per workgroup, at the sizes
where its layout changes: no high bit (n = 12), rows of one lane's width and
below (n = 13, 16), rows over lanes and registers (n = 19, 21), and the largest
(n = 23: 11 and 10 bits, n = 24: 12 and 11). Against the oracle with the number
systems' tolerances, with the linear tiles on and forced to the log-add path;
at n = 23 and 24 by the invariants and the agreement of the two forms."""
import numpy as np
import pytest

import paper_1408_1664_amd as bn
from oracle import oracle as O
from paper_1408_1664_amd import datagen


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["1", "force"])
@pytest.mark.parametrize("n,d", [(10, 3), (12, 3), (13, 1), (13, 4), (16, 3), (19, 2), (21, 3)])
def test_one_level_matches_oracle(n, d, mode, monkeypatch):
    monkeypatch.setenv("BN_LINEAR_TILES", mode)
    ds = datagen.random_dag_dataset(n, 120, 2, 3, 1.0, seed=90 + n)
    ref = O.edge_posteriors(ds.data, ds.arity, d, ess=1.0)
    for precision, tol in (("fp64", 1e-10), ("fp32", 1e-5)):
        print(f"gamma one level n={n} d={d} {precision} mode={mode}", flush=True)
        post, rep = bn.edge_posteriors(ds.data, ds.arity, d, precision=precision)
        assert np.abs(post - ref["post"]).max() <= tol
        assert rep["max_invariant_residual"] <= (1e-9 if precision == "fp64" else 1e-5)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [23, 24])
def test_one_level_largest(n):
    ds = datagen.random_dag_dataset(n, 200, 2, 3, 1.0, seed=90 + n)
    print(f"gamma one level n={n}", flush=True)
    p64, r64 = bn.edge_posteriors(ds.data, ds.arity, 3, precision="fp64")
    p32, r32 = bn.edge_posteriors(ds.data, ds.arity, 3, precision="fp32")
    assert r64["max_invariant_residual"] <= 1e-9 and r32["max_invariant_residual"] <= 1e-5
    assert np.abs(p64 - p32).max() <= 1e-5
