"""The 13-bit alpha tile on plain doubles against the same solve with every
tile computed in the number system (BN_LINEAR_TILES=force): one tile per node
(n = 14), parent sets of up to all 13 bits of it (d beyond the ten low bits,
seeds beyond two per thread), several tiles per workgroup (n = 20, 21). Both
forms meet the number systems' stated tolerances (1e-10 and 1e-5) against the
exact posteriors, so they differ by at most twice those."""
import numpy as np
import pytest

import paper_1408_1664_amd as bn
from paper_1408_1664_amd import datagen


@pytest.mark.gpu
@pytest.mark.parametrize("precision,tol", [("fp64", 2e-10), ("fp32", 2e-5)])
@pytest.mark.parametrize("n,d", [(14, 1), (14, 3), (14, 5), (14, 10), (14, 11), (14, 13),
                                 (15, 4), (16, 6), (20, 2), (20, 6), (21, 4)])
def test_alpha_tile_equals_number_system(n, d, precision, tol, monkeypatch):
    ds = datagen.random_dag_dataset(n, 120, 2, 3, 1.0, seed=90 + n)
    print(f"alpha tile n={n} d={d} {precision}", flush=True)
    post, rep = bn.edge_posteriors(ds.data, ds.arity, d, precision=precision)
    monkeypatch.setenv("BN_LINEAR_TILES", "force")
    ref, rref = bn.edge_posteriors(ds.data, ds.arity, d, precision=precision)
    assert np.abs(post - ref).max() <= tol
    assert abs(rep["log_LV"] - rref["log_LV"]) <= 1e-9 * abs(rref["log_LV"])
