"""Both sweeps in one launch, over the tile widths that the plan chooses: the
whole lattice (FP32-scaled n <= 12, log form n <= 11), 11 bits, and the first
sizes with several layers of tiles. Against the oracle, with the number
systems' stated tolerances (1e-10 and 1e-5)."""
import numpy as np
import pytest

import paper_1408_1664_amd as bn
from oracle import oracle as O
from paper_1408_1664_amd import datagen


@pytest.mark.gpu
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-5)])
@pytest.mark.parametrize("n,d", [(2, 1), (3, 2), (11, 3), (12, 4), (13, 2), (15, 3), (17, 3)])
def test_sweep_tiles(n, d, precision, tol):
    ds = datagen.random_dag_dataset(n, 150, 2, 3, 1.0, seed=70 + n)
    print(f"sweep tiles n={n} d={d} {precision}", flush=True)
    post, rep = bn.edge_posteriors(ds.data, ds.arity, d, precision=precision)
    ref = O.edge_posteriors(ds.data, ds.arity, d, ess=1.0)
    assert np.abs(post - ref["post"]).max() <= tol
    assert abs(rep["log_LV"] - ref["log_LV"]) <= 1e-9 * abs(ref["log_LV"])
