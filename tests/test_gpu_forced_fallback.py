"""The forced fallback of the Gamma tiles on data whose endpoints also fail
every FP64 scale (near-copies over 3000 samples; with d = 5 a tile has 1586
outputs, more than the last chance holds). The list of forced tiles must then
hold the tiles and nothing else: the reported count is one per alpha tile and
one per Gamma tile. Against the oracle at the number systems' tolerances."""
import numpy as np
import pytest

import paper_1408_1664_amd as bn
from oracle import oracle as O


@pytest.mark.gpu
@pytest.mark.parametrize("n,d", [(12, 5), (14, 5), (14, 3)])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32", 1e-5)])
def test_forced_list_holds_the_tiles(n, d, precision, tol, monkeypatch):
    rng = np.random.default_rng(11)
    data = rng.integers(0, 2, (n, 3000)).astype(np.uint8)
    for j in range(1, 4):
        data[j] = data[0] ^ (rng.random(3000) < 0.01)
    arity = np.full(n, 2, np.uint8)
    monkeypatch.setenv("BN_LINEAR_TILES", "force")
    print(f"forced fallback n={n} d={d} {precision}", flush=True)
    post, rep = bn.edge_posteriors(data, arity, d, precision=precision)
    alpha_tiles = n << (n - 14) if n >= 14 else 0
    assert rep["fallback_tiles"] == alpha_tiles + (1 << (n - 12))
    ref = O.edge_posteriors(data, arity, d, ess=1.0)
    assert np.abs(post - ref["post"]).max() <= tol
