"""Device memory that finished blocking calls keep: given back on request, after
which calls run as before, and a failed call leaves nothing behind."""
import numpy as np
import pytest

import paper_1408_1664_amd as bn
from paper_1408_1664_amd import datagen


def _free_bytes():
    import torch
    return torch.cuda.mem_get_info()[0]


@pytest.mark.gpu
def test_release_idle_gives_the_memory_back():
    ds = datagen.random_dag_dataset(19, 200, 2, 3, 1.0, seed=5)
    size = bn.workspace_bytes(19, 3, 200, "fp32")
    assert 16 << 20 < size < 60 << 20
    want, _ = bn.edge_posteriors(ds.data, ds.arity, 3, precision="fp32")
    bn.release_idle()
    before = _free_bytes()
    bn.edge_posteriors(ds.data, ds.arity, 3, precision="fp32")
    assert _free_bytes() <= before - size
    bn.release_idle()
    assert _free_bytes() >= before - (2 << 20)
    got, rep = bn.edge_posteriors(ds.data, ds.arity, 3, precision="fp32")
    assert np.array_equal(got, want) and rep["ms_total"] > 0
    bn.release_idle()


@pytest.mark.gpu
def test_problem_too_large_for_the_device():
    """Refused before anything runs; the next call works."""
    ds = datagen.random_dag_dataset(8, 50, 2, 2, 1.0, seed=6)
    want, _ = bn.edge_posteriors(ds.data, ds.arity, 2, precision="fp64")
    big = np.zeros((31, 4), np.uint8)
    with pytest.raises(bn.BnError, match="memory"):
        bn.edge_posteriors(big, np.full(31, 2, np.uint8), 5, precision="fp64")
    got, _ = bn.edge_posteriors(ds.data, ds.arity, 2, precision="fp64")
    assert np.array_equal(got, want)
