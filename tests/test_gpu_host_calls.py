"""Blocking calls share idle workspaces: results must not depend on the calls
before or beside them. Sizes around the kept block (64 MiB) and the staged
transfer (1 MiB), from several threads, bit for bit against the first answers."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import paper_1408_1664_amd as bn
from paper_1408_1664_amd import datagen

CALLS = [(12, 300, 3, "fp32"), (20, 700, 3, "fp64"), (5, 0, 2, "fp64"), (16, 90, 4, "fp32"),
         (21, 64, 2, "fp32"), (18, 700, 3, "fp32")]


def _answer(call):
    n, m, d, precision = call
    ds = datagen.random_dag_dataset(n, m, 2, 3, 1.0, seed=10 * n + m)
    ps, post, rep = bn.parent_set_posteriors(ds.data, ds.arity, d, precision=precision)
    post2, _ = bn.edge_posteriors(ds.data, ds.arity, d, precision=precision)
    scores = bn.local_scores(ds.data, ds.arity, d)
    one = bn.modular_feature_posterior(ds.data, ds.arity, d, np.zeros_like(scores),
                                       precision=precision)
    assert np.array_equal(post, post2)
    assert one["value"] == pytest.approx(1.0, abs=1e-12)
    return ps, post, scores, np.array([rep["log_LV"]])


@pytest.mark.gpu
def test_blocking_calls_are_independent():
    first = [_answer(c) for c in CALLS]
    order = [k for _ in range(3) for k in range(len(CALLS))]
    with ThreadPoolExecutor(6) as pool:
        for k, got in zip(order, pool.map(lambda k: _answer(CALLS[k]), order)):
            for x, y in zip(first[k], got):
                assert np.array_equal(x, y), CALLS[k]
