"""Local scores by sets of variables (one arity, d <= 4): every family of a set
from one table of counts. Sizes at the edges: sample counts below one group of
four and around a wave's step, in-degree bounds of n - 1 and above, tables from
one variable to 2048 cells. Against the oracle, with the tolerance of the other
score tests."""
import numpy as np
import pytest

import paper_1408_1664_amd as bn
from oracle import oracle as O
from paper_1408_1664_amd import datagen


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["bdeu", "k2"])
@pytest.mark.parametrize("n,r,d,m", [(2, 3, 1, 1), (4, 3, 7, 3), (6, 3, 4, 255), (9, 4, 4, 259),
                                     (7, 6, 3, 64), (12, 3, 0, 130), (20, 3, 2, 1001)])
def test_scores_by_sets(n, r, d, m, kind):
    ds = datagen.random_dag_dataset(n, m, r, min(3, n - 1), 1.0, seed=50 + n + r)
    print(f"score sets n={n} r={r} d={d} m={m} {kind}", flush=True)
    got = bn.local_scores(ds.data, ds.arity, d, score=kind, ess=1.5)
    ref = O.local_scores(ds.data, ds.arity, d, O.K2 if kind == "k2" else O.BDEU, 1.5)
    masks = [x for k in range(min(d, n - 1) + 1) for x in range(1 << (n - 1))
             if bin(x).count("1") == k]
    for i in range(n):
        at = [(x & ((1 << i) - 1)) | ((x >> i) << (i + 1)) for x in masks]
        np.testing.assert_allclose(got[i], ref[i, at], rtol=1e-12, atol=1e-10)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["bdeu", "k2"])
@pytest.mark.parametrize("n,d,m", [(2, 1, 1), (3, 7, 31), (6, 4, 33), (17, 2, 64), (18, 4, 700),
                                   (12, 0, 100), (31, 1, 95)])
def test_binary_scores_by_sets(n, d, m, kind):
    """Sets counted from bit planes, 16 lanes each: n around the 16 lanes that
    unrank a set, sample counts around a plane's word."""
    ds = datagen.random_dag_dataset(n, m, 2, min(3, n - 1), 1.0, seed=60 + n)
    print(f"binary score sets n={n} d={d} m={m} {kind}", flush=True)
    got = bn.local_scores(ds.data, ds.arity, d, score=kind, ess=1.5)
    if n <= 18:
        ref = O.local_scores(ds.data, ds.arity, d, O.K2 if kind == "k2" else O.BDEU, 1.5)
        masks = [x for k in range(min(d, n - 1) + 1) for x in range(1 << (n - 1))
                 if bin(x).count("1") == k]
        for i in range(n):
            at = [(x & ((1 << i) - 1)) | ((x >> i) << (i + 1)) for x in masks]
            np.testing.assert_allclose(got[i], ref[i, at], rtol=1e-12, atol=1e-10)
        return
    # one parent at most: each row against the same pair of variables alone
    for i, j in [(0, 1), (0, n - 1), (n - 1, 0), (15, 16), (16, 15), (n - 2, n - 1)]:
        pair = bn.local_scores(ds.data[[i, j]], [2, 2], 1, score=kind, ess=1.5)
        np.testing.assert_allclose(got[i, [0, 1 + (j if j < i else j - 1)]], pair[0], rtol=1e-12,
                                   atol=1e-10)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["bdeu", "k2"])
@pytest.mark.parametrize("n,r,d,m", [(3, 2, 1, 40), (12, 2, 4, 2000), (17, 2, 3, 700), (11, 3, 4, 1000),
                                     (14, 3, 2, 999), (9, 4, 4, 300), (8, 6, 3, 500), (4, 45, 1, 3000)])
def test_sets_score_as_families_do(n, r, d, m, kind):
    """Scoring a set's families together changes no bit of any score: against
    the same data beside one variable of another arity, whose families are
    scored one by one. Its parent sets without that variable are ranked first
    within each size, in the same order."""
    ds = datagen.random_dag_dataset(n, m, r, min(3, n - 1), 0.5, seed=80 + n + r)
    print(f"score sets against families n={n} r={r} d={d} m={m} {kind}", flush=True)
    got = bn.local_scores(ds.data, ds.arity, d, score=kind, ess=1.5)
    other = np.arange(m, dtype=np.uint8)[None] % (r + 1)
    mixed = bn.local_scores(np.vstack([ds.data, other]), np.append(ds.arity, r + 1), d, score=kind,
                            ess=1.5)
    K = [bn.num_parent_sets(n + 1, k) for k in range(-1, d + 1)]
    L = [bn.num_parent_sets(n, k) for k in range(-1, d + 1)]
    at = np.concatenate([np.arange(K[k], K[k] + L[k + 1] - L[k]) for k in range(d + 1)])
    assert np.array_equal(got, mixed[:n, at])


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,m", [(2, 1, 2016), (2, 1, 2017), (3, 2, 2049), (8, 4, 4096), (10, 3, 2081),
                                   (13, 4, 2048), (13, 4, 2016), (16, 4, 2048)])
def test_a_wave_per_binary_set(n, d, m):
    """Few binary sets with many samples take a wave each (from 64 words of
    samples on): the same bits as family by family, at word counts around the
    64 lanes and on both sides of the number of sets."""
    test_sets_score_as_families_do(n, 2, d, m, "bdeu")
