"""The workloads whose time this library is held to, each a call that its users make.

The problem sizes are those of ``paper_1408_1664_amd.datagen``: its named
workloads (n = 12, 20, 25 and 30), the range of its serving stream (n in
10..22, m in 100..2000, two or three states) and its subset-transform sizes.

* ``solve``: all edge posteriors of one dataset that is already on the GPU, in
  the caller's workspace and on the caller's stream (edge_posteriors_dev).
* ``serve``: a burst of requests of mixed sizes through one Server.
* ``parents``: the posterior of every parent set, host arrays in and out.
* ``scores``: the table of local scores, host arrays in and out.
* ``transform``: the zeta transform of a function on the subset lattice.
"""
from itertools import combinations
from math import comb

import numpy as np
import torch

import paper_1408_1664_amd as bn
from paper_1408_1664_amd import datagen


def _solve(name, n, m, arity, maxdeg, a, d, precision):
    return dict(name=name, kind="solve", n=n, m=m, arity=arity, maxdeg=maxdeg, a=a, d=d,
                precision=precision)


def listed():
    return [
        # the smallest served problem, alone: launches and latency
        _solve("n10_binary_m300_d3_fp32", 10, 300, 2, 3, 1.0, 3, "fp32"),
        # a small study in the plain FP64 form (workload n12_binary_m200_d3)
        _solve("n12_binary_m200_d3_fp64", 12, 200, 2, 3, 1.0, 3, "fp64"),
        # the middle of the served range, three states
        _solve("n16_ternary_m1000_d3_fp32", 16, 1000, 3, 3, 1.0, 3, "fp32"),
        # a medium study, plain FP64 (workload n20_ternary_m1000_d4)
        _solve("n20_ternary_m1000_d4_fp64", 20, 1000, 3, 4, 0.5, 4, "fp64"),
        # the largest served problem, alone, with an odd number of samples
        _solve("n22_ternary_m999_d3_fp32", 22, 999, 3, 3, 1.0, 3, "fp32"),
        # a large study in both forms (workload n25_binary_m2000_d4)
        _solve("n25_binary_m2000_d4_fp32", 25, 2000, 2, 4, 1.0, 4, "fp32"),
        _solve("n25_binary_m2000_d4_fp64", 25, 2000, 2, 4, 1.0, 4, "fp64"),
        # the largest lattice (workload n30_binary_m500_d3)
        _solve("n30_binary_m500_d3_fp32", 30, 500, 2, 3, 1.0, 3, "fp32"),
        # a burst of the serving stream: mixed sizes on one server
        dict(name="serve_48_mixed_d3_fp32", kind="serve", requests=48, d=3, precision="fp32"),
        # structure features beyond edges: whole parent-set tables to the host
        dict(name="parents_n18_binary_m700_d3_fp32", kind="parents", n=18, m=700, arity=2, maxdeg=3,
             a=1.0, d=3, precision="fp32"),
        # the score table alone, for a search that goes on with it elsewhere
        dict(name="scores_n20_ternary_m1000_d4", kind="scores", n=20, m=1000, arity=3, maxdeg=4,
             a=0.5, d=4),
        # the truncated zeta transform on its own
        dict(name="transform_up_2p27_d3", kind="transform", nbits=27, d=3, direction="zeta_up"),
    ]


def draw(rng):
    """One more case: sizes over the whole of each path's range."""
    kind = rng.choices(["solve", "serve", "parents", "scores", "transform"], [14, 1, 2, 2, 2])[0]
    if kind == "serve":
        return dict(kind=kind, requests=rng.randint(8, 48), d=rng.choice([2, 3]),
                    precision=rng.choice(["fp32", "fp32", "fp64"]))
    if kind == "transform":
        return dict(kind=kind, nbits=rng.randint(11, 28), d=rng.randint(1, 5),
                    direction=rng.choice(["zeta_up", "zeta_down"]))
    c = dict(kind=kind, m=int(round(100 * 20 ** rng.random())), arity=rng.choice([2, 2, 3]),
             maxdeg=rng.randint(2, 4), a=rng.choice([0.5, 1.0]), d=rng.choice([2, 3, 3, 4]))
    if kind == "scores":
        c["n"] = rng.randint(10, 26)
        return c
    c["precision"] = rng.choice(["fp32", "fp32", "fp64"])
    # the cost doubles with n, so uniform in n is uniform in its logarithm
    c["n"] = rng.randint(10, 20) if kind == "parents" else \
        rng.randint(10, 28 if c["precision"] == "fp32" else 27)
    return c


# ------------------------------------------------------------------ inputs

_held = {}


def _workspace(size):
    """One device workspace for all solves: they run one after another on one
    stream, so a program keeps one, as large as its largest problem."""
    if _held.get("ws") is None or _held["ws"].numel() < size:
        _held["ws"] = None
        _held["ws"] = torch.empty(size, dtype=torch.uint8, device="cuda")
    return _held["ws"]


def _server():
    """One server for all requests of a program."""
    if "server" not in _held:
        _held["server"] = bn.Server(mem_budget_bytes=8 << 30, max_active=16)
    return _held["server"]


def _dataset(case, seed):
    return datagen.random_dag_dataset(case["n"], case["m"], case["arity"], case["maxdeg"],
                                      case["a"], 1000 + seed)


def _requests(case, seed):
    """Requests of the serving stream's kind, spread over its range of sizes in
    a seeded order; the sizes themselves stay those of the case."""
    rng = np.random.default_rng(case["requests"])
    shapes = [(10 + 13 * int(j) // case["requests"], int(rng.integers(100, 2001)), int(rng.integers(2, 4)))
              for j in rng.permutation(case["requests"])]
    return [datagen.random_dag_dataset(n, m, r, 3, 1.0, 4_000_000 + 1000 * seed + j)
            for j, (n, m, r) in enumerate(shapes)]


def _values(case, seed):
    """What the transform is used on: non-negative terms over many decades.
    Drawn on the GPU (2^nbits values)."""
    g = torch.Generator(device="cuda").manual_seed(7000 + seed)
    u = torch.rand(1 << case["nbits"], dtype=torch.float64, device="cuda", generator=g)
    return torch.exp2(u.mul_(-200.0))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "transform":
        x = _values(case, seed)
        return dict(case=case, x=x, y=torch.empty_like(x))
    if kind == "serve":
        return dict(case=case, server=_server(), requests=_requests(case, seed))
    ds = _dataset(case, seed)
    state = dict(case=case, data=ds.data, arity=ds.arity)
    if kind == "solve":
        n, m, d = case["n"], case["m"], case["d"]
        state["data_dev"] = torch.from_numpy(ds.data).cuda()
        state["ws"] = _workspace(bn.workspace_bytes(n, d, m, case["precision"]))
        state["post"] = torch.zeros(n, n, dtype=torch.float64, device="cuda")
        state["diag"] = torch.zeros(8, dtype=torch.float64, device="cuda")
    return state


def _kept(post, precision):
    """The FP32-scaled form works on 24-bit significands; a program that asks
    for it keeps its posteriors in single precision."""
    if precision != "fp32":
        return post
    return post.float() if isinstance(post, torch.Tensor) else post.astype(np.float32)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        bn.edge_posteriors_dev(state["data_dev"], state["arity"], case["d"], case["precision"],
                               state["ws"], state["post"], state["diag"])
        return dict(post=_kept(state["post"], case["precision"]), log_PD=state["diag"][0])
    if kind == "serve":
        srv = state["server"]
        tickets = [srv.submit(ds.data, ds.arity, case["d"], precision=case["precision"])
                   for ds in state["requests"]]
        return [_kept(srv.poll(t, timeout_us=-1)[1], case["precision"]) for t in tickets]
    if kind == "parents":
        ps, post, rep = bn.parent_set_posteriors(state["data"], state["arity"], case["d"],
                                                 precision=case["precision"])
        return dict(ps=_kept(ps, case["precision"]), post=_kept(post, case["precision"]),
                    log_PD=rep["log_LV"])
    if kind == "scores":
        return bn.local_scores(state["data"], state["arity"], case["d"])
    # the program keeps its function beside the transform
    state["y"].copy_(state["x"])
    bn.subset_transform(state["y"], case["direction"],
                        case["d"] if case["direction"] == "zeta_up" else -1)
    return state["y"]


# -------------------------------------------------------------------- work

def _sets(n, d):
    return sum(comb(n - 1, k) for k in range(min(d, n - 1) + 1))


def _score_flops(n, m, d, arity):
    """One count per sample and set of up to d + 1 variables (each set's table
    serves every family inside it), and three operations per cell and family."""
    d = min(d, n - 1)
    counts = m * sum(comb(n, k) for k in range(1, d + 2))
    cells = n * sum(comb(n - 1, k) * min(m, arity ** (k + 1)) for k in range(d + 1))
    return counts + 3 * cells


def _lattice_flops(n, d):
    """Per node and set without it: d adds of the truncated upward transform, a
    product and an add in each sweep, two products into the downward transform
    and its d adds."""
    return n * 2 ** (n - 1) * (2 * min(d, n - 1) + 6)


def work(case):
    kind = case["kind"]
    if kind == "transform":
        size = 2 ** case["nbits"]
        per = case["d"] if case["direction"] == "zeta_up" else case["nbits"] / 2
        # the transform in place (16 bytes an entry), and the copy that feeds it
        return {"bytes": 32 * size, "flops": size * min(per, case["nbits"] / 2)}
    if kind == "serve":
        got = {"bytes": 0, "flops": 0}
        for ds in _requests(case, 0):
            r = int(ds.arity[0])
            got["bytes"] += ds.n * ds.m + 8 * ds.n * ds.n
            got["flops"] += _score_flops(ds.n, ds.m, case["d"], r) + _lattice_flops(ds.n, case["d"])
        return got
    n, m, d, r = case["n"], case["m"], case["d"], case["arity"]
    if kind == "scores":
        return {"bytes": n * m + 8 * n * _sets(n, d), "flops": _score_flops(n, m, d, r)}
    tables = 8 * n * _sets(n, d) if kind == "parents" else 0
    return {"bytes": n * m + 8 * n * n + tables,
            "flops": _score_flops(n, m, d, r) + _lattice_flops(n, d)}


# ------------------------------------------- the same in plain 64-bit torch

_NEG = float("-inf")


def _exact_scores(data, arity, d, dev):
    """log p(x_i | x_G) (BDeu, sample size 1) as [n, K], sets by size, then by mask."""
    n, m = data.shape
    d = min(d, n - 1)
    K = _sets(n, d)
    out = torch.empty(n, K, dtype=torch.float64, device=dev)
    r = int(arity[0])
    x = torch.from_numpy(np.ascontiguousarray(data)).to(dev).long()
    off = 0
    rank = {}
    for k in range(d + 1):
        order = sorted(combinations(range(n - 1), k), key=lambda c: sum(1 << p for p in c))
        rank.update({c: off + j for j, c in enumerate(order)})
        off += len(order)
    for k in range(d + 1):
        unions = list(combinations(range(n), k + 1))
        bins = r ** (k + 1)
        step = max(1, (1 << 26) // max(m, bins))
        for s in range(0, len(unions), step):
            part = unions[s:s + step]
            u = torch.tensor(part, device=dev)                      # [F, k+1]
            code = torch.zeros(len(part), m, dtype=torch.long, device=dev)
            for j in range(k + 1):
                code = code * r + x[u[:, j]]
            code += torch.arange(len(part), device=dev)[:, None] * bins
            cnt = torch.bincount(code.reshape(-1), minlength=len(part) * bins)
            cnt = cnt.double().reshape([len(part)] + [r] * (k + 1))
            a_jk = 1.0 / bins
            a_j = a_jk * r
            a_jk = torch.tensor(a_jk, dtype=torch.float64, device=dev)
            a_j = torch.tensor(a_j, dtype=torch.float64, device=dev)
            cell = (torch.lgamma(cnt + a_jk) - torch.lgamma(a_jk)).reshape(len(part), -1).sum(1)
            for j in range(k + 1):
                row = cnt.sum(1 + j)
                score = cell + (torch.lgamma(a_j) - torch.lgamma(row + a_j)).reshape(
                    len(part), -1).sum(1)
                at = [rank[tuple(p if p < c[j] else p - 1 for p in c if p != c[j])] for c in part]
                out[u[:, j], torch.tensor(at, device=dev)] = score
    return out


def _drop(s, i):
    """The mask without bit i, closed up."""
    return (s & ((1 << i) - 1)) | ((s >> (i + 1)) << i)


def _zeta(a, bits, up):
    """In-place log-space sums over subsets (up) or supersets of each index."""
    for b in range(bits):
        v = a.view(-1, 2, 1 << b)
        lo, hi = v[:, 0], v[:, 1]
        if up:
            hi.copy_(torch.logaddexp(hi, lo))
        else:
            lo.copy_(torch.logaddexp(lo, hi))


def _exact_solve(data, arity, d, dev):
    """(parent-set posteriors [n, K], edge posteriors [n, n], log P(D)), all in FP64 logs."""
    n, m = data.shape
    d = min(d, n - 1)
    K = _sets(n, d)
    masks = []
    for k in range(d + 1):
        masks += sorted(sum(1 << p for p in c) for c in combinations(range(n - 1), k))
    sizes = torch.tensor([bin(x).count("1") for x in masks], device=dev)
    masks = torch.tensor(masks, device=dev)
    rho = -torch.tensor([comb(n - 1, k) for k in range(d + 1)], dtype=torch.float64, device=dev).log()
    beta = _exact_scores(data, arity, d, dev) + rho[sizes]
    alpha = torch.full((n, 1 << (n - 1)), _NEG, dtype=torch.float64, device=dev)
    for i in range(n):
        alpha[i, masks] = beta[i]
        _zeta(alpha[i], n - 1, True)
    s = torch.arange(1 << n, device=dev)
    pop = torch.zeros(1 << n, dtype=torch.int8, device=dev)
    for i in range(n):
        pop += (s >> i & 1).to(torch.int8)
    del s
    order = torch.sort(pop, stable=True).indices
    del pop
    layers = torch.split(order, [comb(n, k) for k in range(n + 1)])
    L = torch.full((1 << n,), _NEG, dtype=torch.float64, device=dev)
    R = L.clone()
    L[0] = 0.0
    R[-1] = 0.0

    def sweep(X, these, forward):
        acc = torch.full((these.numel(),), _NEG, dtype=torch.float64, device=dev)
        for i in range(n):
            inside = (these >> i & 1).bool()
            term = alpha[i][_drop(these, i)] + X[these ^ (1 << i)]
            acc = torch.logaddexp(acc, torch.where(inside == forward, term, _NEG))
        X[these] = acc

    for k in range(1, n + 1):
        sweep(L, layers[k], True)
        sweep(R, layers[n - k], False)
    del alpha, order, layers
    log_pd = L[-1]
    ps = torch.empty(n, K, dtype=torch.float64, device=dev)
    post = torch.zeros(n, n, dtype=torch.float64, device=dev)
    for v in range(n):
        lv = L.view(-1, 2, 1 << v)[:, 0].reshape(-1)
        g = lv + R.view(-1, 2, 1 << v)[:, 1].reshape(-1)
        _zeta(g, n - 1, False)
        ps[v] = torch.exp(beta[v] + g[masks] - log_pd)
        for u in range(n):
            if u != v:
                p = u if u < v else u - 1
                post[u, v] = ps[v][(masks >> p & 1).bool()].sum()
    return ps, post, log_pd


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "transform":
        if case["nbits"] > 27:
            return None
        y = _values(case, seed).to(dev)
        nbits = case["nbits"]
        if case["direction"] == "zeta_up":
            s = torch.arange(1 << nbits, device=dev, dtype=torch.int32)
            pop = sum((s >> b & 1).to(torch.int8) for b in range(nbits))
            y[pop > case["d"]] = 0.0
        for b in range(nbits):
            v = y.view(-1, 2, 1 << b)
            if case["direction"] == "zeta_up":
                v[:, 1] += v[:, 0]
            else:
                v[:, 0] += v[:, 1]
        return y
    if kind == "serve":
        return [_exact_solve(ds.data, ds.arity, case["d"], dev)[1] for ds in _requests(case, seed)]
    if case["n"] > 25:
        return None  # minutes of log-space sums
    ds = _dataset(case, seed)
    if kind == "scores":
        return _exact_scores(ds.data, ds.arity, case["d"], dev)
    ps, post, log_pd = _exact_solve(ds.data, ds.arity, case["d"], dev)
    if kind == "parents":
        return dict(ps=ps, post=post, log_PD=float(log_pd))
    return dict(post=post, log_PD=log_pd)
