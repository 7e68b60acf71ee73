"""The work that a user of this package has it do, as cases that can be timed and checked.

A case is a dict of plain values: ``kind`` names the entry point, ``graph`` the
graph recipe, the rest sizes and parameters.  ``prepare(case, seed)`` makes
what a program holds before the call (the graph on the GPU, the inputs),
``run(state)`` is one pass through the public entry point.

Kinds
  solve     mqo.solve: the batched search of Alg. 1 - 4 (integers come back)
  grad      mqo.objective and its backward: objective values and gradient
  unrolled  mqo.unrolled_pga and its backward
  pair      mqo.pair_search: OneTwoSwap (MIS) / OneTwoFlip (MaxCut)

Graphs, edges drawn from the seed, sizes fixed by the case
  er        G(n, p), p given or mean degree / (n - 1)
  er_batch  `count` graphs G(n_g, p), n_g evenly spread over [n_lo, n_hi]
  regular   random d-regular
  ba        preferential attachment, m edges per new vertex
  torus     side x side, weights +-1
"""
import types

import numpy as np
import torch

from paper_2605_06921_amd import mqo

DEV = "cuda"


# --------------------------------------------------------------------------
# graphs in the canonical CSR form
# --------------------------------------------------------------------------

def _csr(n, u, v, w=None, vtx_offset=None):
    """Canonical CSR of the undirected edges (u, v), torch int64 on the GPU: duplicates and loops dropped."""
    a, b = torch.minimum(u, v), torch.maximum(u, v)
    key = a * n + b
    if w is None:
        key = torch.unique(key[a != b])
    a, b = key // n, key % n
    rows, cols = torch.cat([a, b]), torch.cat([b, a])
    order = torch.argsort(rows * n + cols)
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=rows.device)
    row_ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return types.SimpleNamespace(
        n=n, row_ptr=row_ptr.to(torch.int32).cpu().numpy(), col_idx=cols[order].to(torch.int32).cpu().numpy(),
        weight=None if w is None else torch.cat([w, w])[order].to(torch.int32).cpu().numpy(),
        vtx_offset=np.array([0, n], dtype=np.int64) if vtx_offset is None else vtx_offset)


def _er_edges(n, p, gen):
    """Edges of G(n, p): all pairs for small n, else the binomial number of distinct random pairs."""
    if n <= 4096:
        hit = torch.rand(n, n, generator=gen, device=DEV) < p
        e = torch.triu(hit, 1).nonzero()
        return e[:, 0], e[:, 1]
    pairs = n * (n - 1) // 2
    m = int(pairs * p)
    u = torch.randint(n, (m + m // 50,), generator=gen, device=DEV)
    v = torch.randint(n, (m + m // 50,), generator=gen, device=DEV)
    a, b = torch.minimum(u, v), torch.maximum(u, v)
    key = torch.unique((a * n + b)[a != b])
    key = key[torch.randperm(key.numel(), generator=gen, device=DEV)[:m]]
    return key // n, key % n


def _regular(n, d, rng):
    """Pairing model; pairs that are loops or repeats are re-paired with random others."""
    stubs = rng.permutation(np.repeat(np.arange(n, dtype=np.int64), d))
    a, b = stubs[0::2].copy(), stubs[1::2].copy()
    while True:
        key = np.minimum(a, b) * n + np.maximum(a, b)
        order = np.argsort(key, kind="stable")
        bad = a == b
        bad[order[1:]] |= key[order[1:]] == key[order[:-1]]
        if not bad.any():
            return a, b
        at = np.concatenate([np.flatnonzero(bad), rng.choice(np.flatnonzero(~bad), size=max(4, int(bad.sum())))])
        at = np.unique(at)
        pool = rng.permutation(np.concatenate([a[at], b[at]]))
        a[at], b[at] = pool[0::2], pool[1::2]


def _ba(n, m, rng):
    """Preferential attachment: edge e leaves vertex e // m; its other end copies a random earlier edge end."""
    e = np.arange(n * m, dtype=np.int64)
    src = e // m
    slot = (rng.random(n * m) * np.maximum(2 * m * src, 1)).astype(np.int64)
    while (slot & 1).any():  # an odd slot is the copied end of an earlier edge: follow it
        slot = np.where(slot & 1, slot[slot >> 1], slot)
        slot[:m] = 0
    return src, (slot >> 1) // m


def make_graph(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)  # noqa: E731
    if case["graph"] == "er":
        n = case["n"]
        return _csr(n, *_er_edges(n, case["p"] if "p" in case else case["degree"] / (n - 1), gen))
    if case["graph"] == "er_batch":
        sizes = np.linspace(case["n_lo"], case["n_hi"], case["count"]).astype(np.int64)
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        us, vs = zip(*[_er_edges(int(s), case["p"], gen) for s in sizes])
        return _csr(int(off[-1]), torch.cat([x + int(o) for x, o in zip(us, off)]),
                    torch.cat([x + int(o) for x, o in zip(vs, off)]), None, off)
    if case["graph"] == "regular":
        return _csr(case["n"], *map(t, _regular(case["n"], case["degree"], rng)))
    if case["graph"] == "ba":
        return _csr(case["n"], *map(t, _ba(case["n"], case["m"], rng)))
    side = case["side"]
    n = side * side
    v = torch.arange(n, device=DEV)
    right, down = v // side * side + (v + 1) % side, (v + side) % n
    w = torch.randint(0, 2, (2 * n,), generator=gen, device=DEV) * 2 - 1
    return _csr(n, torch.cat([v, v]), torch.cat([right, down]), w)


def sizes(case):
    """(rows, stored entries, graphs), the entries by expectation."""
    if case["graph"] == "er":
        n = case["n"]
        return n, n * (case["p"] * (n - 1) if "p" in case else case["degree"]), 1
    if case["graph"] == "er_batch":
        s = np.linspace(case["n_lo"], case["n_hi"], case["count"]).astype(np.int64)
        return int(s.sum()), float((s * (s - 1)).sum() * case["p"]), case["count"]
    if case["graph"] == "regular":
        return case["n"], case["n"] * case["degree"], 1
    if case["graph"] == "ba":
        return case["n"], 2 * case["n"] * case["m"], 1
    return case["side"] ** 2, 4 * case["side"] ** 2, 1


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------

# the paper's own settings for its ER tables: degree-based start, momentum, steps until a
# fixed point (tested every 10), the pair search at the end
PAPER_MIS = dict(problem="mis", steps=200, alpha=0.8, momentum=0.3, rho=0.6, check_every=10, init_mode="degree",
                 init_sigma=0.1, final_search=True)
PAPER_CUT = dict(problem="maxcut", steps=200, alpha=0.0025, momentum=0.8, rho=0.8, check_every=10,
                 init_mode="degree", init_sigma=0.1, final_search=True)


def listed():
    return [
        # one small graph, one trajectory, 1000 steps and one rounding: latency of a single answer
        dict(name="solve_er100_b1", kind="solve", graph="er", n=100, p=0.1, problem="mis", batch=1, steps=1000,
             rounds=1, alpha=0.01, rho=0.05),
        # a sparse regular graph with many restarts, flip resets
        dict(name="solve_reg3_n2000_b256", kind="solve", graph="regular", n=2000, degree=3, problem="maxcut",
             batch=256, steps=200, rounds=10, alpha=0.01, rho=0.05, reset_mode="flip"),
        # throughput: a batch of 128 dense-ish graphs, 512 restarts each
        dict(name="solve_er_batch_b512", kind="solve", graph="er_batch", count=128, n_lo=700, n_hi=800, p=0.15,
             problem="mis", batch=512, steps=200, rounds=4, alpha=0.01, rho=0.05),
        # graphs of a million vertices, irregular and local
        dict(name="solve_er1m_b32", kind="solve", graph="er", n=1_000_000, degree=10, problem="mis", batch=32,
             steps=200, rounds=4, alpha=0.01, rho=0.05),
        dict(name="solve_torus1m_b32", kind="solve", graph="torus", side=1000, problem="maxcut", batch=32,
             steps=200, rounds=8, alpha=0.01, rho=0.05),
        # the paper's ER (3000, 100) and a MaxCut graph of degree 100, its hyper-parameters, 64 chains
        dict(PAPER_MIS, name="paper_er3000_b64", kind="solve", graph="er", n=3000, degree=100, batch=64, rounds=61),
        dict(PAPER_CUT, name="paper_cut1000_b64", kind="solve", graph="er", n=1000, degree=100, batch=64, rounds=91),
        # differentiating through the objective: a hub-rich graph, and a minibatch of small graphs
        dict(name="grad_ba100k_b64", kind="grad", graph="ba", n=100_000, m=4, problem="mis", batch=64),
        dict(name="grad_minibatch_b32", kind="grad", graph="er_batch", count=64, n_lo=100, n_hi=200, p=0.1,
             problem="maxcut", batch=32),
        # learning through 20 unrolled steps, forward and backward
        dict(name="unrolled_reg5_100k_b64", kind="unrolled", graph="regular", n=100_000, degree=5, problem="maxcut",
             batch=64, steps=20, every=5),
        # the paper's searches on their own, from 1-flip optima
        dict(name="swap_er_batch_b512", kind="pair", graph="er_batch", count=128, n_lo=700, n_hi=800, p=0.15,
             problem="mis", batch=512),
        dict(name="flip_torus1m_b32", kind="pair", graph="torus", side=1000, problem="maxcut", batch=32),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["single", "regular", "er_batch", "sparse", "torus", "paper_mis", "paper_cut", "grad", "minibatch",
                       "unrolled", "swap", "flip"])
    if kind == "single":
        return dict(kind="solve", graph="er", n=_log(rng, 50, 400), p=round(rng.uniform(0.04, 0.25), 3), problem="mis",
                    batch=rng.choice([1, 2, 3, 4, 8]), steps=_log(rng, 100, 1000), rounds=rng.choice([1, 2]),
                    alpha=0.01, rho=0.05)
    if kind == "regular":
        return dict(kind="solve", graph="regular", n=2 * _log(rng, 100, 1500), degree=rng.choice([3, 4, 5, 7]),
                    problem=rng.choice(["maxcut", "mis"]), batch=_log(rng, 16, 300), steps=_log(rng, 50, 250),
                    rounds=rng.randint(2, 10), alpha=0.01, rho=0.05, reset_mode=rng.choice(["flip", "zero"]))
    if kind == "er_batch":
        n = _log(rng, 150, 800)
        return dict(kind="solve", graph="er_batch", count=rng.randint(8, 100), n_lo=int(0.85 * n), n_hi=n,
                    p=round(rng.uniform(0.05, 0.2), 3), problem=rng.choice(["mis", "mis", "maxcut"]),
                    batch=_log(rng, 32, 400), steps=rng.choice([100, 150, 200]), rounds=rng.randint(1, 4),
                    alpha=0.01, rho=0.05)
    if kind == "sparse":
        return dict(kind="solve", graph="er", n=_log(rng, 50_000, 1_000_000), degree=rng.choice([6, 8, 10]),
                    problem="mis", batch=rng.choice([8, 13, 16, 24, 32]), steps=_log(rng, 50, 200),
                    rounds=rng.randint(1, 4), alpha=0.01, rho=0.05)
    if kind == "torus":
        return dict(kind="solve", graph="torus", side=_log(rng, 250, 1000), problem="maxcut",
                    batch=rng.choice([8, 12, 16, 30, 32]), steps=_log(rng, 50, 200), rounds=rng.randint(1, 8),
                    alpha=0.01, rho=0.05)
    if kind == "paper_mis":
        return dict(PAPER_MIS, kind="solve", graph="er", n=_log(rng, 800, 3000), degree=rng.choice([40, 70, 100]),
                    batch=rng.choice([16, 33, 64]), rounds=rng.randint(10, 50))
    if kind == "paper_cut":
        return dict(PAPER_CUT, kind="solve", graph="er", n=_log(rng, 400, 1000), degree=rng.choice([40, 70, 100]),
                    batch=rng.choice([16, 33, 64]), rounds=rng.randint(10, 80))
    if kind == "grad":
        return dict(kind="grad", graph=rng.choice(["ba", "ba", "er"]), n=_log(rng, 10_000, 100_000), m=4, degree=8,
                    problem=rng.choice(["mis", "maxcut"]), batch=rng.choice([16, 30, 32, 64]))
    if kind == "minibatch":
        n = _log(rng, 60, 400)
        return dict(kind="grad", graph="er_batch", count=rng.randint(8, 100), n_lo=n // 2, n_hi=n,
                    p=round(rng.uniform(0.05, 0.15), 3), problem=rng.choice(["mis", "maxcut"]),
                    batch=rng.choice([7, 16, 32, 64]))
    if kind == "unrolled":
        return dict(kind="unrolled", graph=rng.choice(["regular", "ba"]), n=2 * _log(rng, 5_000, 50_000), degree=5, m=4,
                    problem=rng.choice(["mis", "maxcut"]), batch=rng.choice([16, 30, 32, 64]),
                    **rng.choice([dict(steps=20, every=5), dict(steps=12, every=4), dict(steps=10, every=1)]))
    if kind == "swap":
        n = _log(rng, 200, 800)
        return dict(kind="pair", graph="er_batch", count=rng.randint(8, 100), n_lo=int(0.85 * n), n_hi=n,
                    p=round(rng.uniform(0.05, 0.2), 3), problem="mis", batch=_log(rng, 32, 400))
    return dict(kind="pair", graph="torus", side=_log(rng, 250, 1000), problem="maxcut",
                batch=rng.choice([8, 12, 16, 30, 32]))


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

GAMMA, LAM, ALPHA = 2.0, 1e-3, 0.01


def _inputs(case, seed, n, G):
    """The iterate of the differentiation calls (uniform in the problem's box) and upstream gradients."""
    gen = torch.Generator(device=DEV).manual_seed(seed + 10**6)
    X = torch.rand(n, case["batch"], generator=gen, device=DEV)
    if case["problem"] == "maxcut":
        X = 2 * X - 1
    up = torch.randn(*((G * case["batch"],) if case["kind"] == "grad" else (n, case["batch"])), generator=gen, device=DEV)
    return X, up.double() if case["kind"] == "grad" else up


def prepare(case, seed):
    graph = make_graph(case, seed)
    dg = mqo.DeviceGraph(graph, DEV)
    s = types.SimpleNamespace(case=case, dg=dg, seed=seed)
    if case["kind"] == "solve":
        keys = ("batch", "rounds", "alpha", "momentum", "rho", "reset_mode", "check_every", "init_mode", "init_sigma",
                "final_search")
        s.params = dict({k: case[k] for k in keys if k in case}, steps_per_round=case["steps"], seed=seed + 10**6)
        s.workspace = mqo.Workspace(DEV)
    elif case["kind"] == "pair":
        X = mqo.init_iterate(case["problem"], dg, case["batch"], seed + 10**6)
        s.Z = mqo.round_evaluate(case["problem"], dg, X)[0]
        mqo.local_search(case["problem"], dg, s.Z, seed + 10**6, 0)
    else:
        s.param = GAMMA if case["problem"] == "mis" else LAM
        s.X, s.up = _inputs(case, seed, dg.n, dg.num_graphs)
        s.alpha = torch.tensor(ALPHA, device=DEV)
    return s


def run(s):
    case = s.case
    if case["kind"] == "solve":
        out = mqo.solve(case["problem"], s.dg, workspace=s.workspace, **s.params)
        return {k: out[k] for k in ("best_value", "best_x", "traj_best_value", "traj_best_x")}
    if case["kind"] == "pair":
        Z = s.Z.clone()
        moves = mqo.pair_search(case["problem"], s.dg, Z, s.seed + 10**6, 1)
        return {"Z": Z, "iterations": moves}
    X = s.X.detach().requires_grad_(True)
    if case["kind"] == "grad":
        f = mqo.objective(X, s.dg, case["problem"], s.param)
        f.backward(s.up)
        return {"f": f.detach(), "grad": X.grad}
    alpha = s.alpha.detach().requires_grad_(True)
    XK = mqo.unrolled_pga(X, alpha, s.dg, case["problem"], s.param, case["steps"], case["every"])
    XK.backward(s.up)
    return {"XK": XK.detach(), "grad_X0": X.grad, "grad_alpha": alpha.grad}


def work(case):
    n, nnz, G = sizes(case)
    B = case["batch"]
    graph = 4 * (n + 1) + 4 * nnz * (2 if case["graph"] == "torus" else 1)
    if case["kind"] == "solve":
        # every step adds each stored entry once per trajectory; where steps may end early, the first chunk of a round
        steps = case["rounds"] * case.get("check_every", case["steps"])
        return {"bytes": graph + n * B + n + 8 * G * (B + 1), "flops": (2 * nnz + 4 * n) * B * steps}
    if case["kind"] == "pair":
        return {"bytes": graph + 2 * n * B, "flops": 2 * nnz * B}
    if case["kind"] == "grad":
        return {"bytes": graph + 8 * n * B + 16 * G * B, "flops": (2 * nnz + 6 * n) * B}
    # forward, and the adjoint's product with the Hessian in every step
    return {"bytes": graph + 16 * n * B, "flops": (2 * nnz + 6 * n) * B * 2 * case["steps"]}


# --------------------------------------------------------------------------
# in 64 bits
# --------------------------------------------------------------------------

def exact(case, seed):
    if case["kind"] not in ("grad", "unrolled"):
        return None  # integers
    graph = make_graph(case, seed)
    n, B, G = graph.n, case["batch"], len(graph.vtx_offset) - 1
    X, up = _inputs(case, seed, n, G)
    X, up = X.double(), up.double()
    rows = torch.from_numpy(np.repeat(np.arange(n), np.diff(graph.row_ptr))).to(DEV)
    cols = torch.from_numpy(graph.col_idx.astype(np.int64)).to(DEV)
    w = None if graph.weight is None else torch.from_numpy(graph.weight).to(DEV).double()[:, None]

    def mul(Y):
        return torch.zeros_like(Y).index_add_(0, rows, Y[cols] if w is None else w * Y[cols])

    mis = case["problem"] == "mis"
    param = float(np.float32(GAMMA if mis else LAM))
    slope = -param if mis else -2.0  # the gradient is const + slope * A x

    def gradient(Y):
        return 1.0 + slope * mul(Y) if mis else -param + slope * mul(Y)

    of_row = torch.from_numpy(np.repeat(np.arange(G), np.diff(graph.vtx_offset))).to(DEV)
    if case["kind"] == "grad":
        fv = X * ((1.0 if mis else -param) + 0.5 * slope * mul(X))
        f = torch.zeros(G, B, dtype=torch.float64, device=DEV).index_add_(0, of_row, fv)
        return {"f": f.reshape(-1), "grad": up.float().double().view(G, B)[of_row] * gradient(X)}
    alpha = float(np.float32(ALPHA))
    lo = 0.0 if mis else -1.0
    xs = [X]
    for _ in range(case["steps"]):
        xs.append((xs[-1] + alpha * gradient(xs[-1])).clamp(lo, 1.0))
    lam, da = up, 0.0
    for x in reversed(xs[:-1]):
        g = gradient(x)
        z = x + alpha * g
        mu = torch.where((z >= lo) & (z <= 1.0), lam, torch.zeros_like(lam))
        da = da + (mu * g).sum()
        lam = mu + alpha * slope * mul(mu)
    return {"XK": xs[-1], "grad_X0": lam, "grad_alpha": da}
