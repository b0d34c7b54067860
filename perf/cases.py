"""The calls a program makes of this framework, as a list of cases that can be timed.

A case is a dict of plain values.  ``prepare`` makes what a program holds before the
call (inputs on the GPU, made from the seed, and the solver handle it keeps), ``run``
is one pass through the public entry points with everything it returns, ``work`` the
bytes and operations of one pass that no implementation can do without, and ``exact``
the same outputs in 64 bits by plain torch and numpy.
"""
import math
import types

import numpy as np
import torch

import paper_2004_08227_amd as M
from paper_2004_08227_amd.autograd import mplp_dual

DTYPES = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # a handful of variables solved exactly as possible, the dual watched every
        # iteration: the smallest call, all launches and latency
        dict(name="tiny_f64_n8_l4", kind="trace", dtype="f64", costs="uniform", n=8, L=4, density=1.0, iters=50),
        # a small fully connected model kept in a handle (the lower end of the pose mix)
        dict(name="small_f32_n20_l8", kind="solve", dtype="f32", costs="pose", n=20, L=8, density=1.0, iters=50),
        # a model that arrives as device tensors, is solved once and dropped: odd sizes,
        # with the creation of the handle in the pass
        dict(name="oneshot_f32_n61_l21", kind="oneshot", dtype="f32", costs="pose", n=61, L=21, density=1.0, iters=50),
        # a serving loop that may not allocate device memory: one model a call
        dict(name="serve_f32_n40_l24", kind="serve", dtype="f32", costs="uniform", n=40, L=24, density=1.0, iters=50),
        # the pose workload (Sec. 7 of the paper): iterate, bound, labelling, state
        dict(name="pose_f32_n200_l64", kind="solve", dtype="f32", costs="pose", n=200, L=64, density=1.0, iters=100),
        # the sparsification study: a large sparse graph, few labels
        dict(name="sparse_f32_n1000_l16", kind="solve", dtype="f32", costs="potts", n=1000, L=16, density=0.05, iters=50),
        # many labels, a ragged count above one wavefront
        dict(name="labels_f32_n40_l100", kind="solve", dtype="f32", costs="uniform", n=40, L=100, density=1.0, iters=50),
        # the FP64 solver at the size of the differentiation workload
        dict(name="double_f64_n100_l32", kind="solve", dtype="f64", costs="uniform", n=100, L=32, density=1.0, iters=50),
        # anytime use: bound and labelling after every iteration, the best labelling kept
        dict(name="gap_f32_n100_l32", kind="gap", dtype="f32", costs="pose", n=100, L=32, density=1.0, iters=20),
        # a learning step: the dual after K iterations and its gradient
        dict(name="train_f32_n100_l32", kind="train", dtype="f32", costs="uniform", n=100, L=32, density=1.0, iters=50, every=10),
        # many models of mixed sizes in one launch
        dict(name="batch_f32_24", kind="batch", dtype="f32", costs="pose", count=24, n=20, n_max=160, L=8, L_max=64, iters=50),
        # structured costs given by two parameters an edge
        dict(name="linear_f32_n200_l64", kind="structured", dtype="f32", costs="linear", n=200, L=64, density=1.0, iters=50),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def draw(rng):
    kind = rng.choice(["trace", "solve", "solve", "solve64", "oneshot", "serve", "sparse", "labels", "gap", "train", "batch",
                       "structured"])
    if kind == "trace":
        return dict(kind="trace", dtype="f64", costs="uniform", n=_log(rng, 4, 32), L=_log(rng, 2, 16), density=1.0,
                    iters=rng.randint(10, 60))
    if kind == "solve":
        return dict(kind="solve", dtype="f32", costs=rng.choice(["pose", "uniform"]), n=_log(rng, 12, 200), L=_log(rng, 4, 64),
                    density=1.0, iters=rng.randint(20, 100))
    if kind == "solve64":
        return dict(kind="solve", dtype="f64", costs=rng.choice(["pose", "uniform"]), n=_log(rng, 8, 120), L=_log(rng, 3, 48),
                    density=1.0, iters=rng.randint(10, 60))
    if kind == "oneshot":
        return dict(kind="oneshot", dtype="f32", costs="pose", n=_log(rng, 12, 120), L=_log(rng, 4, 48), density=1.0,
                    iters=rng.randint(10, 60))
    if kind == "serve":
        return dict(kind="serve", dtype="f32", costs="uniform", n=_log(rng, 8, 80), L=_log(rng, 4, 40), density=1.0,
                    iters=rng.randint(10, 60))
    if kind == "sparse":
        return dict(kind="solve", dtype="f32", costs="potts", n=_log(rng, 100, 1000), L=_log(rng, 4, 24),
                    density=round(rng.uniform(0.02, 0.12), 3), iters=rng.randint(20, 60))
    if kind == "labels":
        return dict(kind="solve", dtype="f32", costs="uniform", n=_log(rng, 8, 60), L=rng.randint(65, 128), density=1.0,
                    iters=rng.randint(20, 60))
    if kind == "gap":
        return dict(kind="gap", dtype="f32", costs="pose", n=_log(rng, 12, 150), L=_log(rng, 4, 64), density=1.0,
                    iters=rng.randint(5, 25))
    if kind == "train":
        return dict(kind="train", dtype="f32", costs="uniform", n=_log(rng, 12, 100), L=_log(rng, 4, 40), density=1.0,
                    iters=rng.randint(10, 50), every=rng.choice([5, 10]))
    if kind == "batch":
        return dict(kind="batch", dtype="f32", costs="pose", count=rng.randint(4, 24), n=rng.randint(8, 24),
                    n_max=rng.randint(60, 150), L=rng.randint(4, 12), L_max=rng.randint(24, 64), iters=rng.randint(10, 50))
    return dict(kind="structured", dtype="f32", costs=rng.choice(["linear", "quad", "weights"]), n=_log(rng, 20, 200),
                L=_log(rng, 6, 64), density=round(rng.choice([1.0, rng.uniform(0.2, 0.9)]), 3), iters=rng.randint(20, 50))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _count(case):
    full = case["n"] * (case["n"] - 1) // 2
    return full if case["density"] >= 1.0 else max(1, int(round(full * case["density"])))


def _edges(case, seed):
    u, v = np.triu_indices(case["n"], 1)
    if case["density"] < 1.0:
        # a random graph with a given number of edges, so that every seed's outputs have one shape
        keep = np.sort(np.random.default_rng(seed).permutation(u.size)[: _count(case)])
        u, v = u[keep], v[keep]
    return np.ascontiguousarray(np.stack([u, v], 1).astype(np.int32))


def _dense(n, L, edges, costs, dtype, seed):
    """(unaries [n, L], pairwise [m, L, L]) on the GPU with the distributions of the
    framework's own workloads, drawn on the device."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    rand = lambda *s: torch.rand(*s, generator=g, device="cuda", dtype=torch.float64)  # noqa: E731
    u, v = (torch.from_numpy(edges[:, k].astype(np.int64)).cuda() for k in (0, 1))
    un = rand(n, L)
    if costs == "pose":
        # labels are points of the unit cube, one of each node planted
        p = rand(n, L, 3)
        q = p[torch.arange(n, device="cuda"), torch.randint(0, L, (n,), generator=g, device="cuda")]
        dq = (q[u] - q[v]).square().sum(1).sqrt()[:, None, None]
        pw = torch.empty((len(edges), L, L), dtype=dtype, device="cuda")
        for lo in range(0, len(edges), 4096):
            s = slice(lo, lo + 4096)
            d = (p[u[s]][:, :, None, :] - p[v[s]][:, None, :, :]).square().sum(3).sqrt() - dq[s]
            pw[s] = (d * d).clamp(max=0.04).to(dtype)
    elif costs == "potts":
        w = 0.1 + 0.9 * rand(len(edges))
        pw = (w[:, None, None] * (1.0 - torch.eye(L, device="cuda", dtype=torch.float64)) + 0.2 * rand(len(edges), L, L)).to(dtype)
    else:
        pw = rand(len(edges), L, L).to(dtype)
    return un.to(dtype).contiguous(), pw.contiguous()


def _structured(case, seed):
    """(unaries [n, L], parameters per edge) as host arrays, float32."""
    r = np.random.default_rng(seed)
    edges = _edges(case, seed)
    un = r.random((case["n"], case["L"])).astype(np.float32)
    m = len(edges)
    if case["costs"] == "weights":
        return edges, un, r.uniform(0.1, 1.0, (m, 1)).astype(np.float32), M.COST_POTTS
    tau = 8.0 if case["costs"] == "linear" else 64.0
    w = r.uniform(0.05, 0.5, m) if case["costs"] == "linear" else r.uniform(0.005, 0.05, m)
    kind = M.COST_TRUNC_LINEAR if case["costs"] == "linear" else M.COST_TRUNC_QUAD
    return edges, un, np.stack([w, np.full(m, tau)], 1).astype(np.float32), kind


def _sizes(case, seed):
    """The sizes of a batch's models: the largest and smallest, and a spread that does
    not depend on the seed (the work of a case is one number)."""
    r = np.random.default_rng(12345 + case["count"])
    ns = r.integers(case["n"], case["n_max"] + 1, case["count"])
    Ls = r.integers(case["L"], case["L_max"] + 1, case["count"])
    ns[0], Ls[0], ns[-1], Ls[-1] = case["n_max"], case["L_max"], case["n"], case["L"]
    return [(int(a), int(b)) for a, b in zip(ns, Ls)]


def _batch_models(case, seed):
    got = []
    for i, (n, L) in enumerate(_sizes(case, seed)):
        e = _edges(dict(n=n, density=1.0), seed)
        un, pw = _dense(n, L, e, case["costs"], torch.float32, seed * 1009 + i)
        got.append(types.SimpleNamespace(n=n, L=L, m=len(e), edges=e, unaries=un.cpu().numpy(), pairwise=pw.cpu().numpy()))
    return got


def prepare(case, seed):
    s = types.SimpleNamespace(case=case)
    kind = case["kind"]
    if kind == "batch":
        s.handle = M.Batch(_batch_models(case, seed))
        s.handle.models = None  # a program that keeps the handle need not keep the host tables
        return s
    if kind == "structured":
        s.edges, un, prm, cost = _structured(case, seed)
        model = types.SimpleNamespace(n=case["n"], L=case["L"], m=len(s.edges), edges=s.edges, unaries=un, pairwise=prm)
        s.handle = M.Solver.from_structured(model, cost)
        return s
    n, L = case["n"], case["L"]
    s.edges = _edges(case, seed)
    s.unaries, s.pairwise = _dense(n, L, s.edges, case["costs"], DTYPES[case["dtype"]], seed)
    if kind in ("solve", "trace", "gap"):
        torch.cuda.synchronize()
        s.handle = M.Solver.from_torch(n, L, s.edges, s.unaries, s.pairwise)
        s.unaries = s.pairwise = None  # copied into the handle
    elif kind == "serve":
        s.U = torch.empty((n, L), dtype=torch.float32, device="cuda")
        s.phi = torch.empty((len(s.edges), 2, L), dtype=torch.float32, device="cuda")
    elif kind == "train":
        s.unaries.requires_grad_(True)
        s.pairwise.requires_grad_(True)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    case = s.case
    kind, k = case["kind"], case["iters"]
    if kind == "batch":
        # (a second pass goes on from the state the first one reached, as a program
        # that checks its duals every k iterations does; likewise below)
        s.handle.iterate(k)
        return {"dual": s.handle.dual_bounds(), "state": [s.handle.get_state(i) for i in range(s.handle.count)]}
    if kind == "gap":
        dual, energy, labels = s.handle.iterate_gap(k)
        U, phi = s.handle.get_state()
        return {"dual": dual, "energy": energy, "labels": labels, "U": U, "phi": phi}
    if kind == "serve":
        dual = M.solve_noalloc(s.edges, s.unaries, s.pairwise, k, s.U, s.phi)
        return {"dual": dual, "U": s.U, "phi": s.phi}
    if kind == "train":
        s.unaries.grad = s.pairwise.grad = None
        loss = mplp_dual(s.unaries, s.pairwise, s.edges, k, case["every"])
        loss.backward()
        return {"loss": loss.detach(), "unaries": s.unaries.grad, "pairwise": s.pairwise.grad}
    if kind == "oneshot":
        with M.Solver.from_torch(case["n"], case["L"], s.edges, s.unaries, s.pairwise) as h:
            return _solved(h, k, False)
    return _solved(s.handle, k, kind == "trace")


def _solved(h, k, trace):
    out = {}
    if trace:
        out["trace"] = h.iterate_trace(k)
    else:
        h.iterate(k)
    out["dual"] = h.dual_bound()
    out["labels"], out["energy"] = h.decode()
    out["U"], out["phi"] = h.get_state()
    return out


def work(case):
    """Each cost read once and each output written once; an update of an edge takes three
    minimizations of a sum over its table (Sec. 4), each an addition and a minimum an entry."""
    item = 8 if case["dtype"] == "f64" else 4
    if case["kind"] == "batch":
        models = [(n, L, n * (n - 1) // 2) for n, L in _sizes(case, 0)]
    else:
        models = [(case["n"], case["L"], _count(case))]
    b = f = 0
    for n, L, m in models:
        tables = m * (L * L if case["costs"] not in ("linear", "quad", "weights") else 2)
        grads = n * L + tables if case["kind"] == "train" else 0
        state = n * L + m * 2 * L if case["kind"] != "train" else 0
        b += item * (n * L + tables + grads + state)
        f += case["iters"] * m * 6 * L * L
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------
def _matchings(n, edges):
    """The schedule of Alg. 1: the circle method's rounds for a complete graph, greedy
    maximal matchings in ascending edge order otherwise; None where that takes long."""
    m = len(edges)
    if m == n * (n - 1) // 2:
        N = n + (n & 1)
        at = {(int(u), int(v)): i for i, (u, v) in enumerate(edges)}
        rounds = []
        for r in range(N - 1):
            pairs = [(N - 1, r)] + [((r + k) % (N - 1), (r - k) % (N - 1)) for k in range(1, N // 2)]
            got = sorted((min(p), max(p)) for p in pairs if max(p) < n)
            if got:
                rounds.append([at[p] for p in got])
        return rounds
    if m * 4 * m // n > 60_000_000:
        return None
    left, rounds = list(range(m)), []
    us, vs = edges[:, 0].tolist(), edges[:, 1].tolist()
    while left:
        used, got, rest = bytearray(n), [], []
        for e in left:
            if used[us[e]] or used[vs[e]]:
                rest.append(e)
            else:
                used[us[e]] = used[vs[e]] = 1
                got.append(e)
        rounds.append(got)
        left = rest
    return rounds


def _sweeps(edges, un, pw, iters, rounds, after=None):
    """`iters` sweeps of the handshake update from phi = 0; `after(U, phi0, phi1)` is called
    after each.  Messages are lists by round, so that autograd can run through them."""
    order = torch.tensor([e for r in rounds for e in r], device=un.device)
    cuts = [len(r) for r in rounds]
    th = pw[order].split(cuts)
    ends = torch.from_numpy(edges.astype(np.int64)).to(un.device)[order]
    us, vs = ends[:, 0].split(cuts), ends[:, 1].split(cuts)
    zero = torch.zeros((len(edges), un.shape[1]), dtype=un.dtype, device=un.device)
    p0, p1 = list(zero.split(cuts)), list(zero.split(cuts))
    U = un
    for _ in range(iters):
        for k, t in enumerate(th):
            au, av = U[us[k]] - p0[k], U[vs[k]] - p1[k]
            p = (t + av[:, None, :]).min(2)[0]
            b = 0.5 * (au - p)
            q = (t + b[:, :, None]).min(1)[0]
            r = (t - q[:, None, :]).min(2)[0]
            p0[k], p1[k] = r, q
            U = U.index_copy(0, us[k], au + r).index_copy(0, vs[k], av + q)
        if after is not None:
            after(U, p0, p1)
    inv = torch.empty_like(order)
    inv[order] = torch.arange(len(order), device=order.device)
    return U, torch.cat(p0)[inv], torch.cat(p1)[inv]


def _bound(U, pw, phi0, phi1):
    e = (pw - phi0[:, :, None] - phi1[:, None, :]).flatten(1).min(1)[0]
    return float(U.min(1)[0].sum() + e.sum())


def _rounded(n, edges, un, pw, U, phi0, phi1):
    """Nodes in ascending order, each the best label given its lower neighbours'."""
    U, un, phi0, phi1 = (t.cpu().numpy() for t in (U, un, phi0, phi1))
    pw = pw.cpu().numpy()
    below = [[] for _ in range(n)]
    for e, (u, v) in enumerate(edges.tolist()):
        below[v].append((e, u))
    x = np.zeros(n, np.int64)
    for v in range(n):
        c = U[v].copy()
        for e, u in below[v]:
            c += pw[e, x[u]] - phi0[e, x[u]] - phi1[e]
        x[v] = int(c.argmin())
    energy = un[np.arange(n), x].sum() + pw[np.arange(len(edges)), x[edges[:, 0]], x[edges[:, 1]]].sum()
    return x.astype(np.int32), float(energy)


def _expanded(case, prm):
    L = case["L"]
    d = torch.arange(L, dtype=torch.float32)
    d = (d[:, None] - d[None, :]).abs()
    p = torch.from_numpy(prm)
    if case["costs"] == "weights":
        return (p[:, 0, None, None] * (d > 0)).cuda()
    if case["costs"] == "quad":
        d = d * d
    return (p[:, 0, None, None] * torch.minimum(d[None], p[:, 1, None, None])).cuda()


def exact(case, seed):
    kind, k = case["kind"], case["iters"]
    if kind == "batch":
        if sum(n * k for n, _ in _sizes(case, seed)) > 160_000:
            return None
        dual, state = [], []
        for mo in _batch_models(case, seed):
            un, pw = (torch.from_numpy(a).cuda().double() for a in (mo.unaries, mo.pairwise))
            U, p0, p1 = _sweeps(mo.edges, un, pw, k, _matchings(mo.n, mo.edges))
            dual.append(_bound(U, pw, p0, p1))
            state.append((U, torch.stack([p0, p1], 1)))
        return {"dual": np.array(dual), "state": state}
    if kind == "structured":
        edges, un, prm, _ = _structured(case, seed)
        un, pw = torch.from_numpy(un).cuda(), _expanded(case, prm)
    else:
        edges = _edges(case, seed)
        un, pw = _dense(case["n"], case["L"], edges, case["costs"], DTYPES[case["dtype"]], seed)
    un, pw = un.double(), pw.double()
    rounds = _matchings(case["n"], edges)
    if rounds is None:
        return None
    if kind == "train":
        un.requires_grad_(True)
        pw.requires_grad_(True)
        U, p0, p1 = _sweeps(edges, un, pw, k, rounds)
        U.min(1)[0].sum().backward()
        with torch.no_grad():
            return {"loss": torch.tensor(_bound(U, pw, p0, p1), dtype=torch.float64), "unaries": un.grad, "pairwise": pw.grad}
    seen = []

    def after(U, p0, p1):
        if kind == "trace":
            seen.append(float(U.min(1)[0].sum()))
        elif kind == "gap":
            at = torch.tensor([e for r in rounds for e in r], device=U.device)
            seen.append(_bound(U, pw[at], torch.cat(p0), torch.cat(p1)))

    U, p0, p1 = _sweeps(edges, un, pw, k, rounds, after if kind in ("trace", "gap") else None)
    out = {"U": U, "phi": torch.stack([p0, p1], 1)}
    if kind == "gap":
        # (labels and their energies are whole choices: a rounding of the state moves them)
        return dict(out, dual=np.array(seen), energy=None, labels=None)
    out["dual"] = _bound(U, pw, p0, p1)
    if kind == "serve":
        return out
    if kind == "trace":
        out["trace"] = np.array(seen)
    out["labels"] = out["energy"] = None
    if case["dtype"] == "f64":
        out["labels"], out["energy"] = _rounded(case["n"], edges, un, pw, U, p0, p1)
    return out
