"""Performance cases of the reachability library: whole calls through its public
entry points, on inputs drawn on the GPU from a seed.

A case names a family of chains (or of general systems), its sizes, the call
and its options.  ``prepare`` builds what a program holds before the call --
the chain in compressed row storage on the GPU, a context and, where the case
keeps one, the system of ``rp_precompute`` -- and ``run`` makes the call.

Families (the generators follow the shapes of chaingen, drawn with torch so
that millions of states take milliseconds; targets drawn twice in a row are
merged):

* ``ruin``     gambler's ruin: a walk on 0..n-1 with up-probability near 0.45
* ``sparse``   K chains of n states, out-degree 1..dmax, uniform targets
* ``mixed``    K such chains with log-uniform sizes nmin..nmax
* ``dense``    every transition present with probability ``density``
* ``program``  model-checker graphs: coin-flip probabilities, successors within
               64 states except for 2% uniform jumps
* ``matrix``   K general systems A x = b, diagonally dominant positive integers
"""
import math

import numpy as np
import torch

import paper_1210_6412_amd as rp

_DEV = "cuda"
_LEAK = {"sparse": 0.02, "mixed": 0.02, "dense": 0.01, "program": 0.011, "ruin": 0.005, "matrix": 0.02}


def listed():
    return [
        # The smallest solve: one 1,000-state walk under the paper's own
        # stopping rule, thousands of tiny sweeps on a system that is kept.
        dict(name="ruin_1k_jacobi_paper", kind="ruin", n=1000, call="solve", keep=True, method="jacobi",
             precision="fp64", stop="delta", tol=1e-12),
        # A batch of small sparse systems of the paper's Table 1 sizes, built
        # and solved in one go: launches and host work count.
        dict(name="table1_40_bicgstab", kind="matrix", K=40, n=313, density=0.004, call="solve", keep=False,
             method="bicgstab", precision="fp64", stop="certified", tol=1e-10),
        # One system of the paper's density experiments, built and solved.
        dict(name="matrix_4k_bicgstab", kind="matrix", K=1, n=4000, density=0.10, call="solve", keep=False,
             method="bicgstab", precision="fp64", stop="certified", tol=1e-10),
        # A training step on one chain: probabilities and their gradient
        # through the autograd function.
        dict(name="sparse_20k_autograd", kind="sparse", K=1, n=20_000, dmax=16, call="autograd", keep=False,
             method="bicgstab", precision="fp64", stop="certified", tol=1e-10),
        # The same chain solved again and again on a kept system: one sweep
        # moves 2 MB, so latency counts.
        dict(name="sparse_20k_jacobi", kind="sparse", K=1, n=20_000, dmax=16, call="solve", keep=True,
             method="jacobi", precision="fp64", stop="certified", tol=1e-10),
        # Long rows (about 820 entries each).
        dict(name="dense_8k_jacobi", kind="dense", n=8192, density=0.10, call="solve", keep=True, method="jacobi",
             precision="fp64", stop="certified", tol=1e-10),
        # A model checker's graph, from the chain to the answer.
        dict(name="program_2m_jacobi", kind="program", n=2_000_000, call="solve", keep=False, method="jacobi",
             precision="fp64", stop="certified", tol=1e-10),
        # Equal chains batched, mixed precision, from the chains to the answers.
        dict(name="batch64_jacobi_f32r", kind="sparse", K=64, n=20_000, dmax=16, call="solve", keep=False,
             method="jacobi", precision="fp32r", stop="certified", tol=1e-10),
        # The benchmark's batch (256 chains of 1,000..200,000 states): Jacobi
        # in FP64 from the chains to the answers ...
        dict(name="mixed256_jacobi_f64", kind="mixed", K=256, nmin=1000, nmax=200_000, dmax=8, call="solve",
             keep=False, method="jacobi", precision="fp64", stop="certified", tol=1e-10),
        # ... in mixed precision on a kept system ...
        dict(name="mixed256_jacobi_f32r", kind="mixed", K=256, nmin=1000, nmax=200_000, dmax=8, call="solve",
             keep=True, method="jacobi", precision="fp32r", stop="certified", tol=1e-10),
        # ... and the gradient: forward solve, adjoint solve, dL/dP.
        dict(name="mixed256_bicgstab_grad", kind="mixed", K=256, nmin=1000, nmax=200_000, dmax=8, call="gradient",
             keep=False, method="bicgstab", precision="fp32r", stop="certified", tol=1e-10),
        # The largest graph, no cache holds it: BiCGStab in FP64 on a kept system.
        dict(name="program_33m_bicgstab", kind="program", n=33_554_432, call="solve", keep=True, method="bicgstab",
             precision="fp64", stop="certified", tol=1e-10),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    c = dict(kind=rng.choice(["ruin", "sparse", "sparse", "mixed", "mixed", "dense", "program", "program", "matrix"]))
    kind = c["kind"]
    if kind == "ruin":
        c["n"] = _log(rng, 100, 4000)
    elif kind == "sparse":
        c["K"] = _log(rng, 1, 128)
        c["n"] = _log(rng, 500, 2_500_000 // c["K"])
        c["dmax"] = rng.choice([4, 8, 13, 16])
    elif kind == "mixed":
        c["K"] = _log(rng, 4, 256)
        c["nmin"] = _log(rng, 300, 3000)
        c["nmax"] = _log(rng, 20_000, 200_000)
        c["dmax"] = rng.choice([5, 8])
    elif kind == "dense":
        c["n"] = _log(rng, 500, 8192)
        c["density"] = round(rng.uniform(0.02, 0.10), 3)
    elif kind == "program":
        c["n"] = _log(rng, 50_000, 4_000_000)
    else:
        c["K"] = rng.choice([1, 1, 5, 40])
        c["n"] = _log(rng, 92, 4000 if c["K"] == 1 else 1000)
        c["density"] = round(rng.uniform(0.004, 0.10), 4)
    c["call"] = "solve" if kind in ("ruin", "dense", "matrix") else rng.choice(["solve", "solve", "gradient", "autograd"])
    c["keep"] = c["call"] == "solve" and rng.random() < 0.5
    c["method"] = "bicgstab" if kind == "matrix" else "jacobi" if kind == "ruin" else rng.choice(["jacobi", "bicgstab"])
    c["precision"] = rng.choice(["fp64", "fp32r"])
    c["stop"], c["tol"] = "certified", 1e-10
    if kind == "ruin":
        c["precision"], c["stop"], c["tol"] = "fp64", "delta", 1e-12
    return c


def _sizes(case):
    """States of each packed chain or system."""
    if case["kind"] == "mixed":
        K = case["K"]
        q = (np.arange(K) + 0.5) / K
        lo, hi = math.log(case["nmin"]), math.log(case["nmax"])
        return np.rint(np.exp(lo + q * (hi - lo))).astype(np.int64)
    return np.full(case.get("K", 1), case["n"], dtype=np.int64)


def _entries(case):
    """Expected stored transitions (matrix entries)."""
    kind, n = case["kind"], float(_sizes(case).sum())
    if kind == "ruin":
        return 2 * n
    if kind in ("sparse", "mixed"):
        return n * (1 + case["dmax"]) / 2
    if kind == "program":
        return 3 * n
    return n * (1 + case["density"] * case["n"])


def work(case):
    """Inputs read once and results written once; two operations per stored
    entry and iteration for about as many iterations as the method needs on
    the family (Jacobi: the error falls by the share of goals and sinks)."""
    n, z = float(_sizes(case).sum()), _entries(case)
    if case["method"] == "jacobi":
        sweeps = math.log(100.0 / case["tol"]) / _LEAK[case["kind"]]
    else:
        sweeps = 2 * 40.0
    nbytes = 12 * z + 4 * n + n + 8 * n
    flops = 2 * z * sweeps
    if case["call"] != "solve":
        nbytes += 8 * n + 8 * z + 8 * n
        flops *= 2
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# inputs

def _rand(g, n):
    return torch.rand(n, generator=g, device=_DEV, dtype=torch.float64)


def _csr(n, rows, cols, redraw):
    """Distinct, sorted transitions (a target drawn twice in a row is drawn
    again): row pointers, rows and columns."""
    key = torch.sort(rows * n + cols)[0]
    while True:
        twice = torch.nonzero(key[1:] == key[:-1]).reshape(-1) + 1
        if twice.shape[0] == 0:
            break
        r = key[twice] // n
        key[twice] = r * n + redraw(r)
        key = torch.sort(key)[0]
    rows, cols = key // n, key % n
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=_DEV)
    ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return ptr, rows, cols


def _weights(g, rows, n):
    """Uniform weights normalised per row (integer sums, so that the same
    seed gives the same bits)."""
    w = torch.randint(1, (1 << 20) + 1, rows.shape, generator=g, device=_DEV)
    total = torch.zeros(n, dtype=torch.int64, device=_DEV).index_add_(0, rows, w)
    return w.double() / total[rows].double()


def _roles(g, offs, n, goals, sinks):
    """Goal and sink states (shares of each chain's states, at least one of
    each), and each state's place in a random order of its chain's others."""
    size = torch.from_numpy(np.diff(offs)).to(_DEV)
    inst = torch.arange(len(offs) - 1, device=_DEV).repeat_interleave(size)
    order = torch.argsort(inst + _rand(g, n) * 0.999, stable=True)
    place = torch.empty(n, dtype=torch.int64, device=_DEV)
    place[order] = torch.arange(n, device=_DEV) - torch.from_numpy(offs[:-1]).to(_DEV)[inst]
    ng = torch.clamp((size * goals).long(), min=1)[inst]
    ns = torch.clamp((size * sinks).long(), min=1)[inst]
    return inst, place < ng, (place >= ng) & (place < ng + ns), place


def _chain(case, g, rng):
    kind = case["kind"]
    sizes = rng.permutation(_sizes(case))
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(offs[-1])
    state = torch.arange(n, device=_DEV)
    if kind == "ruin":
        up = 0.44 + 0.02 * _rand(g, n)
        goal, sink = state == n - 1, state == 0
        inner = state[1:-1]
        rows = torch.cat([state[:1], inner.repeat_interleave(2), state[-1:]])
        cols = torch.cat([state[:1], torch.stack([inner - 1, inner + 1], 1).reshape(-1), state[-1:]])
        one = torch.ones(1, dtype=torch.float64, device=_DEV)
        val = torch.cat([one, torch.stack([1 - up[1:-1], up[1:-1]], 1).reshape(-1), one])
        ptr = torch.zeros(n + 1, dtype=torch.int64, device=_DEV)
        ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
        return n, offs, ptr, rows, cols, val, goal, sink
    if kind == "dense":
        inst, goal, sink, place = _roles(g, offs, n, 0.005, 0.005)
        present = torch.rand(n, n, generator=g, device=_DEV) < case["density"]
        present[sink] = False
        alone = ~present.any(1)
        present[alone, alone] = True
        rows, cols = torch.nonzero(present, as_tuple=True)
        ptr = torch.zeros(n + 1, dtype=torch.int64, device=_DEV)
        ptr[1:] = torch.cumsum(present.sum(1), 0)
        return n, offs, ptr, rows, cols, _weights(g, rows, n), goal, sink
    if kind == "program":
        inst, goal, sink, place = _roles(g, offs, n, 0.01, 0.001)
        absorbing, least, most = goal | sink, 2, 4

        def targets(r):
            m = r.shape[0]
            step = torch.randint(1, 65, (m,), generator=g, device=_DEV)
            t = (r + torch.where(torch.rand(m, generator=g, device=_DEV) < 0.5, -step, step)).abs()
            t = torch.where(t >= n, 2 * (n - 1) - t, t)
            far = torch.randint(0, n, (m,), generator=g, device=_DEV)
            return torch.where(torch.rand(m, generator=g, device=_DEV) < 0.02, far, t)
    else:
        inst, goal, sink, place = _roles(g, offs, n, 0.01, 0.01)
        absorbing, least, most = sink, 1, case["dmax"]
        size, base = torch.from_numpy(sizes).to(_DEV), torch.from_numpy(offs[:-1]).to(_DEV)

        def targets(r):
            k = inst[r]
            return base[k] + torch.minimum((_rand(g, r.shape[0]) * size[k]).long(), size[k] - 1)
    # out-degrees least..most in equal shares, one self-loop on absorbing states
    deg = torch.where(absorbing, torch.ones_like(place), least + place % (most - least + 1))
    rows = state.repeat_interleave(deg)
    cols = torch.where(absorbing[rows], rows, targets(rows))
    ptr, rows, cols = _csr(n, rows, cols, targets)
    if kind == "program":
        # coin flips: 1; 1/2, 1/2; 1/2, 1/4, 1/4 in some order; 1/4 four times
        deg = (ptr[1:] - ptr[:-1])[rows]
        pos = torch.arange(rows.shape[0], device=_DEV) - ptr[rows]
        lead = torch.randint(0, 3, (n,), generator=g, device=_DEV)[rows]
        val = torch.where(deg == 1, 1.0, torch.where(deg == 2, 0.5, torch.where((deg == 3) & (pos == lead), 0.5, 0.25)))
        val = val.double()
    else:
        val = _weights(g, rows, n)
    return n, offs, ptr, rows, cols, val, goal, sink


def _matrix(case, g):
    K, m = case.get("K", 1), case["n"]
    offs = (np.arange(K + 1) * m).astype(np.int64)
    present = torch.rand(K, m, m, generator=g, device=_DEV) < case["density"]
    a = torch.randint(1, 11, (K, m, m), generator=g, device=_DEV) * present
    diag = torch.arange(m, device=_DEV)
    a[:, diag, diag] = 0
    a[:, diag, diag] = a.sum(2) + torch.randint(1, 11, (K, m), generator=g, device=_DEV)
    rhs = torch.randint(1, 11, (K * m,), generator=g, device=_DEV).double()
    return offs, a.double(), rhs


def _gens(seed):
    return torch.Generator(device=_DEV).manual_seed(int(seed)), np.random.Generator(np.random.PCG64(int(seed)))


def _seeds(case, g, offs, goal, sink):
    """dL/dx: one undecided state's probability per chain, weighted."""
    n = goal.shape[0]
    usable = ~(goal | sink)
    order = torch.where(usable, _rand(g, n), torch.full((n,), -1.0, dtype=torch.float64, device=_DEV))
    seed = torch.zeros(n, dtype=torch.float64, device=_DEV)
    sizes = torch.from_numpy(np.diff(offs)).to(_DEV)
    if len(offs) == 2:
        at = order.argmax().reshape(1)
    else:
        inst = torch.arange(len(offs) - 1, device=_DEV).repeat_interleave(sizes)
        best = torch.full((len(offs) - 1,), -1.0, dtype=torch.float64, device=_DEV)
        best = best.scatter_reduce(0, inst, order, "amax")
        at = torch.nonzero(order == best[inst]).reshape(-1)
    seed[at] = 0.5 + _rand(g, at.shape[0])
    return seed


def _inputs(case, seed):
    g, rng = _gens(seed)
    if case["kind"] == "matrix":
        offs, a, rhs = _matrix(case, g)
        k, i, j = torch.nonzero(a, as_tuple=True)
        m = case["n"]
        ptr = torch.zeros(a.shape[0] * m + 1, dtype=torch.int64, device=_DEV)
        ptr[1:] = torch.cumsum((a != 0).sum(2).reshape(-1), 0)
        return dict(row_ptr=ptr.int(), col=(k * m + j).int(), val=a[k, i, j].contiguous(), rhs=rhs,
                    off=[int(v) for v in offs])
    n, offs, ptr, rows, cols, val, goal, sink = _chain(case, g, rng)
    return dict(row_ptr=ptr.int(), col=cols.int(), val=val, goal=goal.to(torch.uint8), off=[int(v) for v in offs],
                seed=_seeds(case, g, offs, goal, sink) if case["call"] != "solve" else None)


# ---------------------------------------------------------------------------
# the call

def _opts(case):
    return dict(tol=case["tol"],
                stop=rp.RP_STOP_DELTA if case["stop"] == "delta" else rp.RP_STOP_CERTIFIED,
                precision=rp.RP_FP64 if case["precision"] == "fp64" else rp.RP_FP32_REFINED)


def _system(s, cls=None):
    if "rhs" in s:
        return rp.rp_matrix_system(s["ctx"], s["row_ptr"], s["col"], s["val"], s["rhs"], s["off"])
    return rp.rp_precompute(s["ctx"], s["row_ptr"], s["col"], s["val"], s["goal"], s["off"], class_out=cls)


def prepare(case, seed):
    s = _inputs(case, seed)
    s.update(call=case["call"], method=0 if case["method"] == "jacobi" else 1, opts=_opts(case),
             ctx=rp.rp_context_create(torch.cuda.current_device()))
    s["sys"] = _system(s) if case["keep"] else None
    if case["call"] == "autograd":
        s["val"].requires_grad_(True)
    return s


def run(s):
    ctx = s["ctx"]
    if s["call"] == "autograd":
        x = rp.reach_prob(s["val"], ctx, s["row_ptr"], s["col"], s["goal"], s["off"], method=s["method"], **s["opts"])
        (grad,) = torch.autograd.grad(x, s["val"], s["seed"])
        return {"x": x.detach(), "grad": grad}
    solve = rp.rp_jacobi if s["method"] == 0 else rp.rp_bicgstab
    if s["sys"] is not None:
        x, _, code = solve(ctx, s["sys"], **s["opts"])
        if code != 0:
            raise RuntimeError(rp.rp_last_error(ctx))
        return {"x": x}
    out = {}
    if "goal" in s:
        out["classes"] = torch.empty(s["goal"].shape[0], dtype=torch.uint8, device=s["goal"].device)
    system = _system(s, out.get("classes"))
    out["x"], _, code = solve(ctx, system, **s["opts"])
    if code != 0:
        raise RuntimeError(rp.rp_last_error(ctx))
    if s["call"] == "gradient":
        out["lam"], out["grad"], _, code = rp.rp_adjoint(ctx, system, out["x"], s["seed"], s["method"], **s["opts"])
        if code != 0:
            raise RuntimeError(rp.rp_last_error(ctx))
    rp.rp_system_destroy(system)
    return out


# ---------------------------------------------------------------------------
# the same in plain torch, 64 bits

def _products(n, ptr, rows, cols, val):
    """v -> P v and v -> v P of a chain."""
    width = int((ptr[1:] - ptr[:-1]).max())
    if width <= 32:  # rows padded to one length, so that a product is a gather and a sum
        pos = torch.arange(rows.shape[0], device=_DEV) - ptr[rows]
        pc = torch.zeros(n, width, dtype=torch.int32, device=_DEV)
        pv = torch.zeros(n, width, dtype=torch.float64, device=_DEV)
        pc[rows, pos] = cols.int()
        pv[rows, pos] = val
        del pos

        def right(v):
            return (v.index_select(0, pc.reshape(-1)).reshape(n, width) * pv).sum(1)
    else:
        dense = torch.zeros(n, n, dtype=torch.float64, device=_DEV)
        dense[rows, cols] = val

        def right(v):
            return dense @ v

    def left(v):
        return torch.zeros(n, dtype=torch.float64, device=_DEV).index_add_(0, cols, v[rows] * val)

    return right, left


def _search(right, start, blocked):
    """States that reach `start` without passing a blocked state."""
    mark = start.double()
    while True:
        more = torch.where(blocked, mark, torch.maximum(mark, (right(mark) > 0).double()))
        if torch.equal(more, mark):
            return mark > 0
        mark = more


def _solve(apply, b):
    """apply(x) = b by BiCGStab, restarted on the true residual until that is
    rounding (all chains of a batch as one system)."""
    x, best, stuck = torch.zeros_like(b), math.inf, 0
    for _ in range(60):
        r = b - apply(x)
        size = float(r.abs().max())
        stuck = 0 if size < 0.5 * best else stuck + 1
        if size == 0.0 or stuck == 3:
            break
        best = min(best, size)
        q, p, d = r.clone(), r.clone(), torch.zeros_like(b)
        rho = first = torch.dot(r, r)
        for _ in range(60):
            v = apply(p)
            alpha = rho / torch.dot(q, v)
            s = r - alpha * v
            t = apply(s)
            omega = torch.dot(t, s) / torch.dot(t, t)
            d = d + alpha * p + omega * s
            r = s - omega * t
            if not float(torch.dot(r, r)) > 1e-16 * float(first):
                break
            new = torch.dot(q, r)
            p = r + (new / rho) * (alpha / omega) * (p - omega * v)
            rho = new
        d = torch.where(torch.isfinite(d), d, torch.zeros_like(d))
        if float((b - apply(x + d)).abs().max()) < size:
            x = x + d
        else:  # a step of the plain iteration, which always converges
            for _ in range(50):
                x = x + (b - apply(x))
    return x


def exact(case, seed):
    g, rng = _gens(seed)
    if case["kind"] == "matrix":
        _, a, rhs = _matrix(case, g)
        return {"x": torch.linalg.solve(a, rhs.reshape(a.shape[0], -1, 1)).reshape(-1)}
    n, offs, ptr, rows, cols, val, goal, sink = _chain(case, g, rng)
    seed_v = _seeds(case, g, offs, goal, sink) if case["call"] != "solve" else None
    if case["kind"] == "ruin":
        p = torch.zeros(n, n, dtype=torch.float64, device=_DEV)
        p[rows, cols] = val
        a = torch.eye(n, dtype=torch.float64, device=_DEV) - p
        fixed = goal | sink
        a[fixed] = 0.0
        a[fixed, fixed] = 1.0
        return {"x": torch.linalg.solve(a, goal.double())}
    right, left = _products(n, ptr, rows, cols, val)
    reach = _search(right, goal, torch.zeros_like(goal))
    lost = _search(right, ~reach, goal)
    undecided = reach & lost & ~goal
    one, m = (reach & ~undecided).double(), undecided.double()
    x = one + _solve(lambda v: m * (v - right(v)), m * right(one))
    out = {"x": x}
    if not case["keep"] and case["call"] != "autograd":
        out["classes"] = None
    if case["call"] == "solve":
        return out
    lam = _solve(lambda v: m * (v - left(v)), m * seed_v)
    if case["call"] == "gradient":
        out["lam"] = lam
    out["grad"] = lam[rows] * x[cols]
    return out
