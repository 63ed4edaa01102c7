"""What is timed: the sparsifier's calls as a user's program makes them, from one small row to the
whole of a 2^28-coordinate gradient, through the package's public entry points.

A case is a dict of plain values; `kind` names the entry point:

* ``noalloc``   sparsify_sample_compact_batched_noalloc on preallocated outputs (a serving loop)
* ``compact``   Plan: batched solve, sample and compact
* ``hybrid``    Plan(hybrid=True): the Q_A / Q_B coding, optionally with the dense ternary vector
* ``layers``    Plan(segments=...): one lambda per layer of a flat gradient
* ``probs``     sparsify_probs: the keep probabilities of one row
* ``aggregate`` aggregate: the workers' average of their sparse lists

Inputs are drawn on the device with a seeded generator (the logistic-regression gradient on the
host): Laplace rows at scales over three decades, normal rows, Student-t(2) with one per cent of the
coordinates a hundred times larger, layers whose scales span four decades, and the minibatch gradient
of a logistic regression on a sparse design. A Plan's output lists are cleared once in `prepare`, so
the entries past a row's survivors are zero and whole lists compare.

Every sum the sparsifier takes is exact and rounded once, and its output is a pure function of
(g, rho, solver, steps, seed), so the outputs of two builds are equal bit for bit.
"""
import math

import numpy as np
import torch

import paper_1710_09854_amd as gs

# Weight tensors of a 50-layer residual network (53 convolutions with their scale and shift, and the
# classifier), in network order: 54 layers, 25,557,032 coordinates.
_R50 = [
    9536, 4224, 36992, 16896, 16896, 16512, 36992, 16896, 16512, 36992, 16896, 33024, 147712,
    66560, 132096, 65792, 147712, 66560, 65792, 147712, 66560, 65792, 147712, 66560, 131584,
    590336, 264192, 526336, 262656, 590336, 264192, 262656, 590336, 264192, 262656, 590336,
    264192, 262656, 590336, 264192, 262656, 590336, 264192, 525312, 2360320, 1052672, 2101248,
    1049600, 2360320, 1052672, 1049600, 2360320, 1052672, 2049000,
]
_R50_TOTAL = sum(_R50)


def _case(kind, rows, d, dist, solver, rho, **more):
    c = {"kind": kind, "rows": rows, "d": d, "dist": dist, "solver": solver, "rho": rho}
    c.update(more)
    return c


def listed():
    return [
        # a single small gradient in a serving loop: launches and latency
        _case("noalloc", 1, 65536, "normal", "exact", 0.1, name="row_65536_exact"),
        # a small model's layer asked for its probabilities, buffers allocated by the call
        _case("probs", 1, 100003, "normal", "greedy", 0.01, name="probs_100003_greedy"),
        # sixteen simulated workers, one gradient each
        _case("compact", 16, 1 << 20, "laplace", "greedy", 0.01, name="workers_16x1M_greedy"),
        # the same workers with the hybrid coding at a high density
        _case("hybrid", 16, 1 << 20, "laplace", "greedy", 0.1, dense=False, name="hybrid_16x1M_greedy"),
        # rows of odd length in a packed matrix: no row but the first starts on a 16-byte boundary
        _case("compact", 5, 300007, "student", "exact", 0.05, name="ragged_5x300007_exact"),
        # a sparse convex problem: most coordinates are exact zeros
        _case("compact", 1, 1 << 22, "logreg", "exact", 0.01, name="logreg_4M_exact"),
        # a network's whole gradient under one lambda
        _case("compact", 1, _R50_TOTAL, "layers", "exact", 0.001, name="resnet50_25M_exact"),
        # the same gradient layer by layer
        _case("layers", 54, _R50_TOTAL, "layers", "greedy", 0.01, name="resnet50_54_layers_greedy"),
        # a large model's share of one device, at a low and a high density
        _case("compact", 1, 1 << 28, "student", "exact", 0.01, name="grad_268M_exact"),
        _case("compact", 1, 1 << 28, "student", "greedy", 0.1, name="grad_268M_greedy"),
        # the variance budget (rho carries eps)
        _case("compact", 16, 1 << 20, "laplace", "variance", 1.0, name="variance_16x1M"),
        # the workers' messages averaged
        _case("aggregate", 16, 1 << 20, "lists", "none", 0.01, name="aggregate_16x1M"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["noalloc", "compact", "compact", "whole", "whole", "hybrid", "layers", "probs", "variance",
                       "aggregate"])
    rho = math.exp(rng.uniform(math.log(0.001), math.log(0.1)))
    solver = rng.choice(["greedy", "exact"])
    dist = rng.choice(["normal", "laplace", "student"])
    if kind == "noalloc":
        return _case("noalloc", 1, _log(rng, 1000, 1 << 21), dist, solver, rho)
    if kind in ("compact", "hybrid", "variance"):
        rows = _log(rng, 2, 64)
        d = _log(rng, 4096, (1 << 25) // rows)
        if rng.random() < 0.5:
            d = max(4, d & ~3)  # rows on 16-byte boundaries
        if kind == "hybrid":
            return _case("hybrid", rows, d, dist, solver, rho, dense=rng.random() < 0.25)
        if kind == "variance":
            return _case("compact", rows, d, dist, "variance", math.exp(rng.uniform(math.log(0.1), math.log(4.0))))
        return _case("compact", rows, d, dist, solver, rho)
    if kind == "whole":
        d = _log(rng, 1 << 16, 1 << 28)
        if d <= 1 << 24 and rng.random() < 0.25:
            return _case("compact", 1, d, "logreg", solver, rho)
        return _case("compact", 1, d, rng.choice([dist, "layers"]), solver, rho)
    if kind == "layers":
        return _case("layers", _log(rng, 8, 200), _log(rng, 1 << 17, 1 << 25), "layers", solver, rho)
    if kind == "probs":
        return _case("probs", 1, _log(rng, 4096, 1 << 26), dist, solver, rho)
    return _case("aggregate", _log(rng, 2, 64), _log(rng, 1 << 14, 1 << 22), "lists", "none", rho)


# ------------------------------------------------------------------------------------------
# Inputs
# ------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _lengths(case):
    """Layer lengths of a flat gradient: the residual network's where case asks for its size, else
    `rows` lengths spread over two decades that add up to d (a function of the sizes alone)."""
    n, d = case["rows"], case["d"]
    if d == _R50_TOTAL and n in (1, 54):
        return list(_R50)
    n = n if case["kind"] == "layers" else 54
    r = np.random.default_rng(d)
    w = 10.0 ** r.uniform(0.0, 2.0, n)
    cut = np.floor(np.cumsum(w) / w.sum() * d).astype(np.int64)
    if d % 2 == 0:
        cut &= ~np.int64(3)  # half of the sizes: every layer starts on a 16-byte boundary
    cut[-1] = d
    return np.diff(np.concatenate([[0], cut])).tolist()


def _gradient(case, seed):
    rows, d, dist = case["rows"], case["d"], case["dist"]
    g = _gen(seed)
    if dist == "logreg":
        # (1/n) sum_n coef_n x_n on a sparse design of 256 samples at a density of 0.1 per cent
        r = np.random.default_rng(seed)
        m = max(1, d // 1000)
        cols = r.integers(0, d, 256 * m)
        coef = np.repeat(r.choice([-1.0, 1.0], 256) / (2.0 * math.log(2.0) * 256), m)
        x = np.bincount(cols, weights=coef * r.standard_normal(256 * m), minlength=d)
        return torch.from_numpy(x.astype(np.float32)).cuda().reshape(1, d)
    if dist == "layers":
        lens = torch.tensor(_lengths(case), device="cuda")
        sig = 10.0 ** (torch.rand(lens.numel(), generator=g, device="cuda") * 4.0 - 5.0)
        x = torch.randn(d, generator=g, device="cuda")
        x *= torch.repeat_interleave(sig, lens, output_size=d)
        return x.reshape(1, d)
    if dist == "student":
        x = torch.randn(rows, d, generator=g, device="cuda")
        e = torch.empty(rows, d, device="cuda").exponential_(generator=g)
        x /= e.sqrt_().clamp_(min=1e-4)  # Student-t(2): normal over the root of a unit exponential
        e.uniform_(generator=g)
        x *= torch.where(e < 0.01, 100.0, 1.0)
        return x
    x = torch.randn(rows, d, generator=g, device="cuda")
    if dist == "laplace":
        e = torch.empty(rows, d, device="cuda").exponential_(generator=g)
        x = torch.copysign(e, x)
    x *= 10.0 ** (torch.rand(rows, 1, generator=g, device="cuda") * 3.0 - 3.0)
    return x


def _solver(case):
    return "greedy" if case["solver"] == "none" else case["solver"]


def _cap(case, d):
    # the survivors of the variance budget are not known beforehand
    return d if case["solver"] == "variance" else gs.capacity_hint(d, case["rho"])


def _lists(case, seed):
    """Ascending lists of rho * d indices a worker, no two alike, as the sampling pass leaves them."""
    rows, d = case["rows"], case["d"]
    g = _gen(seed)
    cap = gs.capacity_hint(d, case["rho"])
    keep = torch.rand(rows, d, generator=g, device="cuda") < case["rho"]
    nnz = keep.sum(dim=1, dtype=torch.int64)
    idx = torch.zeros((rows, cap), dtype=torch.int32, device="cuda")
    val = torch.zeros((rows, cap), dtype=torch.float32, device="cuda")
    for m in range(rows):
        at = keep[m].nonzero().reshape(-1)[:cap]
        idx[m, :at.numel()] = at.to(torch.int32)
        val[m, :at.numel()] = torch.randn(at.numel(), generator=g, device="cuda")
    return idx, val, nnz.clamp_(max=cap)


def prepare(case, seed):
    kind, rows, d, rho = case["kind"], case["rows"], case["d"], case["rho"]
    if kind == "aggregate":
        idx, val, nnz = _lists(case, seed)
        return {"case": case, "idx": idx, "val": val, "nnz": nnz}
    g = _gradient(case, seed)
    s = {"case": case, "seed": int(seed)}
    if kind == "probs":
        s["g"] = g.reshape(-1)
        return s
    n = rows
    rho_dev = torch.full((n,), rho, dtype=torch.float64, device="cuda")
    seeds = torch.arange(n, dtype=torch.int64, device="cuda") + 1000 * (int(seed) + 1)
    s.update(g=g, rho=rho_dev, seeds=seeds)
    if kind == "noalloc":
        cap = _cap(case, d)
        s["out"] = {
            "idx": torch.zeros((n, cap), dtype=torch.int32, device="cuda"),
            "val": torch.zeros((n, cap), dtype=torch.float32, device="cuda"),
            "nnz": torch.zeros(n, dtype=torch.int64, device="cuda"),
            "lam": torch.zeros(n, dtype=torch.float64, device="cuda"),
            "k": torch.zeros(n, dtype=torch.int64, device="cuda"),
            "flags": torch.zeros(n, dtype=torch.int32, device="cuda"),
        }
        return s
    if kind == "layers":
        seg = gs.Segments.from_lengths(_lengths(case))
        p = gs.Plan(seg.segs, seg.max_len, solver=_solver(case), cap_per_row=_cap(case, seg.max_len), segments=seg)
        s["g"] = g.reshape(-1)
    else:
        p = gs.Plan(rows, d, solver=_solver(case), cap_per_row=_cap(case, d), hybrid=kind == "hybrid",
                    dense_q=bool(case.get("dense", False)))
    p.idx.zero_()
    p.val.zero_()
    if kind == "hybrid":
        p.code_b.zero_()
    s["plan"] = p
    return s


# ------------------------------------------------------------------------------------------
# One pass
# ------------------------------------------------------------------------------------------
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "aggregate":
        return {"v": gs.aggregate(state["idx"], state["val"], state["nnz"], case["d"])}
    if kind == "probs":
        o = gs.sparsify_probs(state["g"], case["rho"], solver=_solver(case))
        return {"p": o.p, "lam": o.lam, "k": o.k, "flags": o.flags}
    if kind == "noalloc":
        o = state["out"]
        rc = gs.sparsify_sample_compact_batched_noalloc(state["g"], state["rho"], state["seeds"], o["idx"], o["val"],
                                                        o["nnz"], o["lam"], o["k"], o["flags"], solver=_solver(case))
        if rc != gs.OK:
            raise RuntimeError("noalloc call refused: %d" % rc)
        return o
    p = state["plan"]
    p.run(state["g"], state["rho"], state["seeds"])
    out = {"idx": p.idx, "val": p.val, "nnz": p.nnz, "lam": p.lam, "flags": p.flags}
    if kind == "hybrid":
        out.update(code_b=p.code_b, nnz_b=p.nnz_b, inv=p.inv)
        if p.q is not None:
            out["q"] = p.q
    else:
        out["k"] = p.k
    return out


def work(case):
    kind, d, rho = case["kind"], case["d"], case["rho"]
    n = (1 if kind == "layers" else case["rows"]) * d
    if kind == "aggregate":
        return {"bytes": 8.0 * rho * n + 4.0 * d, "flops": rho * n}
    if kind == "probs":
        return {"bytes": 8.0 * n, "flops": 2.0 * n}
    # variance budget: (sum |g|)^2 / ((1 + eps) sum g^2) coordinates while few are capped, half of
    # n / (1 + eps) for Laplace rows
    kept = n * (0.5 / (1.0 + rho) if case["solver"] == "variance" else rho)
    out = (6.0 if kind == "hybrid" else 8.0) * kept + (n if case.get("dense", False) else 0)
    return {"bytes": 4.0 * n + out, "flops": 2.0 * n}


def tolerance(case):
    # sums are exact and rounded once, and the draws are a fixed function of (seed, index): a change
    # of launch, order or layout changes no bit of any output
    return "exact"


# ------------------------------------------------------------------------------------------
# The same in 64-bit torch
# ------------------------------------------------------------------------------------------
def _solve64(x, rho, solver, iters=2):
    """(lambda, capped mask) of one row by sorting, in fp64."""
    a = x.abs().double()
    n = a.numel()
    if solver == "variance":
        s = torch.sort(a, descending=True).values
        w = torch.cumsum(s, 0)
        h = torch.cumsum(s * s, 0)
        t1 = w[-1] - torch.cat([w.new_zeros(1), w[:-1]])
        t2 = h[-1] - torch.cat([h.new_zeros(1), h[:-1]])
        rhs = rho * h[-1] + t2
        k = int((s * t1 <= rhs).to(torch.int8).argmax())
        lam, v = float(t1[k] / rhs[k]), s[k]
        return lam, (a > v) | (lam * a >= 1.0)
    b = rho * n
    if b >= float((a > 0).sum()):
        return math.inf, a > 0
    total = float(a.sum())
    if solver == "greedy":
        lam = b / total
        for _ in range(iters):
            c = lam * a >= 1.0
            u = float(torch.where(c, 0.0, a).sum())
            if u == 0.0:
                break
            new = (b - float(c.sum())) / u
            if not new > lam:
                break
            lam = new
        return lam, lam * a >= 1.0
    # at most b magnitudes are capped (each counts 1 towards the budget)
    s = torch.topk(a, min(n, int(b) + 2)).values if n <= 1 << 24 else torch.sort(a, descending=True).values[:int(b) + 2]
    w = torch.cat([s.new_zeros(1), torch.cumsum(s, 0)[:-1]])
    k0 = torch.arange(s.numel(), dtype=torch.float64, device=s.device)
    k = int(((b - k0) * s <= total - w).to(torch.int8).argmax())
    lam = (b - k) / (total - float(w[k]))
    return lam, (a > s[k]) | (lam * a >= 1.0)


def _philox64(n, seed):
    """n words of Philox4x32-10 keyed (seed low, seed high) at counters (i / 4, 0, 0, 0)."""
    q = torch.arange((n + 3) // 4, dtype=torch.int64, device="cuda")
    m32 = 0xFFFFFFFF
    c = [q & m32, q >> 32, torch.zeros_like(q), torch.zeros_like(q)]
    k0, k1 = seed & m32, (seed >> 32) & m32
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57  # the low 64 bits: wrapping, as unsigned
        c = [((p1 >> 32) & m32) ^ c[1] ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c[3] ^ k1, p0 & m32]
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return torch.stack(c, dim=1).reshape(-1)[:n]


def _row64(x, rho, solver, seed):
    lam, capped = _solve64(x, rho, solver)
    p = torch.where(capped, 1.0, lam * x.abs().double()) if lam < math.inf else capped.double()
    keep = (_philox64(x.numel(), seed).double() < p * 2.0 ** 32) & (x != 0)
    at = keep.nonzero().reshape(-1)
    cap_at = capped[at]
    inv = 1.0 / lam if 0.0 < lam < math.inf else 0.0
    val = torch.where(cap_at, x[at].double(), torch.sign(x[at]).double() * inv)
    return lam, at, val, cap_at, inv


def exact(case, seed):
    kind, d, rho, solver = case["kind"], case["d"], case["rho"], _solver(case)
    if kind == "aggregate":
        idx, val, nnz = _lists(case, seed)
        v = torch.zeros(d, dtype=torch.float64, device="cuda")
        for m in range(case["rows"]):
            n = int(nnz[m])
            v[idx[m, :n].long()] += val[m, :n].double()
        return {"v": v / case["rows"]}
    g = _gradient(case, seed)
    if kind == "probs":
        x = g.reshape(-1)
        lam, capped = _solve64(x, rho, solver)
        p = torch.where(capped, 1.0, lam * x.abs().double()) if lam < math.inf else capped.double()
        return {"p": p, "lam": torch.tensor([lam], dtype=torch.float64), "k": None, "flags": None}
    if kind == "layers":
        lens = _lengths(case)
        parts = list(torch.split(g.reshape(-1), lens))
        cap = _cap(case, max(1, max(lens)))
    else:
        parts = list(g)
        cap = _cap(case, d)
    rows = len(parts)
    val = torch.zeros((rows, cap), dtype=torch.float64, device="cuda")
    lams, invs, q = [], [], []
    for r, x in enumerate(parts):
        if x.numel() == 0 or not bool((x != 0).any()):
            lams.append(math.inf)
            invs.append(0.0)
            continue
        lam, at, v, cap_at, inv = _row64(x, rho, solver, r + 1000 * (int(seed) + 1))
        lams.append(lam)
        invs.append(inv)
        if kind == "hybrid":
            v = v[cap_at]
        v = v[:cap]
        val[r, :v.numel()] = v
    out = {"idx": None, "val": val, "nnz": None, "lam": torch.tensor(lams, dtype=torch.float64), "flags": None}
    if kind == "hybrid":
        out.update(code_b=None, nnz_b=None, inv=torch.tensor(invs, dtype=torch.float64))
        if case.get("dense", False):
            out["q"] = None
    else:
        out["k"] = None
    return out
