"""Timed workloads of the PDHG library, through its public Python binding.

A case is a dict of plain values.  ``prepare`` draws its LPs on the GPU from
a seed and builds what a user's program keeps (a batch handle whose first
solve has chosen its layouts, start points, objectives), ``run`` is one call
sequence of such a program, ``work`` the bytes and operations it cannot do
without, and ``exact`` the same outputs in FP64 by plain torch operations.

Solves that are cut off stop after at most 192 iterations: the first
restarts are then taken by the rule's iteration term alone, so two
arithmetically equal implementations take the same decisions.  Adaptive steps
amplify rounding from iteration to iteration and stop after 32.
"""
import math

import numpy as np
import torch

from paper_2307_03466_amd import instances, pdhg

DEV = "cuda"
TOL_CUT = 1e-9  # tolerance of the solves that end at their iteration limit


# ----------------------------------------------------------------- cases
def listed():
    return [
        # One 200 x 500 set-cover relaxation in FP64 to a relative KKT error
        # of 1e-4 on a kept handle: thousands of iterations of an instance
        # that fits one compute unit, all latency.
        {"name": "cover_to_tolerance_fp64", "path": "tolerance", "family": "cover", "count": 1, "rows": 200,
         "precision": "fp64"},
        # The smallest call: one host-array LP through the one-shot entry
        # point, setup included (a heuristic solving many unrelated small
        # relaxations).
        {"name": "cover_oneshot_fp32", "path": "oneshot", "family": "cover", "count": 1, "rows": 200, "iters": 192,
         "precision": "fp32"},
        # 256 set-cover relaxations of uneven odd sizes in one handle, each
        # small enough for one compute unit (sub-problems of a search tree).
        {"name": "covers_256_fp32", "path": "solve", "family": "cover", "count": 256, "rows": 61, "rows_max": 263,
         "iters": 192, "precision": "fp32", "adaptive": False, "average": False},
        # One medium binary LP with restarts to the average: too large for
        # one compute unit, too small to fill the chip.
        {"name": "knapsack_5k_average_fp32", "path": "solve", "family": "knapsack", "count": 1, "rows": 5003,
         "iters": 192, "precision": "fp32", "adaptive": False, "average": True},
        # The headline LP: 1M x 2M, 10M nonzeros, uniform columns.
        {"name": "general_1m_fp32", "path": "solve", "family": "general", "count": 1, "rows": 1_000_000,
         "iters": 192, "precision": "fp32", "adaptive": False, "average": False},
        # Full precision with adaptive steps on a general LP a fifth of it.
        {"name": "general_200k_adaptive_fp64", "path": "solve", "family": "general", "count": 1, "rows": 200_001,
         "iters": 32, "precision": "fp64", "adaptive": True, "average": False},
        # Power-law row lengths: mixed pattern and integer rows, the longest
        # tens of thousands of nonzeros, short columns and long rows.
        {"name": "skewed_250k_fp32", "path": "solve", "family": "skewed", "count": 1, "rows": 250_000, "iters": 128,
         "precision": "fp32", "adaptive": False, "average": False},
        # A batch of binary LPs whose sizes span a factor of 50.
        {"name": "uneven_64_fp32", "path": "solve", "family": "knapsack", "count": 64, "rows": 1_000,
         "rows_max": 50_000, "iters": 128, "precision": "fp32", "adaptive": False, "average": False},
        # One round of the pump on 64 equal instances: objective update of
        # every instance, warm re-solve, MIP-feasibility test of the iterate.
        {"name": "pump_round_64x20k_fp32", "path": "pump", "family": "knapsack", "count": 64, "rows": 20_000,
         "iters": 64, "precision": "fp32"},
        # A new objective on a large resident LP and a short warm re-solve.
        {"name": "resolve_300k_fp32", "path": "resolve", "family": "general", "count": 1, "rows": 300_007, "iters": 64,
         "precision": "fp32", "quadratic": False},
        # The L2-distance form of that on a batch: linear and diagonal
        # quadratic objective of every instance, then a warm re-solve.
        {"name": "resolve_l2_16x5k_fp32", "path": "resolve", "family": "knapsack", "count": 16, "rows": 5_000,
         "iters": 64, "precision": "fp32", "quadratic": True},
        # Fix-and-propagate of a batch on the device, 16 fixings at a time.
        {"name": "round_16x2k_fp32", "path": "round", "family": "knapsack", "count": 16, "rows": 2_001, "fix": 16,
         "precision": "fp32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above."""
    kind = rng.randrange(8)
    prec = rng.choice(["fp32", "fp32", "fp64"])
    if kind == 0:
        return {"path": "tolerance", "family": "cover", "count": 1, "rows": rng.randint(60, 240), "precision": "fp64"}
    if kind == 1:
        return {"path": "oneshot", "family": rng.choice(["cover", "knapsack", "general"]), "count": 1,
                "rows": _log(rng, 40, 2_000), "iters": rng.choice([64, 100, 192]), "precision": prec}
    if kind == 2:
        lo = rng.randint(20, 90)
        return {"path": "solve", "family": "cover", "count": rng.randint(8, 300), "rows": lo,
                "rows_max": rng.randint(lo, 270), "iters": rng.choice([64, 192]), "precision": "fp32",
                "adaptive": False, "average": False}
    if kind in (3, 4):
        # one LP, from a few hundred rows to most of the headline size
        adaptive = prec == "fp64" and rng.random() < 0.5
        family = rng.choice(["general", "general", "skewed", "knapsack"])
        top = {"general": 700_000, "skewed": 150_000, "knapsack": 100_000}[family] // (2 if prec == "fp64" else 1)
        return {"path": "solve", "family": family, "count": 1, "rows": _log(rng, 500, top),
                "iters": 32 if adaptive else rng.choice([64, 100, 128]), "precision": prec, "adaptive": adaptive,
                "average": not adaptive and rng.random() < 0.25}
    if kind == 5:
        lo = _log(rng, 300, 3_000)
        return {"path": "solve", "family": "knapsack", "count": rng.randint(4, 48), "rows": lo,
                "rows_max": _log(rng, lo, 40_000), "iters": rng.choice([64, 128]), "precision": prec,
                "adaptive": False, "average": False}
    if kind == 6:
        if rng.random() < 0.5:
            return {"path": "pump", "family": "knapsack", "count": rng.randint(2, 48), "rows": _log(rng, 700, 20_000),
                    "iters": rng.choice([32, 64]), "precision": "fp32"}
        quad = rng.random() < 0.5
        return {"path": "resolve", "family": "knapsack" if quad else "general", "count": rng.randint(1, 12) if quad else 1,
                "rows": _log(rng, 1_000, 8_000 if quad else 250_000), "iters": 64, "precision": prec, "quadratic": quad}
    return {"path": "round", "family": "knapsack", "count": rng.randint(1, 24), "rows": _log(rng, 100, 2_000),
            "fix": rng.choice([4, 16, 64]), "precision": "fp32"}


# --------------------------------------------------- LPs, drawn on the GPU
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _rand(g, n):
    return torch.rand(int(n), generator=g, device=DEV, dtype=torch.float64)


def _randint(g, lo, hi, n):
    return torch.randint(lo, hi, (int(n),), generator=g, device=DEV)


class _System:
    """LPs side by side: one block-diagonal matrix sorted by rows, on the GPU."""

    def __init__(self, ms, ns, row, col, val, c, b, sense, l, u):
        self.ms, self.ns = ms, ns
        self.roff, self.coff = np.concatenate([[0], np.cumsum(ms)]), np.concatenate([[0], np.cumsum(ns)])
        self.M, self.N = int(self.roff[-1]), int(self.coff[-1])
        self.row, self.col, self.val = row, col, val
        self.c, self.b, self.sense, self.l, self.u = c, b, sense, l, u

    def owners(self):
        """The LP of every row and of every column."""
        return (torch.repeat_interleave(torch.arange(len(self.ms), device=DEV), torch.tensor(self.ms, device=DEV)),
                torch.repeat_interleave(torch.arange(len(self.ns), device=DEV), torch.tensor(self.ns, device=DEV)))

    def lps(self):
        ptr = np.concatenate([[0], np.cumsum(torch.bincount(self.row, minlength=self.M).cpu().numpy())])
        col, val = self.col.cpu().numpy(), self.val.cpu().numpy()
        c, b, l, u = (t.cpu().numpy() for t in (self.c, self.b, self.l, self.u))
        sense = self.sense.cpu().numpy().astype(np.uint8)
        out = []
        for q in range(len(self.ms)):
            r0, r1, c0, c1 = (int(v) for v in (self.roff[q], self.roff[q + 1], self.coff[q], self.coff[q + 1]))
            e0, e1 = int(ptr[r0]), int(ptr[r1])
            out.append(instances.LP(
                m=r1 - r0, n=c1 - c0, row_ptr=ptr[r0:r1 + 1] - e0, col_idx=(col[e0:e1] - c0).astype(np.int32),
                val=val[e0:e1], c=c[c0:c1], b=b[r0:r1], senses=sense[r0:r1], l=l[c0:c1], u=u[c0:c1],
                is_int=np.ones(c1 - c0, dtype=np.uint8)))
        return out


def _row_counts(case):
    """Row counts spread evenly over the logarithm of the range, in mixed order."""
    lo, hi, count = case["rows"], case.get("rows_max", case["rows"]), case["count"]
    at = [((q + 1) * 0.6180339887498949) % 1.0 for q in range(count)]
    return [int(round(lo * (hi / lo) ** t)) for t in at]


def _by_rows(row, col, n):
    """Distinct (row, column) pairs sorted by row, then column."""
    key = torch.unique(row * n + col)
    return key // n, key % n


def _covering(case, g):
    """Covering rows, or covering and knapsack rows mixed: every column hits
    3 to 8 rows; binary variables."""
    ms = _row_counts(case)
    cover = case["family"] == "cover"
    ns = [m * 5 // 2 if cover else 2 * m for m in ms]
    M, N = sum(ms), sum(ns)
    mt, nt = torch.tensor(ms, device=DEV), torch.tensor(ns, device=DEV)
    of_col = torch.repeat_interleave(torch.arange(len(ms), device=DEV), nt)
    roff = torch.cumsum(mt, 0) - mt
    deg = _randint(g, 3, 9, N)
    col = torch.repeat_interleave(torch.arange(N, device=DEV), deg)
    own = of_col[col]
    row = roff[own] + torch.minimum((_rand(g, col.numel()) * mt[own]).long(), mt[own] - 1)
    if cover:  # no covering row without a column
        coff = torch.cumsum(nt, 0) - nt
        of_row = torch.repeat_interleave(torch.arange(len(ms), device=DEV), mt)
        extra = coff[of_row] + torch.minimum((_rand(g, M) * nt[of_row]).long(), nt[of_row] - 1)
        empty = torch.bincount(row, minlength=M) == 0
        row = torch.cat([row, torch.arange(M, device=DEV)[empty]])
        col = torch.cat([col, extra[empty]])
    row, col = _by_rows(row, col, N)
    covers = torch.ones(M, dtype=torch.bool, device=DEV) if cover else \
        (_rand(g, M) < 0.5) & (torch.bincount(row, minlength=M) >= 4)
    val = torch.where(covers[row], 1.0, _randint(g, 1, 101, row.numel()).double())
    total = torch.zeros(M, dtype=torch.float64, device=DEV).index_add_(0, row, val)
    b = torch.where(covers, 1.0, 0.3 * total)
    sense = torch.where(covers, ord("G"), ord("L"))
    c = _randint(g, 1, 101, N).double()
    zero = torch.zeros(N, dtype=torch.float64, device=DEV)
    return _System(ms, ns, row, col, val, c, b, sense, zero, zero + 1.0)


def _general(case, g):
    """Mixed rows over uniform columns: geometric row lengths of mean 10 with
    integers up to 20, or power-law lengths with 70 % pattern rows and
    integers up to 127 otherwise."""
    m = case["rows"]
    n = 2 * m
    skewed = case["family"] == "skewed"
    if skewed:
        kmax = min(50_000, max(16, m // 10))
        p = torch.arange(1, kmax + 1, device=DEV, dtype=torch.float64) ** -1.8
        raw = (torch.multinomial(p, m, replacement=True, generator=g) + 1).double()
        lens = torch.clamp((raw * (40.0 * m / raw.sum())).floor(), 1, min(kmax, n // 2)).long()
    else:
        lens = torch.clamp((torch.log1p(-_rand(g, m)) / math.log1p(-0.1)).ceil().long(), 1, n // 2)
    row = torch.repeat_interleave(torch.arange(m, device=DEV), lens)
    row, col = _by_rows(row, _randint(g, 0, n, row.numel()), n)
    top = 127 if skewed else 20
    val = _randint(g, 1, top + 1, row.numel()).double()
    val = torch.where(_rand(g, row.numel()) < 0.5, -val, val)
    if skewed:
        val = torch.where((_rand(g, m) < 0.7)[row], 1.0, val)
    code = _randint(g, 0, 3, n)
    u = torch.where(code == 0, 1.0, torch.where(code == 1, 10.0, math.inf)).double()
    x = _rand(g, n) * torch.clamp(u, max=10.0)
    r = _rand(g, m)
    if skewed:
        sense = torch.where(r < 0.4, ord("G"), torch.where(r < 0.8, ord("L"), ord("E")))
    else:
        sense = torch.where(r < 0.2, ord("E"), ord("G"))
    slack = -torch.log1p(-_rand(g, m))
    # row sums on the host, in order: the same seed gives the same bits
    ptr = np.concatenate([[0], np.cumsum(torch.bincount(row, minlength=m).cpu().numpy())])
    b = torch.from_numpy(np.add.reduceat((val * x[col]).cpu().numpy(), ptr[:-1])).to(DEV)
    b = b + torch.where(sense == ord("G"), -slack, torch.where(sense == ord("L"), slack, 0.0))
    c = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    c = torch.where(torch.isinf(u), c.abs(), c)
    return _System([m], [n], row, col, val, c, b, sense, torch.zeros_like(u), u)


def _system(case, seed):
    g = _gen(seed)
    return (_covering if case["family"] in ("cover", "knapsack") else _general)(case, g), g


def _start(s, g):
    """A primal-dual pair inside the bounds and cones, as an earlier solve leaves it."""
    x0 = s.l + _rand(g, s.N) * torch.clamp(s.u - s.l, max=10.0)
    y0 = _rand(g, s.M)
    y0 = torch.where(s.sense == ord("L"), -y0, torch.where(s.sense == ord("E"), y0 - 0.5, y0))
    return x0, y0, np.exp(0.2 * np.arange(len(s.ms)) % 1.0 - 0.5)


def _pump_update(s, g):
    """Rounding (True: at the upper bound) and blend weights of a pump round."""
    up = _rand(g, s.N) < 0.3
    a = 0.81
    kappa = [math.sqrt(n) / max(1e-30, float(torch.linalg.vector_norm(s.c[s.coff[q]:s.coff[q + 1]])))
             for q, n in enumerate(s.ns)]
    return up, a, kappa


# -------------------------------------------------------- state and pass
class _DeviceArray:
    """A device buffer of a handle, for torch.as_tensor without a copy; the
    tensor keeps this object and so the handle that owns the memory."""

    def __init__(self, owner, ptr, n, typestr):
        self.owner = owner
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": typestr, "data": (ptr, False), "version": 3,
                                         "strides": None}


def prepare(case, seed):
    s, g = _system(case, seed)
    lps = s.lps()
    path = case["path"]
    if path == "oneshot":
        return {"case": case, "lp": lps[0]}
    st = {"case": case}
    if path in ("pump", "resolve"):
        st["x0"], st["y0"], st["omega0"] = _start(s, g)
    if path == "pump":
        up, st["a"], st["kappa"] = _pump_update(s, g)
        up = up.cpu().numpy()
        st["up"] = [up[s.coff[q]:s.coff[q + 1]] for q in range(len(lps))]
    if path == "resolve":
        c, qd = _new_objective(case, s, g)
        c, qd = c.cpu().numpy(), None if qd is None else qd.cpu().numpy()
        st["c"] = [c[s.coff[q]:s.coff[q + 1]] for q in range(len(lps))]
        st["q"] = None if qd is None else [qd[s.coff[q]:s.coff[q + 1]] for q in range(len(lps))]
    if path == "round":
        st["xbar"] = _reference(s, g).cpu().numpy()
    b = st["batch"] = pdhg.Batch(lps, precision=pdhg.FP32 if case["precision"] == "fp32" else pdhg.FP64)
    if path == "round":
        b.fix_propagate(K=case["fix"], xbar=st["xbar"])  # device copies are made by the first call
        return st
    # the first solve chooses layouts; a program that keeps the handle has had it
    b.solve(tol=TOL_CUT, iter_limit=1, **_options(case))
    xp, yp, size = b.device_iterates()
    kind = "<f%d" % size
    st["x"] = torch.as_tensor(_DeviceArray(b, xp, s.N, kind), device=DEV)
    st["y"] = torch.as_tensor(_DeviceArray(b, yp, s.M, kind), device=DEV)
    torch.cuda.synchronize()
    return st


def _options(case):
    return {"adaptive": int(case.get("adaptive", False)), "restart_avg": int(case.get("average", False))}


def _new_objective(case, s, g):
    if case["quadratic"]:  # distance to a rounding: 2 (1 - a) (x^2 / 2 - xhat x), blended with c
        up, a, kappa = _pump_update(s, g)
        scale = torch.repeat_interleave(torch.tensor(kappa, device=DEV, dtype=torch.float64),
                                        torch.tensor(s.ns, device=DEV))
        return a * scale * s.c - 2.0 * (1.0 - a) * up.double(), torch.full_like(s.c, 2.0 * (1.0 - a))
    return s.c * (0.5 + _rand(g, s.N)), None


def _reference(s, g):
    """Values like a relaxation's: most near a bound, some fractional."""
    x = _rand(g, s.N)
    return torch.where(_rand(g, s.N) < 0.7, (x < 0.3).double(), x)


def run(state):
    case = state["case"]
    path = case["path"]
    if path == "oneshot":
        fp32 = case["precision"] == "fp32"
        r = pdhg.solve(state["lp"], tol=TOL_CUT, iter_limit=case["iters"], precision=pdhg.FP32 if fp32 else pdhg.FP64)
        # FP32 iterates are handed over in FP64 arrays
        return [v.astype(np.float32) if fp32 else v for v in (r.x, r.y)] + [r.result["iterations"]]
    b = state["batch"]
    if path == "round":
        xhat, feasible, ignored, mask = b.fix_propagate(K=case["fix"], xbar=state["xbar"])
        return [xhat, feasible, ignored, mask]
    if path == "tolerance":
        r = b.solve(tol=1e-4, iter_limit=100_000)
        return [state["x"], state["y"], r[0]["iterations"]]
    if path == "solve":
        r = b.solve(tol=TOL_CUT, iter_limit=case["iters"], **_options(case))
        return [state["x"], state["y"], np.array([v["iterations"] for v in r])]
    if path == "pump":
        for q in range(case["count"]):
            b.set_blend(q, state["up"][q], state["a"], state["kappa"][q])
    else:
        for q in range(case["count"]):
            b.set_objective(q, state["c"][q])
            if state["q"] is not None:
                b.set_quadratic(q, state["q"][q])
    b.set_start_device(state["x0"].data_ptr(), state["y0"].data_ptr(), omega0=state["omega0"])
    b.solve(warm=True, tol=TOL_CUT, iter_limit=case["iters"])
    if path == "pump":
        return [state["x"], state["y"], b.mip_feasible()]
    return [state["x"], state["y"]]


def work(case):
    """Per iteration every nonzero twice (index and value; the two products
    depend on each other), the vectors of both steps once, one multiplication
    and addition a nonzero and product."""
    lo, hi = case["rows"], case.get("rows_max", case["rows"])
    mean = lo if hi == lo else (hi - lo) / math.log(hi / lo)
    m = mean * case["count"]
    n, per_row = {"cover": (2.5 * m, 13.75), "knapsack": (2 * m, 11.0), "general": (2 * m, 10.0),
                  "skewed": (2 * m, 40.0)}[case["family"]]
    nnz = per_row * m
    if case["path"] == "round":
        return {"bytes": 12 * nnz + 24 * n + 10 * m, "flops": 4 * nnz}
    entry, v = (4, 4) if case["precision"] == "fp32" else (12, 8)
    iters = case.get("iters", 4_000)
    per_iter = 2 * entry * nnz + (4 * v + 5) * m + (8 * v + 4) * n
    once = 12 * nnz + 40 * n + 17 * m if case["path"] == "oneshot" else 0
    return {"bytes": iters * per_iter + once, "flops": iters * (4 * nnz + 10 * (m + n))}


# ------------------------------------------------------------ plain FP64
def _mv(out_len, out, idx, val, x):
    return torch.zeros(out_len, dtype=torch.float64, device=DEV).index_add_(0, out, val * x[idx])


def _pdhg64(s, iters, tol, c=None, qd=None, start=None, adaptive=False, average=False, period=64):
    """PDHG with diagonal preconditioning and KKT restarts, LP by LP, in FP64
    torch operations over all LPs side by side; all run to `iters`, or one
    LP to `tol`.  Returns x, y, iterations."""
    row, col, val, M, N = s.row, s.col, s.val, s.M, s.N
    ri, ci = s.owners()
    count = len(s.ms)
    c = s.c if c is None else c
    qd = torch.zeros_like(c) if qd is None else qd

    def per(owner, v):
        return torch.zeros(count, dtype=torch.float64, device=DEV).index_add_(0, owner, v)

    def ax(x):
        return _mv(M, row, col, val, x)

    def aty(y):
        return _mv(N, col, row, val, y)

    dr, dc = torch.ones(M, dtype=torch.float64, device=DEV), torch.ones(N, dtype=torch.float64, device=DEV)
    for it in range(11):  # ten rounds of row and column maxima, one of sums
        a = (dr[row] * val * dc[col]).abs()
        how = "amax" if it < 10 else "sum"
        r = torch.zeros_like(dr).scatter_reduce_(0, row, a, how)
        k = torch.zeros_like(dc).scatter_reduce_(0, col, a, how)
        dr = torch.where(r > 0, dr / torch.sqrt(r), dr)
        dc = torch.where(k > 0, dc / torch.sqrt(k), dc)
    dr2, dc2 = dr * dr, dc * dc
    bnorm, cnorm = torch.sqrt(per(ri, s.b * s.b)), torch.sqrt(per(ci, c * c))
    bs, cs = torch.sqrt(per(ri, (dr * s.b) ** 2)), torch.sqrt(per(ci, (dc * c) ** 2))
    omega = torch.where((cs > 0) & (bs > 0), cs / bs, 1.0)
    ge, le = s.sense == ord("G"), s.sense == ord("L")
    lf, uf = torch.isfinite(s.l), torch.isfinite(s.u)
    lz, uz = torch.where(lf, s.l, 0.0), torch.where(uf, s.u, 0.0)

    def cone(y):
        return torch.where(ge, y.clamp(min=0), torch.where(le, y.clamp(max=0), y))

    x, y = torch.zeros_like(c), torch.zeros_like(s.b)
    if start is not None:
        x, y = start[0].clone(), start[1].clone()
        omega = torch.tensor(start[2], dtype=torch.float64, device=DEV)
    x, y = torch.minimum(torch.maximum(x, s.l), s.u), cone(y)
    eta = torch.full((count,), 0.99, dtype=torch.float64, device=DEV)

    def kkt(x, y):
        r = s.b - ax(x)
        r = torch.where(ge, r.clamp(min=0), torch.where(le, (-r).clamp(min=0), r))
        qx = qd * x
        g = c + qx - aty(y)
        lam = torch.where(lf & uf, g, torch.where(lf, g.clamp(min=0), torch.where(uf, g.clamp(max=0), 0.0)))
        p = per(ci, c * x + 0.5 * qx * x)
        d = per(ri, s.b * y) + per(ci, lz * lam.clamp(min=0) + uz * lam.clamp(max=0) - 0.5 * qx * x)
        return torch.maximum(torch.maximum(torch.sqrt(per(ri, r * r)) / (1 + bnorm),
                                           torch.sqrt(per(ci, (g - lam) ** 2)) / (1 + cnorm)),
                             (p - d).abs() / (1 + p.abs() + d.abs()))

    k, kr = 0, torch.zeros(count, dtype=torch.int64, device=DEV)
    er = ep = torch.zeros(count, dtype=torch.float64, device=DEV)
    xr, yr = x, y
    xa, ya, na = x, y, torch.zeros(count, dtype=torch.float64, device=DEV)
    while True:
        e, cx, cy = kkt(x, y), x, y
        if average and k:
            ea = kkt(xa, ya)
            use = (k > kr) & (ea < e)
            e = torch.where(use, ea, e)
            cx, cy = torch.where(use[ci], xa, x), torch.where(use[ri], ya, y)
        if k >= iters or (tol > 0 and bool((e <= tol).all())):
            return cx, cy, k
        if k == 0:
            er = e
        else:
            fire = (e <= 0.2 * er) | ((e <= 0.8 * er) & (e > ep)) | ((k - kr) >= 0.36 * k)
            dx = torch.sqrt(per(ci, ((cx - xr) / dc) ** 2))
            dy = torch.sqrt(per(ri, ((cy - yr) / dr) ** 2))
            move = fire & (dx > 1e-10) & (dy > 1e-10)
            omega = torch.where(move, torch.exp(0.5 * torch.log(dy / dx) + 0.5 * torch.log(omega)), omega)
            er, kr = torch.where(fire, e, er), torch.where(fire, k, kr)
            x, y = torch.where(fire[ci], cx, x), torch.where(fire[ri], cy, y)
            xr, yr = torch.where(fire[ci], x, xr), torch.where(fire[ri], y, yr)
            na = torch.where(fire, 0.0, na)
        ep = e
        for _ in range(min(period, iters - k)):
            t, sg = (eta / omega)[ci], (eta * omega)[ri]
            xn = (x + t * dc2 * (aty(y) - c)) / (1 + t * dc2 * qd)
            xn = torch.minimum(torch.maximum(xn, s.l), s.u)
            yn = cone(y + sg * dr2 * (s.b - ax(2 * xn - x)))
            k += 1
            if adaptive:
                dx, dy = xn - x, yn - y
                nx, ny = per(ci, dx * dx / dc2), per(ri, dy * dy / dr2)
                inter = per(ri, dy * ax(dx)).abs()
                grow = (1 + (k + 1.0) ** -0.6) * eta
                shrink = (1 - (k + 1.0) ** -0.3) * (omega * nx + ny / omega) / (2 * inter)
                new = torch.where(inter > 0, torch.minimum(shrink, grow), grow)
                eta = torch.where(nx + ny > 0, new, eta)
            x, y = xn, yn
            if average:
                na = na + 1
                xa = torch.where((na == 1)[ci], x, xa + (x - xa) / na[ci])
                ya = torch.where((na == 1)[ri], y, ya + (y - ya) / na[ri])


def exact(case, seed):
    path = case["path"]
    if path == "round":
        return None  # whole numbers and flags
    s, g = _system(case, seed)
    if path == "oneshot":
        x, y, k = _pdhg64(s, case["iters"], 0.0)
        return [x.cpu().numpy(), y.cpu().numpy(), None]
    if path == "tolerance":
        x, y, k = _pdhg64(s, 100_000, 1e-4)
        return [x, y, None]
    if path == "solve":
        x, y, k = _pdhg64(s, case["iters"], 0.0, adaptive=case["adaptive"], average=case["average"])
        return [x, y, None]
    start = _start(s, g)
    if path == "pump":
        up, a, kappa = _pump_update(s, g)
        scale = torch.repeat_interleave(torch.tensor(kappa, device=DEV, dtype=torch.float64),
                                        torch.tensor(s.ns, device=DEV))
        c, qd = a * scale * s.c + (1.0 - a) * torch.where(up, -1.0, 1.0), None
    else:
        c, qd = _new_objective(case, s, g)
    x, y, k = _pdhg64(s, case["iters"], 0.0, c=c, qd=qd, start=start)
    return [x, y, None] if path == "pump" else [x, y]
