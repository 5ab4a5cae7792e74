"""The work that users of this library have it do, as measurable cases.

Single solves through `binding` (arrowhead, Hermitian arrowhead, DPR1, SVD of a triangular
arrowhead, symmetric tridiagonal) and batched plans through `batch`, from the smallest orders,
where a call is a handful of launches, to V of 2 GiB and the 10,000-problem plan.  Inputs follow
the laws of `workloads`; a case is a dict of plain values:

  entry    arrow | herm | dpr1 | svd | tridiag | batch
  law      arrow: uniform | graded | reducible
  n        order (single problems);  count, nmin, nmax: problems of a batch, n log-uniform
  order    sorted | reversed | shuffled: how the caller presents the poles
  vectors  False: eigenvalues (and their exact shift + mu pairs) only
  neg      dpr1: rho < 0
  mix      batch: "halves" arrowhead and DPR1 in turn; "requests" 60% arrowhead, 25% DPR1, 15% SVD
  replay   batch: one captured plan run again and again; False: a new plan for each pass
"""
import math

import numpy as np
import torch

from paper_1302_7203_amd import batch, binding
from paper_1302_7203_amd import workloads as W

EXACT_N = 4200          # largest order whose reference fits the time a check may take
EXACT_WORK = 40_000_000  # ... and largest sum of n^2 over a batch


def listed():
    return [
        # the smallest calls: one step of an update or a filter, where latency and launches count
        {"name": "arrow_64", "entry": "arrow", "law": "uniform", "n": 64, "order": "sorted", "vectors": True},
        # a rank-one update of a small spectrum, odd order, poles as they come
        {"name": "dpr1_199_shuffled", "entry": "dpr1", "n": 199, "order": "shuffled", "vectors": True, "neg": False},
        # the uniform single solve of the benchmark
        {"name": "arrow_512", "entry": "arrow", "law": "uniform", "n": 512, "order": "sorted", "vectors": True},
        # a column appended to a diagonalised matrix: values and both sets of vectors
        {"name": "svd_777", "entry": "svd", "n": 777, "order": "sorted", "vectors": True},
        # one state coupled to many levels: complex vectors, levels as they come
        {"name": "herm_1025_shuffled", "entry": "herm", "n": 1025, "order": "shuffled", "vectors": True},
        # repeated levels and uncoupled ones: deflated on the device
        {"name": "reducible_2047_shuffled", "entry": "arrow", "law": "reducible", "n": 2047, "order": "shuffled",
         "vectors": True},
        # spectra only, as exact (shift, mu) pairs
        {"name": "values_2048", "entry": "arrow", "law": "uniform", "n": 2048, "order": "sorted", "vectors": False},
        # the graded single solve of the benchmark: 20 decades, 64 tight clusters
        {"name": "graded_4096", "entry": "arrow", "law": "graded", "n": 4096, "order": "sorted", "vectors": True},
        # the largest single solve of the benchmark, V of 2 GiB
        {"name": "arrow_16384", "entry": "arrow", "law": "uniform", "n": 16384, "order": "sorted", "vectors": True},
        # divide and conquer with DPR1 merges
        {"name": "tridiag_1000", "entry": "tridiag", "n": 1000},
        # what a serving loop launches: the requests of one admission in a plan of their own
        {"name": "batch_requests_32", "entry": "batch", "mix": "requests", "count": 32, "nmin": 32, "nmax": 2048,
         "replay": False},
        # the 10,000-problem plan of the benchmark's headline
        {"name": "batch_mixed_10000", "entry": "batch", "mix": "halves", "count": 10000, "nmin": 16, "nmax": 1024,
         "replay": True},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    entry = rng.choices(["arrow", "dpr1", "svd", "herm", "tridiag", "batch"], [8, 5, 3, 2, 2, 4])[0]
    if entry == "tridiag":
        return {"entry": entry, "n": _log_uniform(rng, 64, 1500)}
    if entry == "batch":
        nmax = rng.choice([256, 1024, 2048])
        count = _log_uniform(rng, 8, 2000 if nmax < 2048 else 400)
        return {"entry": entry, "mix": rng.choice(["halves", "requests"]), "count": count, "nmin": 16, "nmax": nmax,
                "replay": rng.random() < 0.5}
    order = rng.choice(["sorted", "sorted", "shuffled", "reversed"])
    if entry == "arrow":
        law = rng.choice(["uniform", "uniform", "graded", "reducible"])
        return {"entry": entry, "law": law, "n": _log_uniform(rng, 16, 16384), "order": order,
                "vectors": rng.random() < 0.85}
    case = {"entry": entry, "n": _log_uniform(rng, 16, 8192), "order": order, "vectors": rng.random() < 0.9}
    if entry == "dpr1":
        case["neg"] = rng.random() < 0.3
    return case


# ---------------------------------------------------------------------------
# inputs

def _ordered(pr, order, rng):
    if order == "sorted":
        perm = np.argsort(-pr.d, kind="stable")
    elif order == "reversed":
        perm = np.argsort(pr.d, kind="stable")
    else:
        perm = rng.permutation(pr.d.size)
    return W.Problem(pr.kind, pr.n, pr.d[perm].copy(), pr.z[perm].copy(), pr.scalar)


def _problem(case, seed):
    rng = np.random.default_rng([seed, 11])
    n, entry = case["n"], case["entry"]
    if entry == "arrow":
        if case["law"] == "graded":
            pr = W.graded_arrow(n, rng)
        elif case["law"] == "reducible":
            pr = W.reducible_arrow(n, rng)
        elif n >= 8192:
            pr = W.uniform_arrow(n, rng, -1e4, 1e4)
        else:
            pr = W.uniform_arrow(n, rng)
    elif entry == "herm":
        pr = W.herm_arrow(n, rng)
    elif entry == "dpr1":
        pr = W.dpr1(n, rng)
        if case["neg"]:
            pr.scalar = -pr.scalar
    else:
        pr = W.svd_arrow(n, rng)
    return _ordered(pr, case["order"], rng)


def _tridiagonal(case, seed):
    rng = np.random.default_rng([seed, 12])
    return rng.uniform(-1.0, 1.0, case["n"]), rng.uniform(-1.0, 1.0, case["n"] - 1)


def _batch_problems(case, seed):
    """The batch's orders and kinds are the case's own, its values the seed's."""
    sizes = np.random.default_rng([case["count"], case["nmax"], 14])
    rng = np.random.default_rng([seed, 13])
    out = []
    for p in range(case["count"]):
        n = int(round(math.exp(sizes.uniform(math.log(case["nmin"]), math.log(case["nmax"])))))
        u = (p % 2) * 0.7 if case["mix"] == "halves" else sizes.uniform()
        out.append(W.uniform_arrow(n, rng) if u < 0.60 else W.dpr1(n, rng) if u < 0.85 else W.svd_arrow(n, rng))
    return out


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    if case["entry"] == "tridiag":
        a, b = _tridiagonal(case, seed)
        return {"entry": "tridiag", "a": torch.from_numpy(a).to(dev), "b": torch.from_numpy(b).to(dev)}
    if case["entry"] == "batch":
        packed = batch.pack(_batch_problems(case, seed))
        pools = {"packed": packed, "in_pool": torch.from_numpy(packed.in_host).to(dev),
                 "out_pool": torch.empty(packed.out_size, dtype=torch.float64, device=dev),
                 "info_pool": torch.empty(packed.info_size, dtype=torch.int32, device=dev)}
        if case["replay"]:
            return {"entry": "batch", "plan": batch.Batch([], device=dev, graph=True, **pools), **pools}
        # as the serving loop: workspace from memory that the program already holds
        pools["workspace"] = torch.empty(batch.workspace_size(packed), dtype=torch.uint8, device=dev)
        return {"entry": "batch", "plan": None, "device": dev, **pools}
    pr = _problem(case, seed)
    return {"entry": case["entry"], "d": torch.from_numpy(pr.d).to(dev), "z": torch.from_numpy(pr.z).to(dev),
            "scalar": float(pr.scalar), "vectors": case["vectors"]}


# ---------------------------------------------------------------------------
# one pass

def run(state):
    entry = state["entry"]
    if entry == "tridiag":
        out = binding.tridiag_eig(state["a"], state["b"])
        return {"lam": out.lam, "V": out.V}
    if entry == "batch":
        if state["plan"] is not None:
            state["plan"].run()
        else:
            plan = batch.Batch([], device=state["device"], packed=state["packed"], in_pool=state["in_pool"],
                               out_pool=state["out_pool"], info_pool=state["info_pool"],
                               workspace=state["workspace"])
            plan.run()
            plan.close()
        return {"out": state["out_pool"], "info": state["info_pool"]}
    d, z, scalar, vectors = state["d"], state["z"], state["scalar"], state["vectors"]
    if entry == "arrow":
        out = binding.arrow_eig(d, z, scalar, vectors=vectors, pairs=not vectors)
    elif entry == "herm":
        out = binding.arrow_eig_herm(d, z, scalar, vectors=vectors, pairs=not vectors)
    elif entry == "dpr1":
        out = binding.dpr1_eig(d, z, scalar, vectors=vectors)
    else:
        out = binding.arrow_svd(d, z, scalar, vectors=vectors)
    got = {"lam": out.lam, "V": out.V, "U": out.U, "shift": out.shift, "mu": out.mu, "info": out.info}
    return {k: v for k, v in got.items() if v is not None}


# ---------------------------------------------------------------------------
# what a pass cannot do without: inputs read once, outputs written once, and per eigenpair and
# pole 40 operations for b in doubled precision, 8 for the shift and its bracket, 3 for each of
# two root-finding passes and 4 for the vector entry

def _single_work(entry, n, vectors):
    cplx = entry == "herm"
    mats = (2 if entry == "svd" or cplx else 1) if vectors else 0
    return {"bytes": (24.0 if cplx else 16.0) * n + 12.0 * n + 8.0 * mats * n * n,
            "flops": (54.0 + (4.0 * mats if vectors else 0.0)) * n * n}


def work(case):
    if case["entry"] == "tridiag":
        n = float(case["n"])
        return {"bytes": 24.0 * n + 8.0 * n * n, "flops": 4.0 / 3.0 * n ** 3}
    if case["entry"] == "batch":
        total = {"bytes": 0.0, "flops": 0.0}
        for pr in _batch_problems(case, 0):
            w = _single_work("svd" if pr.kind == W.KIND_SVD else "arrow", pr.n, True)
            total = {k: total[k] + w[k] for k in total}
        return total
    return _single_work(case["entry"], case["n"], case["vectors"])


# ---------------------------------------------------------------------------
# reference: every zero of the secular function in the variable shifted to its nearer pole,
# bisected in float64 and finished by Newton steps in numpy's longdouble

def _zeros(pole, diff, c, corner, kappa):
    """Zeros of g = (corner - p_i) - kappa t - sum_j c_j / (e_ji - t), t = lambda - p_i, for poles
    p_0 > p_1 > ...: (i, t) per zero, descending.  kappa = 0: corner is the whole constant."""
    LD = np.longdouble
    m = pole.size
    k = np.arange(m + 1 if kappa else m)
    below = np.minimum(k, m - 1)                 # pole under the zero (the last: none under it)
    above = np.maximum(k - 1, 0)
    inner = (k > 0) & (k < m)
    e64 = diff(np.arange(m)[None, :], below[:, None]).astype(np.float64)   # e_j seen from the pole below
    c64 = torch.from_numpy(c.astype(np.float64))
    const = (corner - pole if kappa else np.full(m, corner, dtype=LD))

    def g(e, a, t):
        return a - kappa * t - (c64[None, :] / (e - t[:, None])).sum(1)

    gap = diff(above, below)
    e = torch.from_numpy(e64)
    half = torch.from_numpy(np.where(inner, 0.5 * gap, 1.0).astype(np.float64))
    right = (g(e, torch.from_numpy(const[below].astype(np.float64)), half) < 0).numpy()
    side = np.where(k == 0, 1, np.where(k == m, -1, np.where(right, 1, -1)))
    i = np.where(side > 0, below, above)
    i = np.where(k == m, m - 1, i)
    a = const[i]
    total = c.sum()
    if kappa:
        root = np.abs(a) + np.sqrt(a * a + 4 * total)   # t^2 - side a t - total = 0
        outer = np.where(side * a > 0, root / 2, 2 * total / root)
    else:
        outer = np.full(k.size, total / -corner, dtype=LD)
    hi = np.where(inner, 0.5 * gap, outer) * (1 + LD(1e-6))
    del e64, e
    e = torch.from_numpy(diff(np.arange(m)[None, :], i[:, None]).astype(np.float64))
    a64, s64 = torch.from_numpy(a.astype(np.float64)), torch.from_numpy(side.astype(np.float64))
    hi = torch.from_numpy(hi.astype(np.float64))
    lo = hi * 1e-50
    for _ in range(64):
        mid = torch.where(hi > 4 * lo, torch.sqrt(lo) * torch.sqrt(hi), 0.5 * (lo + hi))
        up = s64 * g(e, a64, s64 * mid) > 0
        lo, hi = torch.where(up, mid, lo), torch.where(up, hi, mid)
    del e
    t = (s64 * 0.5 * (lo + hi)).numpy().astype(LD)
    step = max(1, 4_000_000 // m)
    for at in range(0, k.size, step):
        s = slice(at, at + step)
        E = diff(np.arange(m)[None, :], i[s, None])
        for _ in range(80):   # two or three; more, kept to a factor 8 each, where the constant cancels the sum
            r = 1 / (E - t[s, None])
            w = c[None, :] * r
            move = (a[s] - kappa * t[s] - w.sum(1)) / (kappa + (w * r).sum(1))
            t[s] *= np.clip(1 + move / t[s], LD(0.125), LD(8))
            if np.all(np.abs(move) <= 1e-12 * np.abs(t[s])):
                break
    return i, t


def _solve(entry, d, z, scalar):
    """(lam, V, U) of an irreducible problem in longdouble, rounded to float64."""
    LD = np.longdouble
    order = np.argsort(-(np.abs(d) if entry == "svd" else d), kind="stable")
    dl = d.astype(LD)
    neg = entry == "dpr1" and scalar < 0
    if neg:
        order, dl, scalar = order[::-1], -dl, -scalar
    p, zl = dl[order], (z[order].astype(np.clongdouble) if entry == "herm" else z[order].astype(LD))
    alpha = LD(scalar)
    if entry == "svd":
        diff = lambda j, i: (p[j] - p[i]) * (p[j] + p[i])   # noqa: E731
        pole, num, corner, kappa = p * p, p * zl, alpha * alpha + (zl * zl).sum(), 1
        c = num * num
    else:
        diff = lambda j, i: p[j] - p[i]   # noqa: E731
        pole, num = p, zl
        c = (zl * zl.conj()).real
        corner, kappa = (-1 / alpha, 0) if entry == "dpr1" else (alpha, 1)
    i, t = _zeros(pole, diff, c, corner, kappa)
    lam = pole[i] + t
    n, m = t.size, p.size
    V = np.empty((n, n), dtype=np.complex128 if entry == "herm" else np.float64)
    U = np.empty((n, n)) if entry == "svd" else None
    sigma = np.sqrt(np.maximum(lam, 0)) if entry == "svd" else None
    step = max(1, 4_000_000 // m)
    for at in range(0, n, step):
        s = slice(at, at + step)
        X = num[None, :] / (diff(np.arange(m)[None, :], i[s, None]) - t[s, None])
        norm = np.sqrt((X * X.conj()).real.sum(1) + kappa)
        X = X / (-norm if neg else norm)[:, None]
        V[order[:, None], np.arange(n)[None, s]] = X.T
        if kappa:
            V[n - 1, s] = -1 / norm
        if U is not None:
            U[order[:, None], np.arange(n)[None, s]] = (sigma[s, None] * X / p[None, :]).T
            U[n - 1, s] = -alpha / norm / sigma[s]
    lam = sigma if entry == "svd" else lam
    if neg:
        lam, V = -lam[::-1], V[:, ::-1]
    return lam.astype(np.float64), V, U


def exact(case, seed):
    if case["entry"] == "tridiag":
        # the vectors' signs are the merges' own: values only
        a, b = _tridiagonal(case, seed)
        lam = np.linalg.eigvalsh(np.diag(a) + np.diag(b, 1) + np.diag(b, -1))[::-1].copy()
        return {"lam": lam, "V": None}
    if case["entry"] == "batch":
        probs = _batch_problems(case, seed)
        if sum(pr.n * pr.n for pr in probs) > EXACT_WORK:
            return None
        out = []
        for pr in probs:   # in the pools' order: values, vectors, left vectors
            kind = {W.KIND_ARROW: "arrow", W.KIND_DPR1: "dpr1", W.KIND_SVD: "svd"}[pr.kind]
            lam, V, U = _solve(kind, pr.d, pr.z, pr.scalar)
            out += [lam, V.T.reshape(-1)] + ([U.T.reshape(-1)] if U is not None else [])
        return {"out": np.concatenate(out), "info": None}
    if case["n"] > EXACT_N or case.get("law") == "reducible":
        return None
    pr = _problem(case, seed)
    lam, V, U = _solve(case["entry"], pr.d, pr.z, pr.scalar)
    if not case["vectors"]:
        return {"lam": lam}
    return {"lam": lam, "V": V, "U": U} if U is not None else {"lam": lam, "V": V}
