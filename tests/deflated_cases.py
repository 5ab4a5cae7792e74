"""Reducible arrowheads with a row of zero shaft whose pole lies between the first pass's value of
an ill-conditioned eigenvalue and its final value: the deflated pair's column has to follow from
the final one."""
import numpy as np

from paper_1302_7203_amd import workloads as W


def _with_rows(d, z, alpha, poles):
    d = np.concatenate([d, poles])
    z = np.concatenate([z, np.zeros(len(poles))])
    return W.Problem(W.KIND_ARROW, d.size + 1, d, z, alpha)


def cases():
    """(name, problem) pairs."""
    out = []
    tight = np.array([1.0 + 2.0 ** -52, 1.0, -3.0])
    # first pass 13.238, final 5.5559
    for v in (5.56, 9.397, 13.2):
        out.append((f"pole pair, {v}", _with_rows(tight, np.ones(3), 5.0, [v])))
    out.append(("pole pair, three rows", _with_rows(tight, np.ones(3), 5.0, [6.0, 9.397, 12.0])))
    near = np.array([1.0 + 1e-12, 1.0, -3.0])
    out.append(("pole gap 1e-12", _with_rows(near, np.ones(3), 5.0, [5.55593])))
    # eigenvalue 29 of the reduced problem: 0.2496 after the first pass, 0.8765 in the end
    rng = np.random.default_rng(0)
    pr = W.graded_arrow(100, rng, clusters=8)
    pr.z[rng.choice(99, 20, replace=False)] = 0.0
    for rows in ([0.81], [0.3, 0.5, 0.7, 0.87], []):
        out.append((f"graded 100, rows {rows}", _with_rows(pr.d, pr.z, pr.scalar, rows)))
    for n in (300, 600, 1000, 1279):
        rng = np.random.default_rng(n)
        pr = W.graded_arrow(n - 24, rng, clusters=max(8, n // 14))
        pr.z[rng.choice(n - 25, n // 5, replace=False)] = 0.0
        out.append((f"graded {n}", pr))
    return out


def between(pr, first, final, most=24):
    """`pr` with up to `most` more rows of zero shaft, their poles halfway between the two values
    of the eigenvalues that moved furthest (first, final: descending-index arrays of the reduced
    problem's eigenvalues)."""
    rel = np.abs(first - final) / np.abs(final)
    ks = np.argsort(-rel)[:most]
    poles = [0.5 * (first[k] + final[k]) for k in ks if rel[k] > 1e-12]
    poles = [v for v in dict.fromkeys(poles) if np.all(np.abs(pr.d - v) > 0)]
    return _with_rows(pr.d, pr.z, pr.scalar, poles)
