"""GPU: rounding of the FP64 operator's sums over many source chunks.

A smooth density on a sphere: nearly all terms of a row have one sign, so that every addition rounds at
the size of the sum and the order of the additions shows. Reference: the literal formulas and their
sums in extended precision. Bar: the same terms rounded to FP64 and added the plain way, 512 one after the
other to a chunk and then chunk after chunk; the operator may be no further from the reference than that, in
each half of the vector, over the sampled rows.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LD = np.longdouble
H, KAPPA, TAU, EPS_OUT = 0.5, 0.1257, 0.5, 80.0


def _sphere(n):
    """n points of a spiral on a sphere with the density of a band's projections (4/h² an Å²)."""
    k = np.arange(n) + 0.5
    z, a = 1.0 - 2.0 * k / n, k * np.pi * (3.0 - np.sqrt(5.0))
    s = np.sqrt(1.0 - z * z)
    nv = np.stack([s * np.cos(a), s * np.sin(a), z], 1)
    return np.sqrt(n * H * H / (16.0 * np.pi)) * nv, nv


def _row_terms(x, nv, p, i):
    """The terms of row i of both halves, without the diagonal, in extended precision."""
    n, pi, th, kap, tau = len(x), LD("3.14159265358979323846264338327950288"), LD(EPS_OUT), LD(KAPPA), LD(TAU)
    d = x[i] - x
    r2 = (d * d).sum(1)
    di, dj, nn = d @ nv[i], (d * nv).sum(1), nv @ nv[i]
    reg = (r2 - di * di < tau * tau) & (r2 < 4 * tau * tau)
    r = np.sqrt(np.where(reg, LD(1), r2))
    z = kap * r
    e = np.exp(-z)
    a, b = e * (1 + z), e * (3 + 3 * z + z * z)
    kbar = 4 * pi * (np.exp(-kap * tau) - 1 + kap * tau) / (2 * pi * kap * tau * tau)
    zero = LD(0)
    k11 = np.where(reg, zero, dj * (1 - th * a) / r ** 3)
    k12 = np.where(reg, kbar, (1 - e) / r)
    k21 = np.where(reg, zero, nn * (1 - a) / r ** 3 - di * dj * (3 - b) / r ** 5)
    k22 = np.where(reg, zero, -di * (1 - a / th) / r ** 3)
    w = LD(H) ** 3 / (4 * pi)
    return w * (k11 * p[:n] - k12 * p[n:]), w * (k21 * p[:n] - k22 * p[n:])


def _plain(t):
    """FP64 sum: chunks of 512 one term after the other, the chunks one after the other."""
    t = t.astype(np.float64)
    t = np.append(t, np.zeros(-len(t) % 512)).reshape(-1, 512)
    return np.cumsum(np.cumsum(t, axis=1)[:, -1])[-1]


@pytest.mark.parametrize("n", [12300, 45818, 61439])
def test_operator_is_no_worse_than_plain_sums(n):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    print("case: FP64 sums, n =", n, flush=True)
    x, nv = _sphere(n)
    p = np.concatenate([1.0 + 0.1 * nv[:, 0], 0.02 * (1.0 + 0.1 * nv[:, 1])])
    cols = dict(zip(("px", "py", "pz", "nx", "ny", "nz"), np.concatenate([x, nv], 1).T))
    cols["phi"], cols["w"] = np.zeros(n), np.ones(n)
    t = {k: torch.tensor(np.ascontiguousarray(v), device="cuda") for k, v in cols.items()}
    band = pb.Band(n, gidx=torch.arange(n, device="cuda"), **t)
    ctx = pb.Context(0)
    y = pb.pb_ibim_matvec(ctx, band, pb.params(H, kappa=KAPPA), torch.tensor(p, device="cuda"), pb.PB_FP64).cpu().numpy()
    ctx.close()
    lam = ((1.0 + EPS_OUT) / 2.0, (1.0 + 1.0 / EPS_OUT) / 2.0)
    xl, nl, pl = x.astype(LD), nv.astype(LD), p.astype(LD)
    err = np.zeros((2, 2), dtype=LD)  # half of the vector, (operator, plain)
    for i in np.random.default_rng(n).choice(n, 96, replace=False):
        for half, terms in enumerate(_row_terms(xl, nl, pl, i)):
            e = half * n + i
            ref = LD(lam[half]) * pl[e] + terms.sum()
            plain = lam[half] * p[e] + _plain(terms)
            err[half] += [(y[e] - ref) ** 2, (plain - ref) ** 2]
    err = np.sqrt(err).astype(float)
    print("errors (operator, plain) of the halves:", err.tolist(), flush=True)
    assert (err[:, 0] <= err[:, 1]).all()
