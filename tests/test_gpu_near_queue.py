"""GPU: the near-field walk's queue of hits, and the row starts of the near-field matrix.

Queue. A target's candidates are read 256 at a turn; its hits wait in a queue, are taken 64 at a time, and
what is left (up to 63) is carried to the next turn. All nodes lie in one cell, so the candidates come in index
order: "near" nodes in one corner, within r_c of each other, and "far" ones in the opposite corner, beyond
r_c and without weight, so that they are candidates but add exactly nothing to the near nodes' rows. The order of
the two kinds sets how many hits each turn has. The near nodes' rows are then sums over FP64 near pairs
alone, in both operators: bar 1e-9 of the largest entry for one application (rounding is below 1e-12; a pair lost or
taken twice is a few percent of its row).

The matrix that a solve keeps is filled by the same walk: two steps with it and two with the FP64 operator
from zero, bar 1e-4 (the far nodes' rows are FP32, 1e-5 per application by the operator's bar, and reach the others
through the two steps' coefficients).

Row starts. From 16,384 rows on they come from a scan of two launches in tiles of 4096 values: four steps of a solve as
above, to 1e-3 of the largest entry (1e-5 per application, times the growth over four steps); rows that
start wrong change entries by their own size.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (candidates, hits) of each turn; all but the last have 256 candidates
TURNS = [
    [(256, 63), (256, 256), (100, 1)],  # the queue at its fullest, 63 + 256, and a last turn that completes 64
    [(256, 63), (256, 256), (256, 256), (37, 0)],  # a remainder and nothing after it
    [(256, 64), (256, 0), (256, 65), (256, 127), (5, 1)],  # nothing carried, nothing new, 1 carried, 63 + … = 128
    [(256, 1), (256, 1), (256, 1), (256, 255), (256, 256), (62, 62)],
    [(256, 0), (256, 0), (200, 200)],
]


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    return pb, torch, pb.Context(0)


def _ball(rng, n, centre, radius):
    x = rng.normal(size=(n, 3))
    return centre + radius * x / np.linalg.norm(x, axis=1)[:, None] * rng.random((n, 1)) ** (1 / 3)


def _band(pb, torch, rng, x, w):
    nv = rng.normal(size=x.shape)
    nv /= np.linalg.norm(nv, axis=1)[:, None]
    cols = dict(zip(("px", "py", "pz", "nx", "ny", "nz"), np.concatenate([x, nv], 1).T))
    cols["phi"], cols["w"] = np.zeros(len(x)), w
    t = {k: torch.tensor(np.ascontiguousarray(v), device="cuda") for k, v in cols.items()}
    return pb.Band(len(x), gidx=torch.arange(len(x), device="cuda"), **t)


def _queue_case(pb, torch, turns):
    rng = np.random.default_rng(len(turns))
    near = np.concatenate([rng.permutation(np.arange(c) < h) for c, h in turns])
    x = np.where(near[:, None], _ball(rng, len(near), 0.1, 0.1), _ball(rng, len(near), 0.95, 0.05))
    band = _band(pb, torch, rng, x, np.where(near, rng.uniform(0.5, 1.0, len(near)), 0.0))
    # r_c = 1 holds each corner whole and keeps the two (1.32 apart) asunder; τ = 0.025 leaves most pairs their kernels
    return band, near, pb.params(0.5, tau_k=0.05, near_k=2.0), rng


@pytest.mark.parametrize("turns", TURNS, ids=lambda t: "-".join(str(h) for _, h in t))
def test_queue_of_one_application(env, turns):
    pb, torch, ctx = env
    print("case: near queue, hits per turn", [h for _, h in turns], flush=True)
    band, near, prm, rng = _queue_case(pb, torch, turns)
    p = torch.tensor(rng.normal(size=2 * band.n), device="cuda")
    rows = torch.tensor(np.tile(near, 2), device="cuda")
    ref = pb.pb_ibim_matvec(ctx, band, prm, p, pb.PB_FP64)[rows]
    for precision in (pb.PB_MIXED, pb.PB_TREE):
        y = pb.pb_ibim_matvec(ctx, band, prm, p, precision)[rows]
        assert float((y - ref).abs().max()) <= 1e-9 * float(ref.abs().max())
    hits = int(near.sum())
    assert ctx.tree_info()["near_pairs"] == hits ** 2 + (band.n - hits) ** 2


def _steps(pb, torch, ctx, band, prm, steps):
    atoms = torch.tensor([[0.5, 0.4, 3.0, 1.5, 1.0]], dtype=torch.float64, device="cuda")
    out = []
    for precision in (pb.PB_MIXED, pb.PB_FP64):
        opts = pb.solve_opts(precision=precision, tol=1e-12, max_iter=steps, x0=pb.PB_X0_ZERO)
        out.append(pb.pb_ibim_solve(ctx, band, atoms, prm, opts, allow_noconv=True)[0])
    return out


@pytest.mark.parametrize("turns", TURNS, ids=lambda t: "-".join(str(h) for _, h in t))
def test_queue_of_the_matrix(env, turns):
    pb, torch, ctx = env
    print("case: near matrix queue, hits per turn", [h for _, h in turns], flush=True)
    band, near, prm, _ = _queue_case(pb, torch, turns)
    rows = torch.tensor(np.tile(near, 2), device="cuda")
    a, b = (v[rows] for v in _steps(pb, torch, ctx, band, prm, 2))
    assert float((a - b).abs().max()) <= 1e-4 * float(b.abs().max())


@pytest.mark.parametrize("n", [16385, 20479, 20480, 33000])
def test_row_starts_of_the_matrix(env, n):
    pb, torch, ctx = env
    print("case: near matrix rows, n =", n, flush=True)
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, 3))
    x *= (0.15 * np.sqrt(n) / np.linalg.norm(x, axis=1))[:, None]
    band = _band(pb, torch, rng, x[np.lexsort(x.T[::-1].round(0))], rng.uniform(0.1, 1.0, n))
    a, b = _steps(pb, torch, ctx, band, pb.params(0.5), 4)
    assert float((a - b).abs().max()) <= 1e-3 * float(b.abs().max())
