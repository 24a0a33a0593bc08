"""GPU: cell list, near-field matrix and neighbour search on point sets that stress their limits:
a single node, a full 64-entry chunk and one more, cells with more candidates than the
neighbour search keeps on chip, and many equal distances.

Bars: neighbour lists equal a full sort by (distance, index). The mixed operator within 1e-5 of the
largest entry of the FP64 one, the bar its FP32 far field has everywhere else.
"""
import sys

import numpy as np
import pytest

from oracle import nn_ref

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    return pb, torch, pb.Context(0)


def _cloud(kind, n):
    rng = np.random.default_rng(n)
    if kind == "equal":  # n points on 4 sites
        return rng.uniform(-0.2, 0.2, (4, 3))[np.arange(n) % 4]
    if kind == "lattice":  # spacing 0.125: exact ties everywhere
        m = int(np.ceil(n ** (1 / 3)))
        return (np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n] * 0.125)
    x = rng.normal(size=(n, 3))
    return x / np.linalg.norm(x, axis=1)[:, None] * 0.7 * rng.random((n, 1)) ** (1 / 3)


def _band(pb, torch, x, seed):
    rng = np.random.default_rng(seed)
    nv = rng.normal(size=x.shape)
    nv /= np.linalg.norm(nv, axis=1)[:, None]
    cols = dict(zip(("px", "py", "pz", "nx", "ny", "nz"), np.concatenate([x, nv], 1).T))
    cols["phi"] = rng.uniform(-1, 1, len(x))
    cols["w"] = rng.uniform(0.1, 1, len(x))
    t = {k: torch.tensor(np.ascontiguousarray(v), device="cuda") for k, v in cols.items()}
    return pb.Band(len(x), gidx=torch.arange(len(x), device="cuda"), **t)


CLOUDS = [("ball", 1), ("ball", 15), ("ball", 64), ("ball", 65), ("ball", 500), ("ball", 900), ("equal", 70),
          ("equal", 400), ("lattice", 343)]


@pytest.mark.parametrize("kind,n", CLOUDS)
def test_neighbours(env, kind, n):
    pb, torch, ctx = env
    print(f"case: neighbours {kind} {n}", flush=True)
    sys.stdout.flush()
    x = _cloud(kind, n)
    prm = pb.params(0.5)
    b = _band(pb, torch, x, n)
    pb.pb_nn_prepare(ctx, b, prm)
    nbr, _ = pb.pb_nn_geometry(ctx, b)
    d2 = ((x[:, None, 0] - x[None, :, 0]) ** 2 + (x[:, None, 1] - x[None, :, 1]) ** 2) + \
        (x[:, None, 2] - x[None, :, 2]) ** 2
    order = np.argsort(d2, axis=1, kind="stable")[:, :16]
    ref = np.tile(np.arange(n)[:, None], (1, 16))
    ref[:, : order.shape[1]] = order
    np.testing.assert_array_equal(nbr, ref)
    if n >= 16:
        np.testing.assert_array_equal(ref, nn_ref.knn(x))


@pytest.mark.parametrize("kind,n", CLOUDS)
def test_mixed_operator(env, kind, n):
    pb, torch, ctx = env
    print(f"case: mixed operator {kind} {n}", flush=True)
    sys.stdout.flush()
    prm = pb.params(0.5)
    b = _band(pb, torch, _cloud(kind, n), n)
    p = torch.tensor(np.random.default_rng(n).normal(size=2 * n), device="cuda")
    y = pb.pb_ibim_matvec(ctx, b, prm, p, pb.PB_MIXED)
    y2 = pb.pb_ibim_matvec(ctx, b, prm, p, pb.PB_MIXED)
    ref = pb.pb_ibim_matvec(ctx, b, prm, p, pb.PB_FP64)
    assert torch.equal(y, y2)
    assert float((y - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


@pytest.mark.parametrize("n", [8190, 8191, 8192, 16382, 16383, 16384, 33000])
def test_row_scan_lengths(env, n):
    """Row starts of n + 1 values around the turns of the one-block scan (8192 values each) and its end
    (16,384): a wrong start would put near pairs in other rows."""
    pb, torch, ctx = env
    print("case: row scan, n =", n, flush=True)
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, 3))
    x *= (0.15 * np.sqrt(n) / np.linalg.norm(x, axis=1))[:, None]
    prm = pb.params(0.5)
    b = _band(pb, torch, x[np.lexsort(x.T[::-1].round(0))], n)
    p = torch.tensor(rng.normal(size=2 * n), device="cuda")
    y = pb.pb_ibim_matvec(ctx, b, prm, p, pb.PB_MIXED)
    ref = pb.pb_ibim_matvec(ctx, b, prm, p, pb.PB_FP64)
    assert float((y - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 127, 128, 129, 300])
def test_operator_of_near_pairs_only(env, n):
    """Every pair nearer than r_c: the mixed and the tree operator are then their FP64 near fields alone,
    n sources for each target, around the turns of 64 and the queue of 128. Bar 1e-9 of the largest
    entry: both sides are FP64, and a pair in FP32, left out or taken twice shows at 1e-7 or above."""
    pb, torch, ctx = env
    print("case: near pairs only, n =", n, flush=True)
    prm = pb.params(0.5)
    x = _cloud("ball", n)
    x *= 0.45 * prm.near_k * prm.h / np.linalg.norm(x, axis=1).max()
    b = _band(pb, torch, x, n)
    p = torch.tensor(np.random.default_rng(n).normal(size=2 * n), device="cuda")
    ref = pb.pb_ibim_matvec(ctx, b, prm, p, pb.PB_FP64)
    for precision in (pb.PB_MIXED, pb.PB_TREE):
        y = pb.pb_ibim_matvec(ctx, b, prm, p, precision)
        assert float((y - ref).abs().max()) <= 1e-9 * float(ref.abs().max())
    assert ctx.tree_info()["near_pairs"] == n * n


@pytest.mark.parametrize("n", [8190, 8191, 8192, 16382, 16383, 16384])
def test_near_matrix_row_starts(env, n):
    """A solve keeps its near field as a matrix: four steps with it and four with the FP64 operator from the same
    start give the same iterate, to 1e-3 of its largest entry (1e-5 per application, the bar of the operator
    above, times the growth over four steps); rows that start wrong change entries by their own size."""
    pb, torch, ctx = env
    print("case: near matrix, n =", n, flush=True)
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, 3))
    x *= (0.15 * np.sqrt(n) / np.linalg.norm(x, axis=1))[:, None]
    b = _band(pb, torch, x[np.lexsort(x.T[::-1].round(0))], n)
    atoms = torch.tensor([[0.0, 0.0, 0.0, 1.5, 1.0]], dtype=torch.float64, device="cuda")
    prm = pb.params(0.5)
    out = []
    for precision in (pb.PB_MIXED, pb.PB_FP64):
        opts = pb.solve_opts(precision=precision, tol=1e-12, max_iter=4)
        out.append(pb.pb_ibim_solve(ctx, b, atoms, prm, opts, allow_noconv=True)[0])
    assert float((out[0] - out[1]).abs().max()) <= 1e-3 * float(out[1].abs().max())
