"""GPU: the treecode's tree, batches, lists and segments where they can go wrong: one node, one
leaf and one node more, coincident nodes that no split separates (leaves beyond the depth limit;
fewer than a proxy cluster holds, since a cluster of zero radius is interpolated whatever θ), exact
ties on a lattice, bands on both sides of the switch from sibling to packed batches, and a tree
with more leaves than the wave walk keeps on chip.

Bars: with a vanishing θ the treecode is the dense FP32 far field reordered, 1e-6 as in the other
treecode tests; with the default degree and θ 3e-5 against the exact operator. On the large sets,
volumes with weights of random sign, for which no interpolation error is known beforehand, the
error on sampled rows falls with the degree, as it does only if every source is in exactly one list.
"""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    return pb, torch, pb.Context(0)


def _band(pb, torch, x, seed, w=1.0):
    rng = np.random.default_rng(seed)
    nv = rng.normal(size=x.shape)
    nv /= np.linalg.norm(nv, axis=1)[:, None]
    cols = dict(zip(("px", "py", "pz", "nx", "ny", "nz"), np.concatenate([x, nv], 1).T))
    cols["phi"] = rng.uniform(-1, 1, len(x))
    cols["w"] = w * rng.uniform(0.1, 1, len(x))
    t = {k: torch.tensor(np.ascontiguousarray(v), device="cuda") for k, v in cols.items()}
    return pb.Band(len(x), gidx=torch.arange(len(x), device="cuda"), **t)


def _cloud(kind, n):
    rng = np.random.default_rng(n)
    if kind == "equal":  # n nodes on three sites 40 apart
        return np.array([[0.0, 0, 0], [40, 0, 0], [0, 0, 40.0]])[np.arange(n) % 3]
    if kind == "lattice":
        m = int(np.ceil(n ** (1 / 3)))
        return np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n] * 1.5
    return rng.uniform(-1, 1, (n, 3)) * 0.6 * n ** (1 / 3)


@pytest.mark.parametrize("kind,n", [("cube", 1), ("cube", 64), ("cube", 65), ("cube", 300), ("cube", 3000),
                                    ("equal", 150), ("equal", 300), ("lattice", 1728)])
def test_small_trees(env, kind, n):
    pb, torch, ctx = env
    print(f"case: tree {kind} {n}", flush=True)
    sys.stdout.flush()
    b = _band(pb, torch, _cloud(kind, n), n)
    p = torch.tensor(np.random.default_rng(n).normal(size=2 * n), device="cuda")
    ref = pb.pb_ibim_matvec(ctx, b, pb.params(0.5), p, pb.PB_FP64)
    for kw, bar in ((dict(tree_theta=1e-3), 1e-6), ({}, 3e-5)):
        prm = pb.params(0.5, **kw)
        y = pb.pb_ibim_matvec(ctx, b, prm, p, pb.PB_TREE)
        assert torch.equal(y, pb.pb_ibim_matvec(ctx, b, prm, p, pb.PB_TREE)), "not reproducible"
        assert float((y - ref).norm()) <= bar * float(ref.norm()), kw


@pytest.mark.parametrize("n", [100_000, 250_000, 2_400_000])
def test_large_trees(env, n):
    pb, torch, ctx = env
    print(f"case: tree volume {n}", flush=True)
    sys.stdout.flush()
    h, rng = 0.1, np.random.default_rng(n)
    x = rng.uniform(0, 1, (n, 3)) * (n / 2.4) ** (1 / 3)
    b = _band(pb, torch, x, n, w=1e4)
    p = rng.normal(size=2 * n)
    rows = rng.choice(n, 48, replace=False)
    ref = np.concatenate(oracle.matvec_rows(b.table(), oracle.params(h), p, rows))
    err = []
    for degree in (2, 4, 6):
        y = pb.pb_ibim_matvec(ctx, b, pb.params(h, tree_degree=degree), torch.tensor(p, device="cuda"),
                              pb.PB_TREE).cpu().numpy()
        err.append(np.linalg.norm(np.concatenate([y[rows], y[n + rows]]) - ref) / np.linalg.norm(ref))
    print(f"  {ctx.tree_info()} errors {err}", flush=True)
    assert err[0] > err[1] > err[2]
