"""GPU: the network's backward kernels where their tiles end: bands of a single node, of part
of a tile, of exactly one tile and of several weight-gradient chunks with a remainder, against
the FP64 CPU reference on the GPU's own neighbour lists and features.

Bar: both sides round activations and pre-activation gradients to BF16 at the same points, but
FP32 sums in another order can flip a rounding, 2^-8 of one value; three rounded layers bound
the relative error of a gradient block by 3·2^-8 = 1.2e-2. 2e-2 is taken.
"""
import sys

import numpy as np
import pytest

from oracle import nn_ref
from paper_1709_08070_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def band():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    ctx = pb.Context(0)
    atoms = synth.globule(12, 21)
    prm = pb.params(0.5)
    grid = pb.pb_grid_for_atoms(atoms, prm)
    phi = pb.pb_build_levelset(ctx, torch.tensor(atoms, device="cuda"), prm, grid)
    return pb, ctx, prm, pb.pb_narrowband_compact(ctx, grid, phi, prm)


@pytest.mark.parametrize("n", [1, 31, 64, 65, 257, 1000])
def test_gradients_at_tile_edges(band, n):
    import torch

    pb, ctx, prm, full = band
    print(f"case: nn gradients, first {n} band nodes", flush=True)
    sys.stdout.flush()
    f = {k: getattr(full, k)[:n].contiguous() for k in ("px", "py", "pz", "nx", "ny", "nz", "phi", "w", "gidx")}
    b = pb.Band(n, **f)
    pb.pb_nn_prepare(ctx, b, prm)
    nbr, feat = pb.pb_nn_geometry(ctx, b)
    rng = np.random.default_rng(n)
    w = np.concatenate([np.concatenate([rng.uniform(-1, 1, K * C) * np.sqrt(6.0 / K), rng.normal(0, 0.05, C)])
                        for K, C in nn_ref.layer_shapes()]).astype(np.float32)
    v, u = rng.normal(size=2 * n), rng.normal(size=2 * n)
    net = pb.Net(ctx, seed=1)
    net.set_params(w)
    loss = pb.pb_nn_train_step(ctx, net, b, prm, torch.tensor(v, device="cuda"), torch.tensor(u, device="cuda"), 0.0)
    g = net.grads().astype(np.float64)
    rl, rg = nn_ref.loss_and_grads(b.table(), nbr, feat, v, u, w, (40.5, 0.50625), 1.0)
    assert loss == pytest.approx(rl, rel=2e-2)
    off = 0
    for K, C in nn_ref.layer_shapes():
        for size in (K * C, C):
            x, y = g[off:off + size], rg[off:off + size]
            assert np.linalg.norm(x - y) <= 2e-2 * max(np.linalg.norm(y), 1e-30), (off, size)
            off += size


@pytest.fixture(scope="module")
def wide():
    import torch

    from paper_1709_08070_amd import pb

    ctx = pb.Context(0)
    atoms = synth.globule(1500, 22)
    prm = pb.params(0.5)
    grid = pb.pb_grid_for_atoms(atoms, prm)
    phi = pb.pb_build_levelset(ctx, torch.tensor(atoms, device="cuda"), prm, grid)
    return pb, ctx, prm, pb.pb_narrowband_compact(ctx, grid, phi, prm)


@pytest.mark.parametrize("n", [1, 15, 17, 64, 65, 1000, 65535, 65536, 65537])
def test_forward_at_tile_edges(wide, n):
    """One application where the forward's tiles of 16 nodes and blocks of 4 (up to 65,535 nodes) and 8
    waves end, twice with different inputs: the geometry's rows are shared. The same bound as the
    gradients', of the network's own part of the result."""
    import torch

    pb, ctx, prm, full = wide
    assert full.n >= n
    print(f"case: nn forward, first {n} band nodes", flush=True)
    f = {k: getattr(full, k)[:n].contiguous() for k in ("px", "py", "pz", "nx", "ny", "nz", "phi", "w", "gidx")}
    b = pb.Band(n, **f)
    pb.pb_nn_prepare(ctx, b, prm)
    nbr, feat = pb.pb_nn_geometry(ctx, b)
    rng = np.random.default_rng(n)
    w = np.concatenate([np.concatenate([rng.uniform(-1, 1, K * C) * np.sqrt(6.0 / K), rng.normal(0, 0.05, C)])
                        for K, C in nn_ref.layer_shapes()]).astype(np.float32)
    net = pb.Net(ctx, seed=1)
    net.set_params(w)
    lam = (40.5, 0.50625)
    for _ in range(2):
        v = rng.normal(size=2 * n)
        p = pb.pb_nn_apply(ctx, net, b, prm, torch.tensor(v, device="cuda")).cpu().numpy()
        ref = nn_ref.apply(b.table(), nbr, feat, v, w, lam, 1.0)
        for h in range(2):
            own = ref[h * n:(h + 1) * n] - v[h * n:(h + 1) * n] / lam[h]
            assert np.linalg.norm(p[h * n:(h + 1) * n] - ref[h * n:(h + 1) * n]) <= 2e-2 * np.linalg.norm(own)
