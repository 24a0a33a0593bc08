"""GPU: the level set's Runge–Kutta stages on grids at the edges of their tiles, against the FP64
oracle.

Grids of at least 2,621,440 nodes march along x in runs of four (tiles of 32 × 16 columns, two nodes
per thread); smaller ones take one thread per node in eight slabs of rows. The shapes leave one row,
one column or one plane in the last tile, take the smallest axes, odd and even row lengths, and sit
on both sides of the size rule; the atoms are spread over the whole box, so the reflected ghosts hold
real gradients. A few steps of each flow; bar 1e-10 absolute, that of the whole pipeline.

The van der Waals distance's two-level filter (4,194,304 nodes and more, more than 512 atoms): near the
molecule, on a padded grid, and inside a shell, where boxes keep more than 1024 atoms; bar 1e-13, the same arithmetic
on both sides. Cavities: shells whose voids cross mask words, on axes of more than 128
nodes, so that carries between words and chunks are taken; φ equal to the oracle's to 1e-10.
"""
import numpy as np
import pytest

import oracle
from paper_1709_08070_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [(7, 7, 7), (9, 7, 200), (8, 33, 65), (45, 161, 361),  # 2,615,445: the largest by nodes
          (45, 161, 363), (401, 7, 935), (7, 1025, 366)]


@pytest.fixture(scope="module")
def pbm():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    return pb


@pytest.mark.parametrize("dims", SHAPES, ids=str)
def test_stages_on_edge_shapes(pbm, dims):
    import torch

    h = 0.5
    print("case: level set stages on", dims, flush=True)
    rng = np.random.default_rng(sum(dims))
    ext = h * (np.array(dims) - 1)
    atoms = np.column_stack([rng.uniform(-1.0, 1.0, (40, 3)) + rng.uniform(0, 1, (40, 3)) * ext,
                             rng.uniform(1.2, 2.0, 40), np.zeros(40)])
    prm = pbm.params(h, ls_mode=pbm.PB_LS_SES, probe=0.25, reinit_steps=2)
    grid = pbm.pb_grid()
    grid.nx, grid.ny, grid.nz = dims
    grid.h = h
    origin = (-0.1, 0.2, 0.05)
    for c in range(3):
        grid.origin[c] = origin[c]
    ctx = pbm.Context(0)
    phi = pbm.pb_build_levelset(ctx, torch.tensor(atoms, device="cuda"), prm, grid).cpu().numpy()
    ctx.close()
    ophi, _ = oracle.ses(dims, origin, atoms, oracle.params(h, probe=0.25, reinit_steps=2))
    d = np.max(np.abs(phi - ophi))
    print(f"  max |Δφ| {d:.3e}", flush=True)
    assert d <= 1e-10


@pytest.mark.parametrize("pad,dims", [(0.0, (161, 163, 161)), (90.0, (9, 1001, 467)), (None, (163, 161, 161))],
                         ids=["near", "far", "inside a shell"])
def test_vdw_two_levels(pbm, pad, dims):
    import torch

    h = 0.31
    atoms = synth.shell(60.0) if pad is None else synth.globule(3000, 12)
    origin = -0.5 * h * np.array(dims) if pad is None else atoms[:, :3].min(axis=0) - 2.0 - pad
    print("case: vdW distance in two levels,", dims, "padded by", pad, flush=True)
    grid = pbm.pb_grid()
    grid.nx, grid.ny, grid.nz = dims
    grid.h = h
    for c in range(3):
        grid.origin[c] = origin[c]
    ctx = pbm.Context(0)
    prm = pbm.params(h, ls_mode=pbm.PB_LS_VDW)
    phi = pbm.pb_build_levelset(ctx, torch.tensor(atoms, device="cuda"), prm, grid).cpu().numpy().reshape(dims)
    ctx.close()
    rng = np.random.default_rng(5)
    idx = np.stack([rng.integers(0, d, 20000) for d in dims], 1)
    ends = [np.r_[0:4, d - 4:d] for d in dims]
    idx = np.vstack([idx, np.stack(np.meshgrid(*ends, indexing="ij"), -1).reshape(-1, 3)])
    x = np.asarray(origin) + h * idx
    ref = np.concatenate([(np.sqrt(((q[:, None] - atoms[None, :, :3]) ** 2).sum(2)) - atoms[:, 3]).min(1)
                          for q in np.array_split(x, 64)])
    d = np.max(np.abs(phi[tuple(idx.T)] - ref))
    print(f"  max |Δφ| {d:.3e}", flush=True)
    assert d <= 1e-13
    if pad is None:  # the middle box keeps more than 1024 atoms: its tiles filter from all of them
        c = np.asarray(origin) + h * np.array([80 + 3.5, 80 + 7.5, 80 + 7.5])
        r = 0.5 * h * np.sqrt(7.0**2 + 15.0**2 + 15.0**2)
        dist = np.linalg.norm(atoms[:, :3] - c, axis=1)
        assert np.sum(dist <= (dist - atoms[:, 3]).min() + 2 * r + atoms[:, 3]) > 1024


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_cavities_across_words(pbm, axis):
    import torch

    h = 0.5
    one = synth.shell(5.0, 1.6, 2.2)
    step = np.zeros(5)
    step[axis] = 31.0  # 62 nodes: the voids lie across the 64-node words of z and the chunks of x and y
    atoms = np.vstack([one, one + step, one + 2 * step])
    prm = pbm.params(h, ls_mode=pbm.PB_LS_SES, reinit_steps=2)
    grid = pbm.pb_grid_for_atoms(atoms, prm)
    dims, origin = (grid.nx, grid.ny, grid.nz), tuple(grid.origin)
    print("case: three shells along axis", axis, "on", dims, flush=True)
    ctx = pbm.Context(0)
    phi = pbm.pb_build_levelset(ctx, torch.tensor(atoms, device="cuda"), prm, grid).cpu().numpy()
    ctx.close()
    ophi, ncav = oracle.ses(dims, origin, atoms, oracle.params(h, reinit_steps=2))
    d = np.max(np.abs(phi - ophi))
    print(f"  cavity nodes {ncav}, max |Δφ| {d:.3e}", flush=True)
    assert ncav > 0 and max(dims) > 128
    assert d <= 1e-10
