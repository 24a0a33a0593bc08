"""GPU: the level set's Runge–Kutta stages on grids at the edges of their tiles, against the FP64
oracle.

Grids of at least 2,621,440 nodes march along x in runs of four (tiles of 32 × 16 columns, two nodes
per thread); smaller ones take one thread per node in eight slabs of rows. The shapes leave one row,
one column or one plane in the last tile, take the smallest axes, odd and even row lengths, and sit
on both sides of the size rule; the atoms are spread over the whole box, so the reflected ghosts hold
real gradients. A few steps of each flow; bar 1e-10 absolute, that of the whole pipeline.
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
