"""GPU: right-hand side and energy over the atom counts at which the energy kernel changes the atoms it
takes per block (1, 2, 4 or 8, the choice by turns of 256 CUs) and leaves a partial last group, against the
FP64 oracle on a small band (partial last block of 64 nodes). Both sides sum the same terms in FP64 in other
orders: each term is off by a few 1e-16 and the sums lose about a factor sqrt(n) to cancellation, so the
bar is 1e-12 of the largest entry.
"""
import numpy as np
import pytest

import oracle
from paper_1709_08070_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def born():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    prm = pb.params(0.5, ls_mode=pb.PB_LS_VDW)
    atoms = synth.born_ion()
    ctx = pb.Context(0)
    grid = pb.pb_grid_for_atoms(atoms, prm)
    phi = pb.pb_build_levelset(ctx, torch.tensor(atoms, device="cuda"), prm, grid)
    return pb, ctx, prm, pb.pb_narrowband_compact(ctx, grid, phi, prm)


@pytest.mark.parametrize("n_atoms", [1, 63, 255, 257, 511, 513, 767, 1023, 1025, 2047, 2049, 4097])
def test_rhs_and_energy_by_atom_count(born, n_atoms):
    import torch

    pb, ctx, prm, band = born
    rng = np.random.default_rng(n_atoms)
    atoms = np.column_stack([rng.uniform(-0.5, 0.5, (n_atoms, 3)), np.ones(n_atoms), rng.normal(size=n_atoms)])
    print("case: rhs and energy", n_atoms, "atoms, n =", band.n, flush=True)
    at = torch.tensor(atoms, device="cuda")
    p = rng.normal(size=2 * band.n)
    oprm = oracle.params(0.5)
    g = pb.pb_ibim_rhs(ctx, band, at, prm).cpu().numpy()
    og = oracle.rhs(band.table(), atoms, oprm)
    psi = torch.full((n_atoms + 1,), 7.0, dtype=torch.float64, device="cuda")
    en = pb.pb_solvation_energy(ctx, band, at, prm, torch.tensor(p, device="cuda"), psi)
    og_pol, opsi = oracle.energy(band.table(), atoms, oprm, p)
    psi = psi.cpu().numpy()
    for a, b in ((g[: band.n], og[: band.n]), (g[band.n :], og[band.n :]), (psi[:-1], opsi)):
        assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))
    assert psi[-1] == 7.0
    assert abs(en.g_pol - og_pol) <= 1e-12 * 0.5 * np.sum(np.abs(atoms[:, 4] * opsi))
    assert en.area == pytest.approx(oracle.area(band.table(), 0.5), rel=1e-13)
