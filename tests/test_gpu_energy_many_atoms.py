"""GPU: the energy of many atoms on small bands.

Values: atom counts whose blocks of 2, 4 and 8 atoms are more than one per compute unit, with whole and
partial last blocks, against the FP64 oracle; the same terms in another order, so 1e-12 of the largest entry.

Time: the pairs of a small band may take 1.5 times as long each as those of a large one. A block of 512 threads on
2924 nodes makes 6 turns where 5.7 would do, so 1.05, and its set-up and sums come to about a turn, 1.2; what is above that
is idle time.
"""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1709_08070_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    return pb, torch, pb.Context(0)


@pytest.mark.parametrize("n_atoms", [1026, 1279, 2050, 3073, 8191, 20000])
def test_values(env, n_atoms):
    pb, torch, ctx = env
    print("case: energy of", n_atoms, "atoms", flush=True)
    prm = pb.params(0.5, ls_mode=pb.PB_LS_VDW)
    ion = synth.born_ion()
    grid = pb.pb_grid_for_atoms(ion, prm)
    band = pb.pb_narrowband_compact(ctx, grid, pb.pb_build_levelset(ctx, torch.tensor(ion, device="cuda"), prm, grid), prm)
    rng = np.random.default_rng(n_atoms)
    atoms = np.column_stack([rng.uniform(-0.5, 0.5, (n_atoms, 3)), np.ones(n_atoms), rng.normal(size=n_atoms)])
    p = rng.normal(size=2 * band.n)
    psi = torch.full((n_atoms + 1,), 7.0, dtype=torch.float64, device="cuda")
    en = pb.pb_solvation_energy(ctx, band, torch.tensor(atoms, device="cuda"), prm, torch.tensor(p, device="cuda"), psi)
    g_pol, opsi = oracle.energy(band.table(), atoms, oracle.params(0.5), p)
    psi = psi.cpu().numpy()
    assert np.max(np.abs(psi[:-1] - opsi)) <= 1e-12 * np.max(np.abs(opsi))
    assert psi[-1] == 7.0
    assert abs(en.g_pol - g_pol) <= 1e-12 * 0.5 * np.sum(np.abs(atoms[:, 4] * opsi))


def test_time_per_pair(env):
    pb, torch, ctx = env
    print("case: energy of 20,000 atoms, time per pair", flush=True)
    g = torch.Generator("cuda").manual_seed(1)
    atoms = torch.rand((20000, 5), dtype=torch.float64, device="cuda", generator=g)
    prm, per = pb.params(0.5), []
    for n in (2924, 45818):
        x = [torch.randn(n, dtype=torch.float64, device="cuda", generator=g) * 20.0 for _ in range(6)]
        one = torch.ones(n, dtype=torch.float64, device="cuda")
        band = pb.Band(n, *x, one, one, torch.arange(n, device="cuda"))
        p = torch.ones(2 * n, dtype=torch.float64, device="cuda")
        pb.pb_solvation_energy(ctx, band, atoms, prm, p)
        pb.lib.pb_set_timing(ctx.handle, 1)
        for _ in range(10):
            pb.pb_solvation_energy(ctx, band, atoms, prm, p)
        ms, launches = ctypes.c_double(), ctypes.c_int64()
        pb.lib.pb_kernel_time(ctx.handle, b"energy", ctypes.byref(ms), ctypes.byref(launches))
        pb.lib.pb_set_timing(ctx.handle, 0)
        per.append(ms.value / launches.value / (20000.0 * n))
    print("  ns per pair:", [v * 1e6 for v in per], flush=True)
    assert per[0] <= 1.5 * per[1]
