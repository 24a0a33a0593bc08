"""GPU: the FP64 operator's exponential by table over its whole range: κr from nothing to past where e^{−κr}
underflows, and κ so large that the padding records' κr (1.7e6 κ) no longer fits the table's integer index
(κ > 3.4), against the FP64 oracle on the Born ion. Both sides are FP64 sums of the same 3000 terms in other orders;
bar 1e-12 of the result's norm.
"""
import numpy as np
import pytest

import oracle
from paper_1709_08070_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kappa", [1e-6, 0.02, 0.1257, 1.0, 3.0, 3.6, 40.0, 400.0])
def test_fp64_operator_over_kappa(kappa):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    print("case: FP64 operator, kappa", kappa, flush=True)
    prm = pb.params(0.25, ls_mode=pb.PB_LS_VDW, kappa=kappa)
    atoms = synth.born_ion()
    ctx = pb.Context(0)
    grid = pb.pb_grid_for_atoms(atoms, prm)
    phi = pb.pb_build_levelset(ctx, torch.tensor(atoms, device="cuda"), prm, grid)
    band = pb.pb_narrowband_compact(ctx, grid, phi, prm)
    p = np.random.default_rng(4).normal(size=2 * band.n)
    y = pb.pb_ibim_matvec(ctx, band, prm, torch.tensor(p, device="cuda"), pb.PB_FP64).cpu().numpy()
    ctx.close()
    ref = oracle.matvec(band.table(), oracle.params(0.25, kappa=kappa), p)
    rel = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    print(f"  n={band.n}: {rel:.2e}", flush=True)
    assert rel <= 1e-12
