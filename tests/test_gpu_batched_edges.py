"""GPU: the batched solve's Gram–Schmidt kernels at the edges of their segments (1024 elements, molecules of
less than one, of one and a bit, of many) and of their groups of eight basis vectors (restart lengths around
8 and 16, and 1), on an uneven batch. Every molecule's solution is judged by the exact FP64 operator, applied
on its own: the residual has to meet the tolerance; and a repeated solve returns the same bits.
"""
import numpy as np
import pytest

from paper_1709_08070_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def batch():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    ctx = pb.Context(0)
    prm = pb.params(0.5, ls_mode=pb.PB_LS_VDW)
    mols = [synth.born_ion(0.6), synth.born_ion(1.2), synth.born_ion(2.0), synth.globule(25, 4)]
    at = [torch.tensor(a, device="cuda") for a in mols]
    bands = []
    for a, t in zip(mols, at):
        grid = pb.pb_grid_for_atoms(a, prm)
        bands.append(pb.pb_narrowband_compact(ctx, grid, pb.pb_build_levelset(ctx, t, prm, grid), prm))
    return pb, ctx, prm, at, bands


@pytest.mark.parametrize("restart", [1, 7, 8, 9, 16, 17, 100])
def test_restarts(batch, restart):
    import torch

    pb, ctx, prm, at, bands = batch
    tol = 1e-7
    print("case: batched solve, restart", restart, "n =", [b.n for b in bands], flush=True)
    opts = pb.solve_opts(tol=tol, precision=pb.PB_MIXED, restart=restart, max_iter=2000)
    ps, stats, _ = pb.pb_ibim_solve_batched(ctx, bands, at, prm, opts)
    again, _, _ = pb.pb_ibim_solve_batched(ctx, bands, at, prm, opts)
    for b, a, p, q, st in zip(bands, at, ps, again, stats):
        g = pb.pb_ibim_rhs(ctx, b, a, prm)
        r = g - pb.pb_ibim_matvec(ctx, b, prm, p, pb.PB_FP64)
        rel = float(torch.linalg.norm(r) / torch.linalg.norm(g))
        print(f"  n={b.n}: iters {st.iters}, residual {rel:.2e}", flush=True)
        assert st.converged and rel <= tol * (1 + 1e-6)
        assert np.array_equal(p.cpu().numpy(), q.cpu().numpy())
