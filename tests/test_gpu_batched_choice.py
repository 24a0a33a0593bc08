"""GPU: the batched solve's choice of its far-field kernel belongs to the batch it was made for.

A first call fixes the one-directional kernel (tile 256, two targets per lane) by the environment; later
calls have no such setting and time the kernels of their own batch. Bands of 30,000 nodes and more: the
symmetric kernel, which evaluates half the pairs, is faster there by more than half, so the timing
cannot miss it.
"""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    def band(n):
        k = np.arange(n) + 0.5  # a spiral on a sphere with the density of a band's projections
        z, a = 1.0 - 2.0 * k / n, k * np.pi * (3.0 - np.sqrt(5.0))
        s = np.sqrt(1.0 - z * z)
        nv = np.stack([s * np.cos(a), s * np.sin(a), z], 1)
        cols = dict(zip(("px", "py", "pz", "nx", "ny", "nz"),
                        np.concatenate([np.sqrt(n / (64.0 * np.pi)) * nv, nv], 1).T))
        cols["phi"], cols["w"] = np.zeros(n), np.ones(n)
        t = {c: torch.tensor(np.ascontiguousarray(v), device="cuda") for c, v in cols.items()}
        return pb.Band(n, gidx=torch.arange(n, device="cuda"), **t)

    at = torch.tensor([[0.0, 0.0, 0.0, 1.5, 1.0]], dtype=torch.float64, device="cuda")

    def solve(ctx, sizes, kappa, cfg=None):
        if cfg is not None:
            os.environ["PB_FAR_CFG"] = cfg
        try:
            opts = pb.solve_opts(tol=1e-12, precision=pb.PB_MIXED, max_iter=1)
            return pb.pb_ibim_solve_batched(ctx, [band(n) for n in sizes], [at] * len(sizes),
                                            pb.params(0.5, kappa=kappa), opts, allow_noconv=True)[2]
        finally:
            os.environ.pop("PB_FAR_CFG", None)

    return pb, solve


@pytest.mark.parametrize("sizes,kappa", [((40000, 40000), 0.0), ((30000, 50000), 0.1257)], ids=["unscreened", "sizes"])
def test_other_batches_choose_for_themselves(env, sizes, kappa):
    pb, solve = env
    print("case: batch choice after another batch,", sizes, kappa, flush=True)
    ctx = pb.Context(0)
    first = solve(ctx, (40000, 40000), 0.1257, "2")
    assert first.far_symmetric == 0 and first.far_tile == 256 and first.far_tpl == 2
    assert solve(ctx, sizes, kappa).far_symmetric == 1
    ctx.close()


def test_environment_holds_for_its_call(env):
    pb, solve = env
    print("case: batch choice by the environment", flush=True)
    ctx = pb.Context(0)
    sizes = (40000, 30000)
    assert solve(ctx, sizes, 0.1257).far_symmetric == 1
    second = solve(ctx, sizes, 0.1257, "2")
    assert second.far_symmetric == 0 and second.far_tile == 256 and second.far_tpl == 2
    assert solve(ctx, sizes, 0.1257, "4").far_symmetric == 1
    assert solve(ctx, sizes, 0.1257).far_symmetric == 1
    ctx.close()
