"""GPU: the symmetric kernels' tile shapes against the one-directional kernels at band sizes around
their edges: part of a 128-node tile, one tile and one node more, one sub-block and one node
more, and both sides of each change of shape.

Bars: FP64 against FP64, sums of up to 2·10^4 terms of one sign of size in another order: 1e-12 of
the result's norm. FP32 partial sums hold at most 256 terms, rounded at 6e-8 each: 1.5e-5 at the
worst, 1e-5 (the operator's bar elsewhere) taken.
"""
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [1, 64, 127, 128, 129, 255, 257, 511, 512, 513, 1025, 10239, 10241, 12799, 12801, 13311, 13313, 32769, 61439, 61441]


def _band(pb, torch, n):
    rng = np.random.default_rng(n)
    nv = rng.normal(size=(n, 3))
    nv /= np.linalg.norm(nv, axis=1)[:, None]
    x = nv * (0.15 * np.sqrt(n) + 1.0) * (1.0 + 0.01 * rng.normal(size=(n, 1)))
    x = x[np.lexsort(x.T[::-1].round(0))]
    cols = dict(zip(("px", "py", "pz", "nx", "ny", "nz"), np.concatenate([x, nv], 1).T))
    cols["phi"] = rng.uniform(-1, 1, n)
    cols["w"] = rng.uniform(0.1, 1, n)
    t = {k: torch.tensor(np.ascontiguousarray(v), device="cuda") for k, v in cols.items()}
    return pb.Band(n, gidx=torch.arange(n, device="cuda"), **t)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("kappa,metric", [(0.1257, 0), (0.1257, 2), (0.0, 0), (0.1257, 1)])
def test_tiles(n, kappa, metric):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    print(f"case: tiles n={n} kappa={kappa} metric={metric}", flush=True)
    sys.stdout.flush()
    prm = pb.params(0.5, kappa=kappa, reg_metric=metric)
    b = _band(pb, torch, n)
    p = torch.tensor(np.random.default_rng(n).normal(size=2 * n), device="cuda")
    ctx = pb.Context(0)

    def run(prec, env=None):
        if env:
            os.environ[env[0]] = env[1]
        try:
            y = pb.pb_ibim_matvec(ctx, b, prm, p, prec)
            assert torch.equal(y, pb.pb_ibim_matvec(ctx, b, prm, p, prec)), "not reproducible"
        finally:
            if env:
                del os.environ[env[0]]
        return y

    ref = run(pb.PB_FP64, ("PB_F64_CFG", "0"))
    assert float((run(pb.PB_FP64) - ref).norm()) <= 1e-12 * float(ref.norm())
    if metric != pb.PB_REG_TANGENT:
        for env in (None, ("PB_FAR_CFG", "0"), ("PB_FAR_CFG", "2"), ("PB_FAR_CFG", "4")):
            assert float((run(pb.PB_MIXED, env) - ref).norm()) <= 1e-5 * float(ref.norm()), env
