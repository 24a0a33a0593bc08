"""GPU: right-hand side of large bands with few atoms.

Against the literal formula in FP64 torch on both sides of the rule that lets waves share the
atoms (8 atoms, one per 2048 nodes) and at whole and partial tiles of 256 atoms. Both sum the same at most 293
terms, each off by a few 1e-16, with about a factor sqrt(293) lost to cancellation: bar 1e-13 of the largest entry.

Time: with one atom the kernel does no more than read six arrays and write two, so it may take 1.6 times a
copy of as many bytes.
"""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    return pb, torch, pb.Context(0)


def _band(pb, torch, n):
    g = torch.Generator("cuda").manual_seed(n)
    rand = lambda: torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    x, v = [rand() * 20.0 for _ in range(3)], [rand() for _ in range(3)]
    one = torch.ones(n, dtype=torch.float64, device="cuda")
    return pb.Band(n, *x, *v, one, one, torch.arange(n, device="cuda"))


def _formula(torch, band, atoms):
    g1, g2 = torch.zeros_like(band.px), torch.zeros_like(band.px)
    for x, y, z, _, q in atoms:
        dx, dy, dz = band.px - x, band.py - y, band.pz - z
        r = (dx * dx + dy * dy + dz * dz).sqrt()
        g1 += q / (4.0 * math.pi) / r
        g2 -= q / (4.0 * math.pi) * (dx * band.nx + dy * band.ny + dz * band.nz) / r ** 3
    return torch.cat([g1, g2])


@pytest.mark.parametrize("n,m", [(874, 7), (874, 8), (16383, 8), (600001, 1), (600001, 7), (600001, 8), (600001, 256),
                                 (600001, 257), (600001, 291), (600001, 292), (600001, 293)])
def test_rhs_values(env, n, m):
    pb, torch, ctx = env
    print("case: right-hand side,", n, "nodes,", m, "atoms", flush=True)
    rng = np.random.default_rng(m)
    # atoms away from the nodes, so that no single term swamps the sums
    atoms = np.column_stack([rng.uniform(150.0, 160.0, (m, 3)), np.ones(m), rng.normal(size=m)])
    band = _band(pb, torch, n)
    g = pb.pb_ibim_rhs(ctx, band, torch.tensor(atoms, device="cuda"), pb.params(0.5, eps_in=1.0))
    ref = _formula(torch, band, atoms)
    for a, b in ((g[:n], ref[:n]), (g[n:], ref[n:])):
        assert float((a - b).abs().max()) <= 1e-13 * float(b.abs().max())


def test_one_atom_is_a_copy_in_time(env):
    pb, torch, ctx = env
    import ctypes

    n = 4_000_000
    print("case: time of one atom on", n, "nodes", flush=True)
    band = _band(pb, torch, n)
    at = torch.tensor([[150.0, 150.0, 150.0, 1.0, 1.0]], dtype=torch.float64, device="cuda")
    src, dst = torch.zeros(4 * n, dtype=torch.float64, device="cuda"), torch.empty(4 * n, dtype=torch.float64, device="cuda")
    prm = pb.params(0.5)
    pb.pb_ibim_rhs(ctx, band, at, prm)
    dst.copy_(src)
    pb.lib.pb_set_timing(ctx.handle, 1)
    for _ in range(10):
        pb.pb_ibim_rhs(ctx, band, at, prm)
    ms, launches = ctypes.c_double(), ctypes.c_int64()
    pb.lib.pb_kernel_time(ctx.handle, b"rhs", ctypes.byref(ms), ctypes.byref(launches))
    pb.lib.pb_set_timing(ctx.handle, 0)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(10):
        dst.copy_(src)
    b.record()
    torch.cuda.synchronize()
    kernel, copy = ms.value / launches.value, a.elapsed_time(b) / 10
    print(f"  kernel {kernel * 1e3:.1f} us, copy of as many bytes {copy * 1e3:.1f} us", flush=True)
    assert kernel <= 1.6 * copy
