"""GPU: the band compaction's lists at the edges of its tiles of 4096 nodes and words of 64, against
numpy: less than one tile, exactly one, a partial last one; every interior node in the band (full
words and tiles) and one in a hundred (mostly empty). Indices and values are equal; points and normals
(central differences) differ by the rounding of one division and root: bar 1e-13 relative to the box.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pbm():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb

    return pb


@pytest.mark.parametrize("share", [1.0, 0.01])
@pytest.mark.parametrize("dims", [(5, 7, 9), (16, 16, 16), (3, 3, 700), (33, 17, 67)], ids=str)
def test_band_lists(pbm, dims, share):
    import torch

    h = 0.5
    print("case: band lists", dims, share, flush=True)
    rng = np.random.default_rng(int(1000 * share) + sum(dims))
    inside = np.zeros(dims, bool)
    inside[1:-1, 1:-1, 1:-1] = rng.random(tuple(d - 2 for d in dims)) < share
    inside[1, 1, 1] = True
    phi = np.where(inside, rng.uniform(-0.9, 0.9, dims), 5.0 + rng.random(dims))
    prm = pbm.params(h, grad_scheme=pbm.PB_GRAD_CENTRAL)
    eps = prm.band_k * h
    grid = pbm.pb_grid()
    grid.nx, grid.ny, grid.nz = dims
    grid.h = h
    origin = np.array([-1.0, 2.0, 0.25])
    for c in range(3):
        grid.origin[c] = origin[c]
    ctx = pbm.Context(0)
    band = pbm.pb_narrowband_compact(ctx, grid, torch.tensor(phi.ravel(), device="cuda"), prm)
    ctx.close()
    idx = np.flatnonzero(np.abs(phi.ravel()) < eps)
    assert band.n == len(idx)
    np.testing.assert_array_equal(band.gidx[: band.n].cpu().numpy(), idx)
    ijk = np.stack(np.unravel_index(idx, dims), 1)
    f = phi.ravel()[idx]
    g = np.stack([(phi[tuple((ijk + e).T)] - phi[tuple((ijk - e).T)]) / (2 * h) for e in np.eye(3, dtype=int)], 1)
    n = g / np.linalg.norm(g, axis=1)[:, None]
    t = band.table()
    np.testing.assert_allclose(t[:, 3:6], n, rtol=0, atol=1e-13)
    np.testing.assert_allclose(t[:, :3], origin + h * ijk - f[:, None] * n, rtol=0, atol=1e-13 * h * max(dims))


@pytest.mark.parametrize("what", ["short by one", "node on the edge", "no gradient", "empty"])
def test_band_refusals(pbm, what):
    """The count and the error flags come back together with the nodes: a band that does not fit leaves the
    arrays alone and reports its size; a good call after each refusal returns the band."""
    import torch

    dims, h = (33, 17, 67), 0.5
    rng = np.random.default_rng(3)
    good = np.full(dims, 5.0)
    good[2:-2, 2:-2, 2:-2] = rng.uniform(-0.9, 0.9, tuple(d - 4 for d in dims))
    phi = good.copy()
    if what == "node on the edge":
        phi[0, 5, 5] = 0.1
    elif what == "no gradient":
        phi[8:13, 6:11, 20:25] = 0.3
    elif what == "empty":
        phi[:] = 5.0
    prm = pbm.params(h, grad_scheme=pbm.PB_GRAD_CENTRAL)
    grid = pbm.pb_grid()
    grid.nx, grid.ny, grid.nz = dims
    grid.h = h
    print("case: band refusal,", what, flush=True)
    ctx = pbm.Context(0)
    n = int(np.count_nonzero(np.abs(good) < prm.band_k * h))
    band = pbm.Band.alloc(n - 1 if what == "short by one" else n + 30, "cuda")
    band.px.fill_(7.0)
    with pytest.raises(pbm.PBError) as e:
        pbm.pb_narrowband_compact(ctx, grid, torch.tensor(phi.ravel(), device="cuda"), prm, band)
    if what == "short by one":
        assert e.value.status == pbm.PB_ECAPACITY and f"needs {n} nodes" in str(e.value)
        assert bool((band.px == 7.0).all())
    else:
        assert e.value.status == pbm.PB_EGEOM
    assert pbm.pb_narrowband_compact(ctx, grid, torch.tensor(good.ravel(), device="cuda"), prm).n == n
    ctx.close()
