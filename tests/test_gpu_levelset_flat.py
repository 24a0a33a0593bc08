"""GPU: the level set's stages on flat grids take no more time per node than on others.

A flat grid and a compact one of about as many nodes, one molecule; the best of three calls each.
Bar: 1.4 times the other's time per node. The stages of both do the same work per node, the reflected ghosts
of a short axis cost index arithmetic only, and clocks differ by a few percent; lanes without a node or
one XCD with twice the rows show as 1.5 and more.
"""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1709_08070_amd import pb, synth

    return pb, torch, pb.Context(0), synth.born_ion()


def _time_per_node(env, dims):
    pb, torch, ctx, atoms = env
    grid = pb.pb_grid()
    grid.nx, grid.ny, grid.nz = dims
    grid.h = 0.5
    for c in range(3):
        grid.origin[c] = -0.25 * dims[c]
    at = torch.tensor(atoms, device="cuda")
    best = np.inf
    for _ in range(4):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        pb.pb_build_levelset(ctx, at, pb.params(0.5), grid)
        best = min(best, time.perf_counter() - t0)
    return best / np.prod(dims)


@pytest.mark.parametrize("flat,compact", [((620, 610, 7), (16, 410, 400)), ((300, 260, 34), (16, 410, 400)),
                                          ((300, 9, 300), (300, 300, 9))],
                         ids=str)
def test_flat_grids(env, flat, compact):
    print("case: level set times", flat, compact, flush=True)
    a, b = _time_per_node(env, flat), _time_per_node(env, compact)
    print(f"  {a * 1e9:.3f} and {b * 1e9:.3f} ns a node", flush=True)
    assert a <= 1.4 * b
