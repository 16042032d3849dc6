"""The exact model's forward splat by the block polynomial for Gaussians on the corner of a block, where
the series is worst, against the same Gaussians by forward differences (lists cut into slices too short
for the polynomial)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import dev
from paper_2506_22280_amd import _lib

pytestmark = pytest.mark.gpu

CULL = 7.0


def _still(mu, scale, quat, rho, pitch, angles, nu, nv):
    """A scene without motion: geometry, lattice (one cell across all depths) and inputs."""
    geom = dict(sid=1000.0, sdd=1500.0, nu=nu, nv=nv, pitch_u=pitch, pitch_v=pitch, off_u=0.0,
                off_v=0.0)
    grid = dict(R=1, nx=4, ny=4, nz=4, origin=[-900.0] * 3, spacing=[600.0] * 3)
    f = lambda a: np.ascontiguousarray(a, dtype=np.float32)   # noqa: E731
    return geom, grid, (f(np.zeros((1, 4, 4, 4, 3))), f(mu), f(scale), f(quat), f(rho), f(angles),
                        f(np.zeros((len(angles), 1))))


def _render(geom, grid, ins, G=None, entries=None, **tuning):
    t = [dev(a) for a in ins]
    n, T = ins[1].shape[1], len(ins[5])
    tuning = dict(dict(slices=1, cull_radius=CULL, capacity=n * T * 60), **tuning)
    ws = _lib.Workspace("cuda")
    proj = _lib.project_fwd(geom, grid, *t, ws, tuning=tuning)
    out = None if G is None else _lib.project_bwd(geom, grid, *t, dev(G), ws, tuning=tuning,
                                                  reuse_fwd=True)
    torch.cuda.synchronize()
    diag = ws.diagnostics()
    assert diag["overflow"] == 0 and diag["nonfinite"] == 0
    # (so that a list has a thousand entries at least)
    tiles = ((geom["nu"] + 15) // 16) * ((geom["nv"] + 15) // 16)
    assert diag["instances"] >= (entries or 1000 * T * tiles)
    return proj.cpu().numpy(), out


# next to the axis: round footprints, whose q has hardly a gradient but a curvature. The plain series
# is off by 5.3e-5, 5.6e-5, 7.4e-5, 7.4e-6 and 7.3e-7 of the peak there.
@pytest.mark.parametrize("pitch,size", [(4.34, 0.67), (5.0, 1.0), (6.0, 1.5), (4.5, 2.0),
                                        (3.0, 2.0)])
def test_gaussians_on_a_block_corner(pitch, size):
    print("case: %.2f mm Gaussians on a block's corner, pitch %.2f mm" % (size, pitch), flush=True)
    n, nu, nv = 512, 32, 32
    px = pitch * 1000.0 / 1500.0    # the means meet the detector at column 15, row 16
    rng = np.random.default_rng(3)
    mu = np.stack([rng.uniform(-30, 30, n), -0.5 * px * np.ones(n), 0.5 * px * np.ones(n)])
    mu[1:] *= (1000.0 - mu[0]) / 1000.0
    geom, grid, ins = _still(mu, np.full((3, n), size), rng.standard_normal((4, n)), np.ones(n),
                             pitch, np.array([0.0]), nu, nv)
    lanes = _render(geom, grid, ins, entries=n, cull_radius=5.0)[0]   # one list of them all
    # lists of 32: forward differences
    columns = _render(geom, grid, ins, entries=n, cull_radius=5.0, slices=16)[0]
    ref = oracle.project(geom, grid, *ins)
    err = [float(np.abs(x - ref).max() / ref.max()) for x in (lanes, columns, lanes - columns + ref)]
    print("forward max err / max %.2e, by columns %.2e, between them %.2e" % tuple(err), flush=True)
    # the limit on folded records, and at most 60 additions in turn on each side
    assert err[2] <= 4e-6 + 60 * 2.0 ** -24
