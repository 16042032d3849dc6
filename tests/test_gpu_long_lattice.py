"""The control-point gradient on lattices that are long along one axis: cells past 2^19, and more blocks
of control points than a launch has threads for in one dimension. Bars: the suite's for gradients."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import check_grads, dev
from paper_2506_22280_amd import _lib, synth

pytestmark = pytest.mark.gpu


def _check(dims, origin, R, axis, first, reach):
    """300 Gaussians whose cells along the axis (spacing 1 mm) start at index `first`, their means on a
    grid on which FP32 is exact."""
    n = 300
    rng = np.random.default_rng(R + axis)
    p = synth.tiny(seed=R, n=n, nviews=2, det=48)
    p.grid = dict(R=R, nx=dims[0], ny=dims[1], nz=dims[2], origin=list(origin),
                  spacing=[1.0 if a == axis else 40.0 for a in range(3)])
    p.mu[axis] = origin[axis] + first + rng.integers(0, 16 * reach, n) / 16.0
    p.coef = np.zeros((R, dims[2], dims[1], dims[0], 3), np.float32)
    part = [slice(None)] * 5
    part[3 - axis] = slice(max(first - 4, 0), first + reach + 4)
    p.coef[tuple(part)] = rng.normal(0, 0.05, p.coef[tuple(part)].shape)
    p.w = rng.normal(0, 1, (2, R)).astype(np.float32)
    G = rng.normal(0, 1, (2, 48, 48)).astype(np.float32)
    ins = (p.coef, p.mu, p.scale, p.quat, p.rho, p.angles, p.w)
    args = (p.geom, p.grid) + tuple(dev(a) for a in ins)
    ws = _lib.Workspace("cuda")
    _lib.project_fwd(*args, ws)
    out = _lib.project_bwd(*args, dev(G), ws, reuse_fwd=True)
    torch.cuda.synchronize()
    assert ws.diagnostics()["overflow"] == 0
    ref = oracle.project_bwd(p.geom, p.grid, *ins, grad_proj=G)
    assert np.abs(ref["g_coef"]).max() > 0
    check_grads({k: out[k] for k in ref}, ref)


@pytest.mark.parametrize("R", [1, 2])
def test_cells_past_2_to_the_19(R):
    print("case: 600000 control points along x, rank %d" % R, flush=True)
    nx = 600000
    _check((nx, 1, 1), (32.0 - nx, 0.0, 0.0), R, 0, nx - 64, 60)


@pytest.mark.parametrize("dims,axis", [((1, 1, (1 << 23) + 72), 2), ((4100, 4100, 1), 1)])
def test_blocks_past_2_to_the_32_threads(dims, axis):
    print("case: lattice of %d x %d x %d control points" % dims, flush=True)
    origin = [0.0, 0.0, 0.0]
    origin[axis] = -32.0
    _check(dims, origin, 2, axis, 4, 60)
