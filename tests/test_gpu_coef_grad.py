"""The control-point gradient where its 4x4x1 blocks of control points end: lattices smaller than a
block, one point past it, Gaussians outside the lattice (whose weights the end points collect), one
and two tiles of rank components, both numbers of waves. Bars: the suite's for gradients."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import check_grads, dev, oracle_inputs, problem_tensors
from paper_2506_22280_amd import _lib, synth

pytestmark = pytest.mark.gpu


def _problem(dims, R, n=400):
    p = synth.tiny(seed=R, n=n, nviews=2, det=48)
    rng = np.random.default_rng(R + dims[0])
    # the Gaussians fill +-32 mm, the lattice about +-24
    h = [48.0 / max(d - 1, 1) for d in dims]
    p.grid = dict(R=R, nx=dims[0], ny=dims[1], nz=dims[2], origin=[-24.0] * 3, spacing=h)
    p.coef = rng.normal(0, 0.05 * min(h), (R, dims[2], dims[1], dims[0], 3)).astype(np.float32)
    p.w = rng.normal(0, 1, (2, R)).astype(np.float32)
    return p, rng


def _backward(p, G):
    t = problem_tensors(p)
    args = (p.geom, p.grid, t["coef"], t["mu"], t["scale"], t["quat"], t["rho"], t["angles"],
            t["w"])
    ws = _lib.Workspace("cuda")
    _lib.project_fwd(*args, ws)
    out = _lib.project_bwd(*args, dev(G), ws, reuse_fwd=True)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("dims,R", [((1, 1, 1), 1), ((3, 4, 5), 5), ((4, 5, 9), 6), ((5, 3, 2), 8),
                                    ((13, 9, 17), 3), ((41, 38, 11), 2)])
def test_coef_grad_blocks(dims, R):
    print("case: coefficient gradient, lattice %s, rank %d" % (dims, R), flush=True)
    p, rng = _problem(dims, R)
    G = rng.normal(0, 1, (2, 48, 48)).astype(np.float32)
    ref = oracle.project_bwd(p.geom, p.grid, *oracle_inputs(p), grad_proj=G)
    out = _backward(p, G)
    check_grads({k: out[k] for k in ref}, ref)


@pytest.mark.parametrize("R", [3, 6])
def test_coef_grad_keeps_infinities_local(R):
    print("case: one infinite pixel gradient, rank %d" % R, flush=True)
    p, rng = _problem((13, 9, 17), R)
    G = rng.normal(0, 1, (2, 48, 48)).astype(np.float32)
    G[0, 3, 5] = np.inf
    out = _backward(p, G)
    hit = ~np.isfinite(out["g_rho"].cpu().numpy())
    bad = ~np.isfinite(out["g_coef"].cpu().numpy()).all(axis=(0, 4))
    assert hit.any() and not hit.all() and bad.any()
    reach = np.zeros_like(bad)
    dims = (13, 9, 17)
    for i in np.nonzero(hit)[0]:
        c = [int(np.floor((float(p.mu[a, i]) + 24.0) / p.grid["spacing"][a])) for a in range(3)]
        s = [np.unique(np.clip(np.arange(c[a] - 1, c[a] + 3), 0, dims[a] - 1)) for a in range(3)]
        reach[np.ix_(s[2], s[1], s[0])] = True
    assert not (bad & ~reach).any() and not reach.all()
