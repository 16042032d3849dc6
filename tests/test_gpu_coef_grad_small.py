"""The control-point gradient's two kernels (a wave per control point at rank 1, 4x4x1 blocks above) on a
lattice of a single point, and a non-finite pixel gradient at rank 1, which must stay with the control
points that its Gaussians reach."""
import numpy as np
import pytest

import oracle
from gpu_helpers import check_grads, oracle_inputs
from test_gpu_coef_grad import _backward, _problem


pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,R", [((1, 1, 1), 2), ((1, 1, 1), 6), ((2, 1, 1), 3)])
def test_single_control_points(dims, R):
    print("case: lattice %s, rank %d" % (dims, R), flush=True)
    p, rng = _problem(dims, R)
    G = rng.normal(0, 1, (2, 48, 48)).astype(np.float32)
    ref = oracle.project_bwd(p.geom, p.grid, *oracle_inputs(p), grad_proj=G)
    out = _backward(p, G)
    check_grads({k: out[k] for k in ref}, ref)


def test_rank_1_keeps_infinities_local():
    print("case: one infinite pixel gradient, rank 1", flush=True)
    dims = (13, 9, 17)
    p, rng = _problem(dims, 1)
    G = rng.normal(0, 1, (2, 48, 48)).astype(np.float32)
    clean = _backward(p, G)["g_coef"].cpu().numpy()
    G[0, 3, 5] = np.inf
    out = _backward(p, G)
    hit = ~np.isfinite(out["g_rho"].cpu().numpy())
    got = out["g_coef"].cpu().numpy()
    bad = ~np.isfinite(got).all(axis=(0, 4))
    assert hit.any() and not hit.all() and bad.any()
    reach = np.zeros_like(bad)
    for i in np.nonzero(hit)[0]:
        c = [int(np.floor((float(p.mu[a, i]) + 24.0) / p.grid["spacing"][a])) for a in range(3)]
        s = [np.unique(np.clip(np.arange(c[a] - 1, c[a] + 3), 0, dims[a] - 1)) for a in range(3)]
        reach[np.ix_(s[2], s[1], s[0])] = True
    assert not (bad & ~reach).any() and not reach.all()
    # elsewhere the sums are those of the finite gradient, added in the same order
    assert np.array_equal(got[:, ~reach], clean[:, ~reach])
