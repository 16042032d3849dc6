"""The dynamic volume at the edges of its bricks and of the recurrence along z: ragged grids, needles
and pancakes in any direction, deviations on both sides of the recurrence's limit (0.85 voxels)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import dev
from paper_2506_22280_amd import _lib, synth

pytestmark = pytest.mark.gpu


# deviations in voxels (lowest, highest): all direct, on both sides, all by the recurrence, needles
# (each axis drawn by itself)
@pytest.mark.parametrize("dims", [(8, 8, 8), (9, 17, 3), (33, 7, 12)])
@pytest.mark.parametrize("lo,hi", [(0.15, 0.5), (0.7, 1.0), (1.0, 5.0), (0.1, 6.0)])
def test_phi_shapes(dims, lo, hi):
    print("case: phi %s, deviations %g to %g voxels" % (dims, lo, hi), flush=True)
    rng = np.random.default_rng(int(100 * lo) + dims[0])
    n, h = 70, 1.5
    d = np.array(dims)
    v = dict(nx=dims[0], ny=dims[1], nz=dims[2], origin=[-5.0, 3.0, -9.0], spacing=[h] * 3)
    pos = rng.uniform(-2.0, d + 1.0, (n, 3))
    f32 = lambda x: np.ascontiguousarray(x, dtype=np.float32)   # noqa: E731
    mu = f32((np.array(v["origin"]) + h * pos).T)
    scale = f32(h * np.exp(rng.uniform(np.log(lo), np.log(hi), (3, n))))
    quat, rho = f32(rng.normal(0, 1, (4, n))), f32(rng.uniform(0.2, 1.0, n))
    p = synth.small_phantom(seed=1)
    phi = _lib.phi_grid(p.grid, dev(p.coef), dev(mu), dev(scale), dev(quat), dev(rho),
                        torch.zeros(p.grid["R"], device="cuda"), v, _lib.Workspace())
    ix = np.stack(np.meshgrid(*[np.arange(k) for k in dims], indexing="ij"), -1).reshape(-1, 3)
    x = np.array(v["origin"]) + h * ix
    eps = 2.0 ** -24
    moved = 4 * eps * (np.abs(mu).max() + 9.0)   # roundings of the centre in voxel units
    ref, bar = np.zeros(len(ix)), np.zeros(len(ix))
    for i in range(n):
        W = np.linalg.inv(_factor(scale[:, i], quat[:, i]))
        aW, dx = np.abs(W), x - mu[:, i].astype(np.float64)
        u = dx @ W.T
        e = 0.5 * (u ** 2).sum(1)
        val = rho[i] * np.exp(-e)
        ref += val
        # beyond 5 deviations along an axis a voxel may be left out
        bar += np.where(e > 12.49, val, 0.0)
        # the exponent is a sum of products of up to this size (its start three voxels off), each
        # through at most 40 roundings from the parameters to the value; 16 more outside it
        size = 0.5 * (((np.abs(dx) + [0, 0, 3 * h]) @ aW.T) ** 2).sum(1)
        bar += val * ((40 * size + 16) * eps + (np.abs(u) @ aW.sum(1)) * moved)
    err = np.abs(phi.cpu().numpy().reshape(dims[::-1]).transpose(2, 1, 0).ravel() - ref)
    assert np.all(err <= bar + 1e-30), (err / (bar + 1e-30)).max()


def _factor(scale, quat):
    """M with Sigma = M M^T: the rotation times the deviations."""
    w, x, y, z = quat.astype(np.float64) / np.linalg.norm(quat.astype(np.float64))
    R = np.array([[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
                  [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
                  [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]])
    return R * scale.astype(np.float64)


@pytest.mark.parametrize("R", [1, 3, 8])
def test_phi_lattice_combined_or_not(R):
    """The ranks combined once per lattice point, or per Gaussian where the workspace is too small for
    that: both against the oracle's warp. Bar: the suite's for volumes."""
    print("case: phi, rank %d, combined lattice and not" % R, flush=True)
    p = synth.lung_phantom("phi", 40, 32, 32, 8.0, 2, min(R, 3), 25.0, 3)
    p.grid["R"], p.coef = R, np.concatenate([p.coef] * 3)[:R]   # (the phantom has few modes)
    v = dict(nx=21, ny=19, nz=23, origin=[-100.0, -90.0, -110.0], spacing=[10.0] * 3)
    w = np.random.default_rng(R).normal(0, 0.5, R).astype(np.float32)
    mu_t, cov_t = oracle.deform(p.grid, p.coef, p.mu, p.scale, p.quat, w[None])
    z, y, x = np.meshgrid(*[np.arange(v[k]) for k in ("nz", "ny", "nx")], indexing="ij")
    pts = np.stack([v["origin"][a] + 10.0 * q.ravel() for a, q in enumerate((x, y, z))])
    ref = oracle.phi(mu_t[0], cov_t[0], p.rho, pts)
    args = (p.grid, dev(p.coef), dev(p.mu), dev(p.scale), dev(p.quat), dev(p.rho), dev(w), v)
    ws = _lib.Workspace()
    got = [_lib.phi_grid(*args, ws, capacity=c, grow=False).cpu().numpy().ravel()
           for c in (40 * 27, 1 << 16)]
    points = p.grid["nx"] * p.grid["ny"] * p.grid["nz"]
    assert 40 * 27 * 8 + 512 < 16 * points <= (1 << 16) * 8, points
    assert ws.diagnostics()["instances"] <= 40 * 27
    for g in got:
        assert np.abs(g - ref).max() <= 1e-4 * np.abs(ref).max()
