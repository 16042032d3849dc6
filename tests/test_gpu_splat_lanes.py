"""The exact model's splats where lists are long enough for the forward's block polynomial (one slice,
over a thousand entries a list): amplitudes of both signs and zero, records of the plain, the folded
and the direct form, direct ones set aside from groups of the others, more Gaussians that meet one
half of a block than are kept apart, and Gaussians on the corner of a block, where the series is worst.

Forward bar, per unit of the image of the Gaussians' magnitudes: the limit on folded records (4e-6) and
the FP32 evaluation (2e-6 for Gaussians of a pixel or more); the footprints reach 7 deviations, which
leaves out 2e-11. Gradients: the suite's bars."""
import math

import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import check_grads, dev
from paper_2506_22280_amd import _lib
from splat_ref import bound, reach, record

pytestmark = pytest.mark.gpu

CULL, PLAIN, FOLD = 7.0, 2.0e-6, 4.0e-6
# deviations in pixels at the mean, aspect, pitch (mm); the wanted share of folded and direct records
SCENES = {
    "plain": dict(pitch=0.8, size=(1.5, 4.0), aspect=2.0, folded=(0.0, 0.01), direct=(0.0, 0.01)),
    "folded": dict(pitch=4.6, size=(4.0, 5.0), aspect=1.1, folded=(0.5, 1.0), direct=(0.0, 0.1)),
    "mixed": dict(pitch=1.6, size=(1.0, 3.0), aspect=2.0, folded=(0.02, 1.0), direct=(0.03, 0.1)),
    "halves": dict(pitch=0.4, size=(2.5, 4.0), flat=0.2, folded=(0.0, 0.01), direct=(0.0, 0.01)),
}


def _scene(name, n, nu, nv):
    s = SCENES[name]
    rng = np.random.default_rng(len(name))
    pitch = s["pitch"]
    px = pitch * 1000.0 / 1500.0    # a pixel at the axis (mm)
    half = np.array([0.5 * nu, 0.5 * nu, 0.5 * nv]) * px
    mu = rng.uniform(-1, 1, (3, n)) * half[:, None]
    mu[1] = np.clip(mu[1], -100, 100)
    scale = px * np.exp(rng.uniform(*np.log(s["size"]), n)) * np.ones((3, 1))
    quat = rng.standard_normal((4, n))
    if "flat" in s:                 # thin along the detector's columns
        scale[2] *= s["flat"]
        quat = np.array([1.0, 0.0, 0.0, 0.0])[:, None] * np.ones(n)
    else:
        scale = scale * np.exp(rng.uniform(-0.5, 0.5, (3, n)) * math.log(s["aspect"]))
    rho = rng.uniform(0.2, 1.0, n) / scale[0]
    rho[rng.random(n) < 0.2] *= -1.0
    rho[::50] = 0.0
    return mu, scale, quat, rho, pitch


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


@pytest.mark.parametrize("name", list(SCENES))
def test_long_lists_match_oracle(name):
    print("case: long lists, %s records" % name, flush=True)
    nu, nv, angles = 40, 24, np.array([0.3, 1.9])
    mu, scale, quat, rho, pitch = _scene(name, 6000, nu, nv)
    share = np.zeros(2)
    for a in angles:
        f = record(mu, scale, quat, pitch, a)
        ok, _, _, ru, rv = reach(f, CULL)
        b = np.where(ok, bound(f, ru, rv), np.inf)
        share += np.array([((b > PLAIN) & (b <= FOLD)).mean(), (b > FOLD).mean()]) / len(angles)
    print("folded %.3f, direct %.3f" % tuple(share), flush=True)
    for got, want in zip(share, (SCENES[name]["folded"], SCENES[name]["direct"])):
        assert want[0] <= got <= want[1]
    geom, grid, ins = _still(mu, scale, quat, rho, pitch, angles, nu, nv)
    G = np.random.default_rng(1).normal(0, 1, (2, nv, nu)).astype(np.float32)
    proj, out = _render(geom, grid, ins, G)
    ref = oracle.project(geom, grid, *ins)
    size = oracle.project(geom, grid, *ins[:4], np.abs(ins[4]), *ins[5:])
    err = float((np.abs(proj - ref)).max() / size.max())
    print("forward max err / max magnitude %.2e" % err, flush=True)
    assert err <= 6e-6
    gref = oracle.project_bwd(geom, grid, *ins, grad_proj=G)
    check_grads({k: out[k] for k in gref}, gref)


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


def test_a_vanishing_denominator_stays_with_its_gaussian():
    """Wide, thin sheets among ordinary Gaussians, level with the source's orbit and below it: on the
    rays of the row of block centres at the middle of the detector, which run parallel to them, their
    denominator vanishes, while their values are zero there."""
    print("case: thin level sheets among plain records", flush=True)
    nu, nv, angles = 40, 24, np.array([0.3])
    mu, scale, quat, rho, pitch = _scene("plain", 6000, nu, nv)
    mu[2, ::150], scale[:, ::150] = -20.0, np.array([400.0, 400.0, 1e-4])[:, None]
    quat[:, ::150], rho[::150] = np.array([1.0, 0.0, 0.0, 0.0])[:, None], 1.0
    geom, grid, ins = _still(mu, scale, quat, rho, pitch, angles, nu, nv)
    proj, _ = _render(geom, grid, ins)
    ref = oracle.project(geom, grid, *ins)
    size = oracle.project(geom, grid, *ins[:4], np.abs(ins[4]), *ins[5:])
    assert np.isfinite(proj).all()
    assert np.abs(proj - ref).max() / size.max() <= 6e-6


@pytest.mark.parametrize("pitch,size", [(0.5, 0.25), (0.5, 0.4), (1.5, 0.4)])
def test_narrow_gaussians_keep_the_accuracy_of_the_columns(pitch, size):
    """Gaussians of a fraction of a pixel: the exponent at a block's centre is in the hundreds and must
    cancel at the peak, so the lists that may go by the polynomial are held to what the same Gaussians
    give by forward differences (short lists), half as far again for the chance of two maxima."""
    print("case: Gaussians of %.2f pixels, pitch %.1f mm" % (size, pitch), flush=True)
    nu, nv, n, angles = 40, 24, 8000, np.array([0.3, 1.9])
    rng = np.random.default_rng(11)
    px = pitch * 1000.0 / 1500.0
    mu = rng.uniform(-1, 1, (3, n)) * (0.5 * px * np.array([nu, nu, nv]))[:, None]
    scale = size * px * np.exp(rng.uniform(-0.5, 0.5, (3, n)) * math.log(3.0))
    geom, grid, ins = _still(mu, scale, rng.standard_normal((4, n)), rng.uniform(0.2, 1.0, n), pitch,
                             angles, nu, nv)
    ref = oracle.project(geom, grid, *ins)
    err = [float(np.abs(_render(geom, grid, ins, slices=k)[0] - ref).max() / ref.max())
           for k in (1, 16)]
    print("forward max err / max %.2e, by columns %.2e" % tuple(err), flush=True)
    assert err[0] <= 1.5 * err[1]
