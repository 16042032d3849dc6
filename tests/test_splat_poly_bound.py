"""The bound by which the splats' set-up chooses between the plain, the folded and the direct
evaluation (csrc/splat_poly.h, compiled for the host) against the errors of the series in FP64, over
Gaussians of a sixth of a pixel to six pixels, round and elongated, near the axis and off it, on
detector pitches of 0.4 to 11 mm."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2506_22280_amd import build
from splat_ref import bound, reach, record, series_errors

FIELDS = ("Huu", "Huv", "Hvv", "gu", "gv", "Guu", "Guv", "Gvv")


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    d = tmp_path_factory.mktemp("bound")
    src, lib = str(d / "bound.hip"), str(d / "bound.so")
    with open(src, "w") as fh:
        fh.write('#include "splat_poly.h"\n'
                 'extern "C" void bounds(int n, const float *a, float *out) {\n'
                 '  for (int i = 0; i < n; ++i, a += 10) out[i] = poly_error(\n'
                 '    a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9]);\n}\n')
    subprocess.run([build.HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-shared", "-fPIC",
                    "-I" + build.CSRC, src, "-o", lib], check=True, capture_output=True)
    fn = ctypes.CDLL(lib).bounds

    def run(f, ru, rv):
        a = np.stack([f[k] for k in FIELDS] + [ru, rv], 1).astype(np.float32)
        out = np.empty(len(ru), np.float32)
        fn(len(ru), np.ascontiguousarray(a).ctypes.data_as(ctypes.c_void_p),
           out.ctypes.data_as(ctypes.c_void_p))
        return out.astype(np.float64)

    return run


def _limit(name):
    with open(os.path.join(build.CSRC, "splat_poly.h")) as fh:
        return float(re.search(r"#define %s ([0-9.e-]+)f" % name, fh.read()).group(1))


def _sample(rng, m, pitch, aspect, angle):
    """Records of m Gaussians and the centres of blocks that they meet, half of them at the peak."""
    mu = rng.uniform(-1, 1, (3, m)) * np.array([125.0, 95.0, 128.0])[:, None]
    mu *= rng.choice([0.05, 1.0], m)
    size = pitch * np.exp(rng.uniform(np.log(0.15), np.log(6.0), m))
    scale = size * np.exp(rng.uniform(-0.5, 0.5, (3, m)) * np.log(aspect))
    f = record(mu, scale, rng.standard_normal((4, m)), pitch, angle)
    ok, cu, cv, ru, rv = reach(f)
    f = {k: v[ok] for k, v in f.items()}
    cu, cv, ru, rv = cu[ok], cv[ok], ru[ok], rv[ok]
    far = rng.random(len(cu)) < 0.5
    du = np.where(far, cu + rng.uniform(-1, 1, len(cu)) * (ru - abs(cu)), rng.uniform(-4, 4, len(cu)))
    dv = np.where(far, cv + rng.uniform(-1, 1, len(cu)) * (rv - abs(cv)), rng.uniform(-4, 4, len(cu)))
    return f, ru, rv, du, dv


@pytest.mark.parametrize("pitch", [0.4, 0.8, 1.6, 2.0, 3.0, 4.2, 6.0, 11.0])
@pytest.mark.parametrize("aspect", [1.0, 3.0, 9.0])
def test_bound_holds(compiled, pitch, aspect):
    rng = np.random.default_rng(int(10 * pitch + aspect))
    f, ru, rv, du, dv = _sample(rng, 6000, pitch, aspect, 0.7)
    b = compiled(f, ru, rv)
    assert np.allclose(b, bound(f, ru, rv), rtol=2e-4, atol=0)
    plain, fold = series_errors(f, du, dv)
    # (the bound is to second order: held to it where a series may be used at all, with room to 1e-3)
    use = b <= 1e-3
    assert use.any() and np.all(plain[use] <= b[use])
    folded = b <= _limit("POLY_FOLD")
    assert np.all(fold[folded] <= 0.5 * b[folded] + 1e-12)


def test_bound_reports_a_vanishing_denominator(compiled):
    f = {k: np.array([v]) for k, v in zip(FIELDS, (1e-2, 0.0, 1e-2, 0.05, 0.0, 2.5e-3, 0.0, 0.0))}
    assert not np.isfinite(compiled(f, np.array([12.0]), np.array([12.0])))[0]
