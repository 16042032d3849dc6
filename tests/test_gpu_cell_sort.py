"""The cell sort where its passes change form: one block of Gaussians, the last number of blocks whose
counts the passes sum themselves and the first that they scan, one, two and three digits of keys. The
gradients say which Gaussian stood where: every group against the same problem with its Gaussians
in another order, which only changes the order of sums."""
import numpy as np
import pytest
import torch

from gpu_helpers import check_grads, dev
from paper_2506_22280_amd import _lib, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 1025, 96 * 1024, 96 * 1024 + 1])
@pytest.mark.parametrize("points", [2, 16, 40])
def test_cell_sort_orders(n, points):
    print("case: cell sort, %d Gaussians, %d^3 control points" % (n, points), flush=True)
    rng = np.random.default_rng(n + points)
    R, h = 1, 60.0 / (points - 1)
    grid = dict(R=R, nx=points, ny=points, nz=points, origin=[-30.0] * 3, spacing=[h] * 3)
    coef = rng.normal(0, 0.05 * h, (R, points, points, points, 3))
    mu = rng.uniform(-33.0, 33.0, (3, n))
    scale = rng.uniform(0.5, 1.0, (3, n))
    quat, rho = rng.normal(0, 1, (4, n)), rng.uniform(0.2, 1.0, n)
    geom = synth.geometry(24, 24, 5.0)
    G = rng.normal(0, 1, (1, 24, 24))
    angles, w = np.array([0.4]), rng.normal(0, 1, (1, R))

    def grads(order):
        args = (geom, grid, dev(coef), dev(mu[:, order]), dev(scale[:, order]),
                dev(quat[:, order]), dev(rho[order]), dev(angles), dev(w))
        ws = _lib.Workspace("cuda")
        proj = _lib.project_fwd(*args, ws)
        out = _lib.project_bwd(*args, dev(G), ws, reuse_fwd=True)
        torch.cuda.synchronize()
        assert ws.diagnostics()["overflow"] == 0
        back = np.argsort(order)
        res = {k: v.cpu().numpy() for k, v in out.items() if v is not None}
        for k in ("g_mu", "g_scale", "g_quat"):
            res[k] = res[k][:, back]
        res["g_rho"] = res["g_rho"][back]
        res["proj"] = proj.cpu().numpy()
        return res

    check_grads(grads(rng.permutation(n)), grads(np.arange(n)))
