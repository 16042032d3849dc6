"""FP64 reference of the splats' block polynomial (csrc/splat_poly.h): a Gaussian's record on the
detector, its series over an 8x8 block by division of the quadratics, and the bound on the plain
series' error."""
import math

import numpy as np

HL = 0.5 / math.log(2.0)
S, T = np.meshgrid(np.arange(8) - 3.5, np.arange(8) - 3.5, indexing="ij")   # pixels about the centre


def record(mu, scale, quat, pitch, angle, sid=1000.0, sdd=1500.0):
    """H, g, G of undeformed Gaussians: q = 1 + 2 g.d + d^T G d, E = d^T H d in pixels from (us, vs)."""
    w, x, y, z = quat / np.linalg.norm(quat, axis=0)
    R = np.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                  2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                  2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)])
    W = R.reshape(3, 3, -1).transpose(2, 1, 0) / scale.T[:, :, None]
    ct, st = math.cos(angle), math.sin(angle)
    m = np.array([sid * ct, sid * st, 0.0])[None] - mu.T
    beta = (sid - (ct * mu[0] + st * mu[1])) / sdd
    dot = lambda a, b: (a * b).sum(1)   # noqa: E731
    mw = np.einsum("nij,nj->ni", W, m)
    Du, Dv = pitch * (-st * W[:, :, 0] + ct * W[:, :, 1]), pitch * W[:, :, 2]
    c = dot(mw, mw)
    pa, pb = dot(mw, Du) / c, dot(mw, Dv) / c
    Dup, Dvp, k = Du - pa[:, None] * mw, Dv - pb[:, None] * mw, beta * beta
    return dict(Huu=k * dot(Dup, Dup), Huv=k * dot(Dup, Dvp), Hvv=k * dot(Dvp, Dvp),
                gu=-beta * pa, gv=-beta * pb,
                Guu=k * dot(Du, Du) / c, Guv=k * dot(Du, Dv) / c, Gvv=k * dot(Dv, Dv) / c)


def reach(f, cull=5.0):
    """Whether the cut-off footprint is an ellipse, its centre, and how far from the mean the blocks
    that it meets may have theirs."""
    r2 = cull * cull
    b00, b01, b11 = (f["H" + k] - r2 * f["G" + k] for k in ("uu", "uv", "vv"))
    det = b00 * b11 - b01 * b01
    ok = (b00 > 0) & (det > 0)
    det = np.where(ok, det, 1.0)
    cu = r2 * (b11 * f["gu"] - b01 * f["gv"]) / det
    cv = r2 * (b00 * f["gv"] - b01 * f["gu"]) / det
    k2 = r2 + (f["gu"] * cu + f["gv"] * cv) * r2
    hu, hv = np.sqrt(np.maximum(k2 * b11 / det, 0)), np.sqrt(np.maximum(k2 * b00 / det, 0))
    return ok, cu, cv, abs(cu) + hu + 4.0, abs(cv) + hv + 4.0


def bound(f, ru, rv):
    """The bound on the plain series' error in units of the Gaussian's peak."""
    q = 1.0 - 2.0 * (abs(f["gu"]) * ru + abs(f["gv"]) * rv)
    iq = np.where(q > 0.5, 1.0 / np.where(q > 0.5, q, 1.0), np.inf)
    el = 7.0 * iq * (abs(f["gu"]) + abs(f["gv"]) + f["Guu"] * ru + abs(f["Guv"]) * (ru + rv) +
                     f["Gvv"] * rv)
    c = 12.25 * iq * (f["Guu"] + 2 * abs(f["Guv"]) + f["Gvv"])
    rho2 = 12.25 * iq * (f["Huu"] + 2 * abs(f["Huv"]) + f["Hvv"])
    return (0.5 * (rho2 + 0.5) * (el ** 3 + 2 * el * c + c * c) +
            (rho2 + 0.61 * np.sqrt(rho2)) * c * c)


def series_errors(f, du, dv):
    """Largest errors, in units of the peak, of the plain and the folded series over the block whose
    centre lies (du, dv) from the mean."""
    E = {(2, 0): -HL * f["Huu"], (1, 1): -2 * HL * f["Huv"], (0, 2): -HL * f["Hvv"]}
    Q = {(2, 0): f["Guu"], (1, 1): 2 * f["Guv"], (0, 2): f["Gvv"], (1, 0): 2 * f["gu"],
         (0, 1): 2 * f["gv"], (0, 0): np.ones_like(du)}

    def shift(p):   # the quadratic about the block's centre
        a, b, c = p[2, 0], p[1, 1], p[0, 2]
        d, e, o = (p.get(k, 0.0) for k in ((1, 0), (0, 1), (0, 0)))
        return {(2, 0): a, (1, 1): b, (0, 2): c, (1, 0): d + 2 * a * du + b * dv,
                (0, 1): e + 2 * c * dv + b * du,
                (0, 0): o + d * du + e * dv + a * du * du + b * du * dv + c * dv * dv}

    E, Q = shift(E), shift(Q)
    q00 = Q[0, 0]
    p = {k: v / q00 for k, v in Q.items() if k != (0, 0)}

    def divide(num, upto):   # num / (1 + p), degree by degree
        y = {}
        for d in range(upto + 1):
            for j in range(d + 1):
                i = d - j
                y[i, j] = num.get((i, j), 0.0 * du) - sum(
                    v * y[i - a, j - b] for (a, b), v in p.items() if i >= a and j >= b)
        return y

    y = divide({k: v / q00 for k, v in E.items()}, 5)
    # log2(1 + p) / 2 by its derivative along the ray: d/dr log(1 + p) = p' / (1 + p), p' = sum k p_k
    lg = divide({k: sum(k) * v for k, v in p.items()}, 5)
    lg = {k: HL * v / max(sum(k), 1) for k, v in lg.items()}
    base = -0.5 * np.log2(q00)
    plain = {k: y[k] - (lg[k] if 0 < sum(k) <= 2 else 0.0) for k in y if sum(k) <= 4}
    fold = {k: y[k] - (lg[k] if 0 < sum(k) <= 3 else 0.0) for k in y if sum(k) <= 4}
    for i, j, into in ((5, 0, {(3, 0): 15.5, (1, 0): -47.3125}),
                       (4, 1, {(2, 1): 12.5, (0, 1): -21.0625}),
                       (3, 2, {(1, 2): 9.25, (3, 0): 6.375, (1, 0): -58.96875})):
        for k, v in into.items():
            fold[k] = fold[k] + v * y[i, j]
            fold[k[::-1]] = fold[k[::-1]] + v * y[j, i]
    at = lambda P: sum(v[:, None, None] * S ** i * T ** j for (i, j), v in P.items())   # noqa: E731
    exact = at(E) / at(Q) - 0.5 * np.log2(at(Q))
    out = []
    for P in (plain, fold):
        err = abs(np.exp2(at(P) + base[:, None, None]) - np.exp2(exact))
        out.append(err.reshape(len(du), -1).max(1))
    return out
