"""The normal equations of the temporal-weight fit at the edges of their slices: one slice and
several, remainders of four pixels, and the entry point without a workspace."""
import numpy as np
import pytest
import torch

from gpu_helpers import dev
from paper_2506_22280_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,R,npix", [(1, 1, 1), (3, 2, 7), (2, 8, 4096), (2, 3, 4097), (1, 4, 4095),
                                      (3, 5, 12291), (1, 2, 300001)])
def test_lm_normal_eq_slices(T, R, npix):
    print("case: normal equations T=%d R=%d npix=%d" % (T, R, npix), flush=True)
    rng = np.random.default_rng(T + R + npix)
    imgs = rng.normal(0, 1, (T, R + 1, npix)).astype(np.float32)
    meas = rng.normal(0, 1, (T, npix)).astype(np.float32)
    h = np.full(R, 0.25, dtype=np.float32)   # (a power of two: exact)
    I = imgs.astype(np.float64)
    V = np.concatenate([(I[:, 1:] - I[:, :1]) * 4.0, (I[:, 0] - meas)[:, None]], 1)
    iu = np.triu_indices(R)
    terms = lambda G: np.concatenate(   # noqa: E731
        [G[:, iu[0], iu[1]], G[:, :R, R], G[:, R, R][:, None]], 1)
    ref = terms(V @ V.transpose(0, 2, 1))
    # each factor is rounded once, each product and sum once; a sum has at most 21 + 24 + npix/65536
    # terms along any path in slices (4 x 4 pixels and a remainder per thread, the trees, the
    # slices), npix/256 + 9 in one
    size = terms(np.abs(V) @ np.abs(V).transpose(0, 2, 1)) * 2.0 ** -24
    dI, dP, dh = dev(imgs), dev(meas), dev(h)
    out = _lib.lm_normal_eq(dI, dP, dh, R)
    assert np.all(np.abs(out.cpu().numpy() - ref) <= (4 + 45 + npix / 65536) * size)
    one = torch.empty_like(out)
    ptr = lambda x: x.data_ptr()   # noqa: E731
    s = torch.cuda.current_stream().cuda_stream
    assert _lib.load().digs_lm_normal_eq(T, R, npix, ptr(dI), ptr(dP), ptr(dh), ptr(one), s) == 0
    assert np.all(np.abs(one.cpu().numpy() - ref) <= (4 + npix / 256 + 9 + 4) * size)
    # a view's result does not depend on the others in the call
    last = _lib.lm_normal_eq(dI[-1:].clone(), dP[-1:].clone(), dh, R)
    assert torch.equal(out[-1:], last)
