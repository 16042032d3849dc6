"""The normal equations of the temporal-weight fit at the largest views that go whole and the smallest
that are sliced: both entry points, with the workspace that is asked for."""
import numpy as np
import pytest
import torch

from gpu_helpers import dev
from paper_2506_22280_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,R,npix", [(2, 1, 24576), (2, 1, 24577), (3, 4, 12288), (3, 4, 12289)])
def test_lm_whole_and_sliced(T, R, npix):
    print("case: normal equations T=%d R=%d npix=%d" % (T, R, npix), flush=True)
    whole = npix * (R + 2) <= 73728
    assert (_lib.load().digs_lm_workspace_size(T, R, npix) == 0) == whole
    rng = np.random.default_rng(R + npix)
    imgs = rng.normal(0, 1, (T, R + 1, npix)).astype(np.float32)
    meas = rng.normal(0, 1, (T, npix)).astype(np.float32)
    h = np.full(R, 0.25, dtype=np.float32)   # (a power of two: exact)
    I = imgs.astype(np.float64)
    V = np.concatenate([(I[:, 1:] - I[:, :1]) * 4.0, (I[:, 0] - meas)[:, None]], 1)
    iu = np.triu_indices(R)
    terms = lambda G: np.concatenate(   # noqa: E731
        [G[:, iu[0], iu[1]], G[:, :R, R], G[:, R, R][:, None]], 1)
    ref, size = terms(V @ V.transpose(0, 2, 1)), terms(np.abs(V) @ np.abs(V).transpose(0, 2, 1))
    dI, dP, dh = dev(imgs), dev(meas), dev(h)
    out = _lib.lm_normal_eq(dI, dP, dh, R)
    one = torch.empty_like(out)
    ptr = lambda x: x.data_ptr()   # noqa: E731
    s = torch.cuda.current_stream().cuda_stream
    assert _lib.load().digs_lm_normal_eq(T, R, npix, ptr(dI), ptr(dP), ptr(dh), ptr(one), s) == 0
    # each factor is rounded once, each product and sum once; in one piece a sum has npix/256 + 9
    # terms along its longest path, in slices at most 45
    assert np.all(np.abs(one.cpu().numpy() - ref) <= (4 + npix / 256 + 13) * size * 2.0 ** -24)
    if whole:
        assert torch.equal(out, one)
    else:
        assert np.all(np.abs(out.cpu().numpy() - ref) <= (4 + 45) * size * 2.0 ** -24)
