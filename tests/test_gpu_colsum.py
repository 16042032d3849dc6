"""The column sums on both sides of their dispatch: the last numbers of rows and columns that a
thread per column takes and the first that sixteen waves share, and more columns than a launch has
threads for those."""
import pytest
import torch

from paper_2506_22280_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N", [(1, 257), (63, 1 << 16), (64, (1 << 16) + 1), (65, 63),
                                 (1, (1 << 16) + 1), (63, 1 << 18),
                                 (64, (1 << 28) + 1)])
def test_colsum_dispatch(M, N):
    print("case: colsum M=%d N=%d" % (M, N), flush=True)
    # whole numbers: every order of the sums is exact
    if M * N < 1 << 28:
        X = torch.randint(-8, 9, (M, N), device="cuda").float()
        ref = X.sum(0)
    else:
        X = (torch.arange(N, device="cuda") % 7).float().expand(M, N).contiguous()
        ref = X[0] * M
    out = _lib.colsum(X, torch.full((N,), 7.0, device="cuda"))
    assert torch.equal(out, ref)
