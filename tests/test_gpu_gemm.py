"""The matrix products and column sums of the warm-start network at the edges of their tiles and of
their dispatch: remainders of rows, columns and K, one, four and sixteen waves over K, narrow and
wide tiles, and operands that start at an address that is a multiple of four bytes only."""
import numpy as np
import pytest
import torch

from gpu_helpers import dev
from paper_2506_22280_amd import _lib

pytestmark = pytest.mark.gpu


def _bf16(x):
    return torch.from_numpy(x).bfloat16().double().numpy()


def _odd(x):
    """x on the device, one float past an aligned address, and the buffer around it."""
    w = torch.zeros(x.size + 9, device="cuda")
    w[1:1 + x.size] = dev(x.ravel())
    return w[1:1 + x.size].view(x.shape), w


# narrow tiles with 1, 4, 16 waves over K, wide with 1, 4, 16
@pytest.mark.parametrize("M,N,K", [(17, 5, 31), (33, 100, 257), (16, 3, 1061),
                                   (8197, 257, 33), (4130, 66, 300), (1009, 70, 1055)])
def test_gemm_tiles(M, N, K):
    print("case: gemm tiles M=%d N=%d K=%d" % (M, N, K), flush=True)
    rng = np.random.default_rng(M + N + K)
    f = lambda *s: rng.normal(0, 1, s).astype(np.float32)   # noqa: E731
    A, B, C0, bias, gate = f(M, K), f(K, N), f(M, N), f(N), f(M, N)
    prod, mag = _bf16(A) @ _bf16(B), np.abs(_bf16(A)) @ np.abs(_bf16(B))
    ref = np.where(gate > 0, np.maximum(prod + C0 + bias, 0.0), 0.0)
    # products of BF16 values are exact in FP32; K + 2 FP32 additions in any order, each rounded
    # or truncated
    bar = (K + 3) * 2.0 ** -23 * (mag + np.abs(C0) + np.abs(bias))
    for ta in (False, True):
        for tb in (False, True):
            dA, dB = _odd(A.T.copy() if ta else A)[0], _odd(B.T.copy() if tb else B)[0]
            C, around = _odd(C0)
            _lib.gemm_bf16(dA, dB, C, transA=ta, transB=tb, bias=dev(bias), accumulate=True,
                           relu=True, gate=_odd(gate)[0])
            assert np.all(np.abs(C.cpu().numpy() - ref) <= bar), (ta, tb)
            assert not around[0].item() and not around[1 + M * N:].any().item()


@pytest.mark.parametrize("M,N", [(1, 1), (15, 63), (17, 65), (300, 200)])
def test_colsum_rows_and_columns(M, N):
    print("case: colsum M=%d N=%d" % (M, N), flush=True)
    X = np.random.default_rng(M + N).normal(0, 1, (M, N)).astype(np.float32)
    out = _lib.colsum(_odd(X)[0], torch.full((N,), 7.0, device="cuda")).cpu().numpy()
    ref, mag = X.astype(np.float64).sum(0), np.abs(X.astype(np.float64)).sum(0)
    assert np.all(np.abs(out - ref) <= M * 2.0 ** -24 * mag)
