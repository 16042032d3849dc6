"""The matrix products where their dispatch leaves the network's sizes: fewer waves over K as the tiles
of C fill the chip, tiles down the columns of C, tiles staged through LDS (B transposed, or the shortest
K), remainders of each, and a result of 2^32 numbers."""
import numpy as np
import pytest
import torch

from paper_2506_22280_amd import _lib

pytestmark = pytest.mark.gpu


def _operands(M, N, K, ta, tb, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    f = lambda *s: torch.randn(s, generator=g, device="cuda")   # noqa: E731
    return f(*((K, M) if ta else (M, K))), f(*((N, K) if tb else (K, N))), f


# direct: at most 4 waves and one over K, down the columns; staged (B transposed): each limit of K and
# past the last; staged for the shortest K
@pytest.mark.parametrize("M,N,K", [(1030, 1029, 1000), (2050, 1050, 999), (1029, 2070, 230),
                                   (70, 65537, 40), (1041, 2051, 65), (2049, 1537, 250),
                                   (2050, 2070, 400), (3073, 2049, 530), (2051, 2040, 31)])
def test_gemm_dispatch(M, N, K):
    for ta in (False, True):
        for tb in (False, True):
            print("case: gemm M=%d N=%d K=%d, transposed %d %d" % (M, N, K, ta, tb), flush=True)
            A, B, f = _operands(M, N, K, ta, tb, M + N + K)
            C0, bias, gate = f(M, N), f(N), f(M, N)
            C = C0.clone()
            _lib.gemm_bf16(A, B, C, transA=ta, transB=tb, bias=bias, accumulate=True, relu=True,
                           gate=gate)
            a = (A.T if ta else A).bfloat16().double()
            b = (B.T if tb else B).bfloat16().double()
            ref = a @ b + C0.double() + bias.double()
            ref = torch.where(gate > 0, ref.clamp(min=0.0), torch.zeros_like(ref))
            mag = a.abs() @ b.abs() + C0.abs() + bias.abs()
            # products of BF16 values are exact in FP32; K + 2 FP32 additions in any order, each
            # rounded or truncated
            assert bool(((C - ref).abs() <= (K + 3) * 2.0 ** -23 * mag).all()), (ta, tb)


@pytest.mark.parametrize("tb", [False, True])
def test_gemm_of_2_to_the_32_results(tb):
    M = N = 65536
    K = 1000
    print("case: gemm M=%d N=%d K=%d, B transposed %d" % (M, N, K, tb), flush=True)
    A, B, _ = _operands(M, N, K, False, tb)
    C = torch.full((M, N), 7.0, device="cuda")
    _lib.gemm_bf16(A, B, C, transB=tb)
    rng = np.random.default_rng(0)
    rows = torch.from_numpy(np.r_[0, M - 1, rng.integers(0, M, 6)]).cuda()
    a, b = A[rows].bfloat16().double(), (B.T if tb else B).bfloat16().double()
    bar = (K + 1) * 2.0 ** -23 * (a.abs() @ b.abs())
    assert bool(((C[rows] - a @ b).abs() <= bar).all())
    cols = torch.from_numpy(np.r_[0, N - 1, rng.integers(0, N, 6)]).cuda()
    a, b = A.bfloat16().double(), (B[cols].T if tb else B[:, cols]).bfloat16().double()
    bar = (K + 1) * 2.0 ** -23 * (a.abs() @ b.abs())
    assert bool(((C[:, cols] - a @ b).abs() <= bar).all())
