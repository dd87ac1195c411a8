"""The digit kernel of the batched GEMV against the staged fixed-scale product
(the plane route): every column class, ragged rows and k, unaligned leading
dimensions, the digit counts of few and many moduli, extreme digits."""
import numpy as np
import pytest

from tests.gpu_util import bits, device

pytestmark = pytest.mark.gpu


def _compare(A, X, r, pad, flags=0):
    import paper_2606_06510_amd as oz
    import torch
    dev = device()
    m, k = A.shape
    n = X.shape[1]

    def put(M):
        T = torch.zeros((M.shape[1], M.shape[0] + pad), dtype=torch.float64, device=dev)
        T[:, :M.shape[0]] = torch.from_numpy(np.ascontiguousarray(M.T)).to(dev)
        return T[:, :M.shape[0]].t()
    Ad, Xd, Y, C = put(A), put(X), put(np.full((m, n), np.nan)), put(np.full((m, n), np.nan))
    oz.gemv(Ad, Xd, r, flags=flags, Y=Y)
    plan = oz.Plan(m, n, k, r, oz.OZ2_SCALE_FIXED | flags, device=dev)
    plan.deconstruct(Ad, Xd)
    plan.residue_gemm()
    plan.reconstruct(C)
    torch.cuda.synchronize()
    y, c = oz.from_device_colmajor(Y), oz.from_device_colmajor(C)
    assert np.array_equal(bits(y), bits(c))


@pytest.mark.parametrize("n", [1, 2, 3, 4, 6, 8, 9, 16])
@pytest.mark.parametrize("m,k,r,pad", [(65, 33, 8, 0), (130, 1031, 12, 3), (63, 8, 16, 1),
                                       (34, 700, 14, 0)])
def test_column_classes(n, m, k, r, pad):
    rng = np.random.default_rng(m + k + n)
    A = (rng.random((m, k)) - 0.5) * np.exp(rng.standard_normal((m, k)))
    X = (rng.random((k, n)) - 0.5) * np.exp(rng.standard_normal((k, n)))
    if n > 2:
        A[m // 2, ::2] *= 1e250      # T2 row
        X[k // 2, 1] = np.inf        # T1 column
    _compare(A, X, r, pad, flags=8 if n > 2 else 0)   # NO_FALLBACK: the integers' values


@pytest.mark.parametrize("r", [9, 12, 13, 16])
@pytest.mark.parametrize("k", [40, 9000])
def test_extreme_digits(r, k):
    """rows of equal signs at the width's limit: the largest digit sums"""
    v = np.array([1.0, 1 - 2.0 ** -53, 0.75, 0.5 + 2.0 ** -9])
    A = np.resize(v, (40, k)) * np.where(np.arange(40) % 2, 1.0, -1.0)[:, None]
    X = np.resize(v[::-1], (k, 5)) * np.where(np.arange(5) % 2, -1.0, 1.0)
    _compare(A, X, r, 0)
