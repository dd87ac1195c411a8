"""The digit kernel of the batched GEMV against the staged fixed-scale product
(the plane route): every column class, ragged rows and k, unaligned leading
dimensions, the digit counts of few and many moduli, extreme digits."""
import numpy as np
import pytest

from tests.gpu_util import bits, device

pytestmark = pytest.mark.gpu


def _compare(A, X, r, pad, flags=0, reuse=False):
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
    if reuse:      # another X first: A's side of the workspace stays
        ws = torch.empty(oz.ozaki2_gemv_workspace_bytes(m, k, n, r), dtype=torch.uint8, device=dev)
        oz.gemv(Ad, torch.ones_like(Xd).t().contiguous().t(), r, flags=flags, Y=Y, workspace=ws)
        oz.gemv(Ad, Xd, r, flags=flags | oz.OZ2_REUSE_A_SCALES, Y=Y, workspace=ws)
    else:
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


# X split over several workgroups per column (k above 8192, few rows or A's
# scales kept): partial chunks, columns that are flagged (by an entry of the
# last chunk, by infinities, and a zero one), the rows at which it is not split
@pytest.mark.parametrize("reuse", [False, True])
@pytest.mark.parametrize("m,n,k", [(3, 1, 8192), (3, 1, 8193), (5, 3, 8705), (70, 16, 20000), (33, 7, 70001),
                                   (8191, 2, 8200), (8192, 2, 8200)])
@pytest.mark.parametrize("flags", [0, 8])    # flagged entries native, or the integers' values
def test_split_columns(m, n, k, reuse, flags):
    rng = np.random.default_rng(m + k)
    A, X = rng.random((m, k)) - 0.5, rng.random((k, n)) - 0.5
    A[m // 2, ::2] *= 1e250
    if n > 1:
        X[k - 1, 0] = 1e-300
        X[k // 2, n - 1] = -np.inf
    if n > 2:
        X[:, 1] = 0.0
    _compare(A, X, 12, 1 if m == 5 else 0, flags=flags, reuse=reuse)
