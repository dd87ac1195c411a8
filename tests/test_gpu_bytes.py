"""The byte-residue route of the one-call products against the plane route of
the staged API: the same integers, so the same bits in every unflagged entry
(and the same fallback in the others)."""
import numpy as np
import pytest

import synth
from tests.gpu_util import bits, device

pytestmark = pytest.mark.gpu


def _both(m, n, k, r, flags=0, seed=0, pad=0, edit=None):
    import paper_2606_06510_amd as oz
    import torch
    dev = device()
    rng = np.random.default_rng(seed)
    A = (rng.random((m, k)) - 0.5) * np.exp(0.5 * rng.standard_normal((m, k)))
    B = (rng.random((k, n)) - 0.5) * np.exp(0.5 * rng.standard_normal((k, n)))
    if edit:
        edit(A, B)
    Cin = rng.standard_normal((m, n))

    def put(X):
        T = torch.zeros((X.shape[1], X.shape[0] + pad), dtype=torch.float64, device=dev)
        T[:, :X.shape[0]] = torch.from_numpy(np.ascontiguousarray(X.T)).to(dev)
        return T[:, :X.shape[0]].t()
    Ad, Bd, C1, C2 = put(A), put(B), put(Cin), put(Cin)
    oz.matmul(Ad, Bd, r, flags=flags, C=C1)
    plan = oz.Plan(m, n, k, r, flags, device=dev)
    plan.deconstruct(Ad, Bd)
    plan.residue_gemm()
    plan.reconstruct(C2)
    torch.cuda.synchronize()
    return (oz.from_device_colmajor(C1), oz.from_device_colmajor(C2))


def _same(x, y):
    assert np.array_equal(np.isnan(x), np.isnan(y))
    ok = ~np.isnan(x)
    assert np.array_equal(bits(x)[ok], bits(y)[ok])


@pytest.mark.parametrize("r", range(8, 17))
def test_every_moduli_count(r):
    _same(*_both(150, 90, 300, r, seed=r))


# tile edges of both kernels, one and several K-stages, the 256-k bound of the
# short reduction and the 32768-k bound of an exact slab
@pytest.mark.parametrize("shape", [(1, 1, 1), (17, 3, 63), (64, 16, 64), (129, 127, 65),
                                   (256, 256, 256), (257, 255, 257), (300, 270, 320),
                                   (1100, 1030, 700), (130, 70, 32768), (140, 60, 32833),
                                   (70, 260, 70000)])
@pytest.mark.parametrize("r", [12, 16])
def test_shapes(shape, r):
    _same(*_both(*shape, r, seed=sum(shape)))


@pytest.mark.parametrize("shape", [(2048, 2304, 192), (4352, 4096, 128), (2100, 2100, 4300)])
def test_many_tiles(shape):
    """the launches of whole rounds, several moduli per workgroup, an
    incomplete last share of the XCDs"""
    _same(*_both(*shape, 13, seed=5))


@pytest.mark.parametrize("name", ["ACCUMULATE", "SCALE_FIXED", "QUANT_TZ", "NO_FALLBACK",
                                  "FORCE_FALLBACK"])
def test_flags(name):
    import paper_2606_06510_amd as oz

    def edit(A, B):
        A[3, ::2] *= 1e200      # T2
        A[7, 5] = np.nan        # T1
        B[2, 9] = np.inf
        A[11] = 0.0
    flags = getattr(oz, "OZ2_" + name)
    _same(*_both(210, 140, 330, 12, flags=flags, seed=3, pad=3, edit=edit))


def test_extreme_digits():
    """entries whose quantised integers reach the widest digits: powers of two
    and their neighbours, both signs, against a constant operand"""
    def edit(A, B):
        v = np.array([1.0, -1.0, 1 - 2.0 ** -53, -(1 - 2.0 ** -53), 0.5, 2.0 ** -40])
        A[:] = np.resize(v, A.shape)
        B[:] = np.where(np.arange(B.shape[1]) % 2, 1.0, -1.0 + 2.0 ** -52)
    for r in (8, 12, 15):
        _same(*_both(130, 130, 2000, r, edit=edit))


@pytest.mark.parametrize("case", [(5, 70, 90, 33, 12), (3, 200, 66, 129, 15), (40, 65, 64, 64, 8)])
def test_batches_side_by_side(case):
    import paper_2606_06510_amd as oz
    import torch
    b, m, n, k, r = case
    dev = device()
    gen = torch.Generator(device=dev).manual_seed(1)
    A = torch.rand((b, k + 1, m + 3), generator=gen, dtype=torch.float64, device=dev) - 0.5
    B = torch.rand((b, n, k + 2), generator=gen, dtype=torch.float64, device=dev) - 0.5
    A[1, :, 4] *= 1e-30
    A[1, 3, 4] = 1e200          # a fallback row in one problem only
    C = torch.full((b, n + 1, m + 1), 7.0, dtype=torch.float64, device=dev)
    oz.ozaki2_dgemm_strided_batched(m, n, k, A, m + 3, A.stride(0), B, k + 2, B.stride(0), C, m + 1,
                                    C.stride(0), b, r)
    torch.cuda.synchronize()
    assert torch.all(C[:, n] == 7.0) and torch.all(C[:, :, m] == 7.0)
    for i in range(b):
        D = oz.matmul(A[i, :k, :m].t(), B[i, :, :k].t(), r)
        assert torch.equal(C[i, :n, :m].t(), D), i


# the one-launch scan and codes of short rows: whole and partial groups of four
# k, its last k and the first beyond it, partial blocks of 16 rows, odd leading
# dimensions, scales by the products' maxima and fixed
@pytest.mark.parametrize("m,n,k,pad", [(1, 17, 1, 0), (16, 33, 3, 1), (255, 240, 64, 0), (257, 130, 255, 3),
                                       (100, 300, 1021, 2), (300, 100, 1024, 0), (129, 64, 1025, 0)])
@pytest.mark.parametrize("flags", [0, 2])
def test_short_rows_scan(m, n, k, pad, flags):
    def edit(A, B):
        A[m // 2] = 0.0
        A[m - 1, k - 1] *= 2.0 ** 900
        B[k // 2, n - 1] = np.inf
        B[k - 1, n // 2] = 2.0 ** -1060        # a subnormal entry beside normal ones
        if m > 8:
            A[5] = 2.0 ** -1062 * np.arange(k)  # a row of subnormals
            A[3, 0] = np.nan
    _same(*_both(m, n, k, 12, flags=flags, seed=m, pad=pad, edit=edit))


@pytest.mark.parametrize("flags", [0, 32])   # 32: OZ2_KEEP_RESIDUES, the plane route
def test_zero_blocks_in_rows_of_small_entries(flags):
    """rows and columns below 1/2 with whole zero blocks of 64 k (banded,
    block-sparse operands), beyond the rows that one workgroup holds: exact
    against the oracle"""
    import oracle
    import paper_2606_06510_amd as oz
    rng = np.random.default_rng(9)
    m, n, k = 70, 66, 1300
    A, B = 1e-3 * (rng.random((m, k)) + 0.1), 1e-12 * (rng.random((k, n)) + 0.1)
    A[:, 64:128] = 0.0
    A[5, 128:1280] = 0.0
    A[6, :1280] = 0.0
    A[7] *= 1e-290
    B[640:704, ::2] = 0.0
    B[192:256, 3] *= 1e-3
    dev = device()
    C = oz.matmul(oz.to_device_colmajor(A, dev), oz.to_device_colmajor(B, dev), 12, flags=flags)
    got, res = oz.from_device_colmajor(C), oracle.dgemm(A, B, 12)
    emu = (~np.isin(np.arange(m), res.fallback_rows))[:, None] & ~np.isin(np.arange(n), res.fallback_cols)
    assert emu.mean() > 0.9
    assert np.array_equal(bits(got)[emu], bits(res.C)[emu])


def test_blocks_under_capture_take_the_pool_as_it_is():
    """a batch captured when the internal workspace holds fewer problems than
    would run side by side: no allocation, the same results on every replay"""
    import paper_2606_06510_amd as oz
    import torch
    dev = device()
    b, m, n, k, r = 7, 130, 70, 90, 12
    gen = torch.Generator(device=dev).manual_seed(3)
    A = torch.rand((b, k, m), generator=gen, dtype=torch.float64, device=dev) - 0.5
    B = torch.rand((b, n, k), generator=gen, dtype=torch.float64, device=dev) - 0.5
    A[2, ::2, 5] *= 1e200       # a fallback row in one problem
    C, D = torch.zeros((b, n, m), dtype=torch.float64, device=dev), None

    def call(count, out, stream=None):
        oz.ozaki2_dgemm_strided_batched(m, n, k, A, m, m * k, B, k, n * k, out, m, m * n, count, r,
                                        stream=stream)
    oz.ozaki2_finalize()
    call(2, C)                  # the pool holds two problems (1 MiB at least)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(b, C, stream=side.cuda_stream)
    seen = []
    for i in range(3):
        A.add_(0.25 * i)
        C.zero_()
        graph.replay()
        torch.cuda.synchronize()
        seen.append((A.clone(), C.clone()))
    for Ai, Ci in seen:
        A.copy_(Ai)
        D = torch.zeros_like(C)
        call(b, D)
        torch.cuda.synchronize()
        assert torch.equal(Ci, D)


def test_a_captured_workspace_outlives_growing_calls():
    """a batch captured on a small workspace, then the same batch called plainly,
    which grows it: the captured buffer stays allocated (looked up on the host
    before the graph runs again) and the graph still gives the right results"""
    import ctypes
    import paper_2606_06510_amd as oz
    import torch
    dev = device()
    b, m, n, k, r = 9, 140, 75, 80, 12
    gen = torch.Generator(device=dev).manual_seed(4)
    A = torch.rand((b, k, m), generator=gen, dtype=torch.float64, device=dev) - 0.5
    B = torch.rand((b, n, k), generator=gen, dtype=torch.float64, device=dev) - 0.5
    C, D = (torch.zeros((b, n, m), dtype=torch.float64, device=dev) for _ in range(2))

    def call(count, out, stream=None):
        oz.ozaki2_dgemm_strided_batched(m, n, k, A, m, m * k, B, k, n * k, out, m, m * n, count, r,
                                        stream=stream)

    def buffers():
        out = (ctypes.c_void_p * 8)()
        return out[:oz.load().oz2_pool_buffers(out, 8)]
    oz.ozaki2_finalize()
    assert buffers() == []
    call(2, C)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(b, C, stream=side.cuda_stream)
    taken = buffers()
    assert len(taken) == 1
    for i in range(3):
        A.add_(0.25 * i)
        C.zero_()
        call(b, D)
        torch.cuda.synchronize()
        assert taken[0] in buffers() and len(buffers()) == 2
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(C, D), i
    del graph
    oz.ozaki2_finalize()
    assert buffers() == []


@pytest.mark.parametrize("m,n,k", [(64, 64, 64), (1, 1, 1), (17, 64, 3), (64, 15, 33), (50, 49, 64)])
@pytest.mark.parametrize("r", [8, 11, 12, 13, 16])
def test_small_batches_digit_counts(m, n, k, r):
    """the single-launch kernel (six, seven or eight digits by the widest
    entry of a problem) against the byte-residue route, problem by problem:
    full-mantissa entries, powers of two next to their neighbours, one
    nonzero per row (the widest scales), unaligned leading dimensions"""
    import paper_2606_06510_amd as oz
    import torch
    dev = device()
    rng = np.random.default_rng(r + m)
    A = rng.random((4, k, m)) - 0.5
    B = rng.random((4, n, k)) - 0.5
    v = np.array([1.0, -1.0, 1 - 2.0 ** -53, -(1 - 2.0 ** -53), 0.5, 2.0 ** -40])
    A[1], B[1] = np.resize(v, (k, m)), np.resize(v[::-1], (n, k))
    A[2] *= np.arange(k)[:, None] == np.arange(m)[None, :] % k
    B[2] *= np.arange(k)[None, :] == np.arange(n)[:, None] % k
    A[3], B[3] = np.abs(A[3]) + 1, -np.abs(B[3]) - 1
    for pad in (0, 1):
        Ap, Bp = np.zeros((4, k, m + pad)), np.zeros((4, n, k + pad))
        Ap[:, :, :m], Bp[:, :, :k] = A, B
        Ad, Bd = torch.from_numpy(Ap).to(dev), torch.from_numpy(Bp).to(dev)
        C = torch.full((4, n, m + pad), 7.0, dtype=torch.float64, device=dev)
        oz.ozaki2_dgemm_strided_batched(m, n, k, Ad, m + pad, Ad.stride(0), Bd, k + pad, Bd.stride(0),
                                        C, m + pad, C.stride(0), 4, r)
        torch.cuda.synchronize()
        assert torch.all(C[:, :, m:] == 7.0)
        for i in range(4):
            D = oz.matmul(Ad[i, :, :m].t(), Bd[i, :, :k].t(), r)
            assert torch.equal(C[i, :, :m].t(), D), (i, pad)


# the fused products and reconstruction (k <= 256, tiles that fill the chip):
# ragged edges of the 128 x 128 tiles, several turns of a workgroup, one to
# four K-stages, odd leading dimensions, fallback entries beside C_in
@pytest.mark.parametrize("m,n,k,r,pad,flags", [(2040, 1801, 70, 12, 0, 0), (1793, 2047, 256, 11, 1, 1),
                                               (4300, 4100, 17, 10, 0, 1), (2047, 2047, 190, 12, 3, 9),
                                               (2048, 2048, 129, 12, 0, 16)])
def test_fused_short_k(m, n, k, r, pad, flags):
    def edit(A, B):
        A[m // 2, ::2] *= 1e200     # T2
        A[m - 1, 1] = np.nan        # T1
        B[2, n - 1] = np.inf
        A[5] = 0.0
        A[40:60] = np.round(A[40:60] * 4)    # few significant bits, exact zeros
        B[:, 100:120] = np.round(B[:, 100:120] * 4)
    _same(*_both(m, n, k, r, flags=flags, seed=k, pad=pad, edit=edit))


# the same with the fewest moduli: 10 and 11 residue bytes, the last word of a
# lane's residues partly or wholly zero
@pytest.mark.parametrize("m,n,k,r,pad,flags", [(2040, 1801, 70, 8, 0, 0), (2047, 2047, 256, 8, 1, 1),
                                               (4300, 4100, 17, 9, 0, 1), (1793, 2047, 129, 9, 3, 9)])
def test_fused_short_k_few_moduli(m, n, k, r, pad, flags):
    def edit(A, B):
        A[m // 2, ::2] *= 1e200     # T2
        B[2, n - 1] = np.nan        # T1
        A[:300] *= 2.0 ** -520      # results around the smallest normal number
        B[:, :400] *= 2.0 ** -500
        A[40:60] = np.round(A[40:60] * 4)
    _same(*_both(m, n, k, r, flags=flags, seed=k, pad=pad, edit=edit))


def test_fused_short_k_subnormal_and_small_integers():
    """results around and below the smallest normal number, in some rows and
    columns only (the words' rounding), and integers of few bits"""
    def edit(A, B):
        A[:300] *= 2.0 ** -540
        B[:, :400] *= 2.0 ** -482
        B[:, 100:200] *= 2.0 ** -33
        A[300:420] = np.sign(A[300:420])
        B[:, 400:500] = np.sign(B[:, 400:500])
    x, y = _both(2050, 1900, 60, 12, seed=1, edit=edit)
    _same(x, y)
    small = np.abs(x[:300, :400])
    assert np.count_nonzero(small < 2.0 ** -1022) > 1000 and np.count_nonzero(small >= 2.0 ** -1022) > 100


# the fallback inside the reconstruction's launch (up to two of its workgroups
# per CU: 1024 x 1024) and in a launch of its own beyond: flagged rows and
# columns, more of them than one tile, C_in, all rows, none
@pytest.mark.parametrize("m,n,k", [(1, 18, 5), (200, 333, 70), (1024, 1024, 96), (1024, 1040, 96)])
@pytest.mark.parametrize("flags", [0, 1, 8, 17])
def test_fallback_beside_the_reconstruction(m, n, k, flags):
    def edit(A, B):
        A[m // 3:m // 3 + 70, ::2] *= 1e200   # T2
        A[m - 1, k - 1] = np.inf              # T1
        B[1, n // 2] = np.nan
        B[::2, n - 1] *= 1e-200
    _same(*_both(m, n, k, 12, flags=flags, seed=n, pad=1, edit=edit))


# the native FP64 of flagged entries at the edges of its slabs of 32 k (two in
# flight, a loop of its own for those k cuts short), beside the reconstruction
# and in its own launch, 64 x 32 and 64 x 64 tiles, rows within and beyond the
# gathered panel.  Row 0 of A and column 0 of B, which stand in for what lies
# outside a tile, are not finite.
@pytest.mark.parametrize("k", [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 161, 223, 257])
@pytest.mark.parametrize("m,n,flags", [(70, 40, 0), (150, 66, 16), (1040, 1040, 0), (1040, 1040, 16)])
def test_fallback_slab_edges(m, n, k, flags):
    import paper_2606_06510_amd as oz
    rng = np.random.default_rng(k)
    A, B = rng.random((m, k)) - 0.5, rng.random((k, n)) - 0.5
    A[0], B[k - 1, 0] = np.nan, np.inf
    A[m // 3, ::2] *= 1e-200
    A[m - 1, k - 1] = -np.inf
    B[::2, n // 2] *= 1e-200
    dev = device()
    C = oz.from_device_colmajor(oz.matmul(oz.to_device_colmajor(A, dev), oz.to_device_colmajor(B, dev), 12,
                                          flags=flags))
    with np.errstate(invalid="ignore"):
        ref, den = A @ B, np.abs(A) @ np.abs(B)
        diff = np.abs(C - ref)
    rows = np.full(m, bool(flags & 16))
    rows[[0, m // 3, m - 1]] = True
    cols = np.isin(np.arange(n), [0, n // 2])
    native = rows[:, None] | cols
    assert np.array_equal(np.isnan(C), np.isnan(ref))
    inf = np.isinf(ref)
    assert np.array_equal(C[inf], ref[inf])
    ok = native & np.isfinite(ref)
    # two dot products of k terms, each within k u / (1 - k u) of the exact one
    assert np.all(diff[ok] <= 2.02 * (k + 1) * 2.0 ** -53 * den[ok])
    assert np.all(diff[~native] <= 1e-13 * np.sqrt(k))


@pytest.mark.parametrize("flags", [0, 2])
def test_one_call_product_on_a_plans_workspace(flags):
    """the one-call product between two passes of a plan, on the plan's own
    workspace: the plan's tables, built by its first pass, are still there"""
    import paper_2606_06510_amd as oz
    import torch
    m, n, k, r = 1000, 900, 70, 12      # short k: the residues are the larger part
    rng = np.random.default_rng(6)
    dev = device()
    Ad = oz.to_device_colmajor(rng.random((m, k)) - 0.5, dev)
    Bd = oz.to_device_colmajor(rng.random((k, n)) - 0.5, dev)
    plan = oz.Plan(m, n, k, r, flags, device=dev)
    C = [oz.colmajor_empty(m, n, device=dev) for _ in range(3)]

    def run(out):
        plan.deconstruct(Ad, Bd)
        plan.residue_gemm()
        plan.reconstruct(out)
    run(C[0])
    oz.matmul(Ad, Bd, r, flags=flags, C=C[1], workspace=plan.workspace)
    run(C[2])
    torch.cuda.synchronize()
    assert torch.equal(C[0], C[1]) and torch.equal(C[0], C[2])
