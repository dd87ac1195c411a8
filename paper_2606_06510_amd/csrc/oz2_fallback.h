// The native-FP64 fallback of flagged rows and columns, shared by its own
// launch (reconstruct.hip) and the one-call products' small reconstructions
// (bytes.hip).
#pragma once
#include "oz2_device.h"

namespace {

// Native FP64 for flagged entries.  Work = (flagged rows of A) x (all
// columns) + (all unflagged rows) x (flagged columns of B), in 64 x 64 (or
// 64 x 32) output tiles walked by a grid-stride loop over the device-side counts (no host
// synchronisation; every workgroup exits when the tiles are exhausted).  A
// tile stages 64 rows x 32 k of A and 32 k x 64 columns of B through LDS (the
// next two slabs' loads held in registers while the current one is multiplied);
// each wave owns a 32 x 32 quarter as 2 x 2 blocks of
// v_mfma_f64_16x16x4_f64: A[i][k] from lane i + 16 k, B[k][j] from lane
// j + 16 k, and D[i][j] in lane j + 16 (i % 4), element i / 4.  The products
// and sums are FP64 in a fixed order (deterministic, not the order of a
// sequential dot product): the result lies within the FP64 dot-product
// error bound, which is the contract for flagged entries.
constexpr int FB_T = 64, FB_K = 32;
typedef double v4d __attribute__((ext_vector_type(4)));

struct FbShared {
  double sa[FB_K][FB_T + 2];   // [k][row]
  double sb[FB_T][FB_K + 2];   // [column][k]: the writes run along k (as [k][column] they met
                               // in a few banks)
  int rowid[FB_T], colid[FB_T], arow[FB_T];
};

template <int FC>
__device__ __forceinline__ void fallback_tiles(
    FbShared& S, const Oz2Dims& d, const double* __restrict__ A, int lda, const double* __restrict__ B,
    int ldb, double* C, int ldc, int na, int nb, const int* __restrict__ listA,
    const int* __restrict__ listB, const uint32_t* __restrict__ fA, const double* __restrict__ panel,
    int cap, int first, int stride) {
  constexpr int NJ = FC / 32;   // 16-column blocks per wave
  auto& sa = S.sa;
  auto& sb = S.sb;
  int *rowid = S.rowid, *colid = S.colid, *arow = S.arow;
  const bool acc = (d.flags & 1u) != 0;
  const bool force = (d.flags & 16u) != 0;
  // part 1: ceil(na/64) x ceil(n/64) tiles; part 2: ceil(m/64) x ceil(nb/64) tiles
  const int t1r = (na + FB_T - 1) / FB_T, t1c = (d.n + FC - 1) / FC;
  const int t2r = (d.m + FB_T - 1) / FB_T, t2c = (nb + FC - 1) / FC;
  const long long tiles1 = (long long)t1r * t1c, total = tiles1 + (long long)t2r * t2c;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wr = 32 * (w >> 1), wc = FC / 2 * (w & 1);
  const int kr = lane >> 4, cl = lane & 15;
  for (long long tile = first; tile < total; tile += stride) {
    // A rows come from the gathered panel when the tile's list rows all lie
    // in it (row r of the list at panel[r + l cap]), else from A itself
    const double* As = A;
    int ldas = lda;
    if (tile < tiles1) {
      const int tr = (int)(tile / t1c), tc = (int)(tile % t1c);
      const int nr = min(FB_T, na - tr * FB_T), nc = min(FC, d.n - tc * FC);
      const bool inpanel = panel != nullptr && (tr + 1) * FB_T <= cap;
      if (inpanel) {
        As = panel;
        ldas = cap;
      }
      if (t < FB_T) {
        rowid[t] = t < nr ? listA[tr * FB_T + t] : -1;
        arow[t] = t < nr ? (inpanel ? tr * FB_T + t : rowid[t]) : -1;
        colid[t] = t < nc ? tc * FC + t : -1;
      }
    } else {
      const long long u = tile - tiles1;
      const int tr = (int)(u / t2c), tc = (int)(u % t2c);
      const int nr = min(FB_T, d.m - tr * FB_T), nc = min(FC, nb - tc * FC);
      if (t < FB_T) {
        const int i = tr * FB_T + t;
        // rows already recomputed in part 1 (flagged rows) are skipped here
        rowid[t] = (t < nr && !(force || (fA[i] & (OZ2_T1 | OZ2_T2)))) ? i : -1;
        arow[t] = rowid[t];
        colid[t] = t < nc ? listB[tc * FC + t] : -1;
      }
    }
    __syncthreads();
    // Slab loads: thread t takes A entries (row t % 64, k t / 64 + 4 q) and B
    // entries (column t / 32 + 8 q, k t % 32).  Two slabs are in flight: with one,
    // each slab of 32 k waited out the memory latency (50 flagged rows of 6000 x
    // 4000: 94 tiles, 390 us).  No load stands under a branch, where it could not
    // be counted and both slabs were waited for at each: rows and columns beyond
    // the tile's are read at its first place (their sums are not stored), and
    // the slabs that k may cut short have a loop of their own, with clamped k
    // and zeros beyond it.
    const double* pa = As + max(arow[t & 63], 0);
    const double* pb[FC / 8];
#pragma unroll
    for (int q = 0; q < FC / 8; ++q) pb[q] = B + (size_t)max(colid[(t >> 5) + 8 * q], 0) * ldb + (t & 31);
    struct Slab {
      double a[8], b[FC / 8];
    };
    auto load = [&](int l0, Slab& s, auto whole) {
      const double* p = pa + (size_t)(l0 + (t >> 6)) * ldas;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        s.a[q] = whole ? p[(size_t)(4 * q) * ldas] : pa[(size_t)min(l0 + (t >> 6) + 4 * q, d.k - 1) * ldas];
      const int lb = whole ? l0 : min(l0, d.k - 1 - (t & 31));
#pragma unroll
      for (int q = 0; q < FC / 8; ++q) s.b[q] = pb[q][lb];
    };
    v4d cacc[2][NJ];
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < NJ; ++bj) cacc[bi][bj] = v4d{0.0, 0.0, 0.0, 0.0};
    // slab l0 from s; s then takes slab l0 + 64 (if `more`); whole: both end at k or before
    auto step = [&](int l0, Slab& s, bool more, auto whole) {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int l = (t >> 6) + 4 * q;
        sa[l][t & 63] = whole || l0 + l < d.k ? s.a[q] : 0.0;
        if (q < FC / 8)
          sb[(t >> 5) + 8 * q][t & 31] = whole || l0 + (t & 31) < d.k ? s.b[q < FC / 8 ? q : 0] : 0.0;
      }
      __syncthreads();
      if (more) load(l0 + 2 * FB_K, s, whole);
#pragma unroll
      for (int kk = 0; kk < FB_K; kk += 4) {
        const double a0 = sa[kk + kr][wr + cl], a1 = sa[kk + kr][wr + 16 + cl];
#pragma unroll
        for (int bj = 0; bj < NJ; ++bj) {
          const double b0 = sb[wc + 16 * bj + cl][kk + kr];
          cacc[0][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, cacc[0][bj], 0, 0, 0);
          cacc[1][bj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, cacc[1][bj], 0, 0, 0);
        }
      }
      __syncthreads();
    };
    Slab even, odd;
    const std::true_type whole{};
    const std::false_type cut{};
    load(0, even, cut);
    load(FB_K, odd, cut);
    int l0 = 0;
    for (; d.k - l0 >= 4 * FB_K; l0 += 2 * FB_K) {
      step(l0, even, true, whole);
      step(l0 + FB_K, odd, true, whole);
    }
    for (; l0 < d.k; l0 += 2 * FB_K) {
      step(l0, even, d.k - l0 > 2 * FB_K, cut);
      if (d.k - l0 > FB_K) step(l0 + FB_K, odd, d.k - l0 > 3 * FB_K, cut);
    }
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < NJ; ++bj)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = rowid[wr + 16 * bi + 4 * v + kr], j = colid[wc + 16 * bj + cl];
          if (i >= 0 && j >= 0) {
            double* o = C + (size_t)i + (size_t)j * ldc;
            *o = acc ? *o + cacc[bi][bj][v] : cacc[bi][bj][v];
          }
        }
    __syncthreads();   // rowid / colid are rewritten by the next tile
  }
}

}  // namespace
