// Batched GEMV Y = A X (X: k x nrhs, nrhs <= 16), Alg. 2's fused form: every
// element of A is read in FP64, quantised on the fly and multiplied on the
// matrix units, and nothing of A is written back.  The scaling is the fixed
// rule of Alg. 1's bound mu = k max|A~| max|X~| (OZ2_SCALE_FIXED: a row's scale
// depends on that row alone), so A is read twice: for its row maxima, then by
// the product.
//
// The integers Y~ = A~ X~ are formed exactly.  With at most 16 columns every
// element of A meets few multiplications, so what an element costs is its
// conversion, and residues modulo r moduli cost r conversions (127 operations
// per element at r = 13: 1.53 ms for 16384^2 x 8, 1.4 TB/s).  Here an element
// is its eight balanced base-256 digits -- the bytes of a + 0x0080..80, two
// instructions -- and the products of digits of equal weight are summed in
// int32 by v_mfma_i32_16x16x64_i8:
//     Y~ = sum_w 256^w sum_l sum_p a_p(l) x_{w-p}(l).
// The inner sums over (l, p) are ONE contraction: the A operand is the
// elements' bytes as they stand, and column (w, b) of the B operand holds the
// reversed digits of x(l, b) shifted by 7 - w bytes (two 64-bit shifts of the
// same registers for each w).  A wave's 64 k-bytes are 8 elements of 16 rows.
// The weights needed are 2 D - 1 or fewer, D the digits of the widths (7 for r
// = 12; 4 for r = 8).  |sums| <= 8 * 2^14 per element stay below 2^31 for the
// at most 8200 elements a wave takes.
//
// What bounds it: the two reads of A.  Per 8 x 16 elements the matrix unit
// takes 16 NT cycles (NT tiles of 16 columns, 7 for 8 right-hand sides), the
// conversion some 20 instructions per element.
#include <algorithm>

#include "oz2_device.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int GT = 256;        // threads per workgroup: 4 waves, each a quarter of k

// digits of a finite x scaled by 2^sc, rounded (RN-even, or toward zero), as
// the eight bytes of a two's complement number; t2: a nonzero x gives zero
__device__ __forceinline__ uint64_t digits(double x, int sc, unsigned tz, bool& t2) {
  const double y = ldexp(x, sc);
  const double a = tz ? trunc(y) : rint(y);
  t2 = (x != 0.0) && (a == 0.0);
  return digit_bytes(a) ^ 0x0080808080808080ull;
}

__device__ __forceinline__ int row_scale(unsigned long long b, int width) {
  return b >= kInfBits ? 0 : width - (b ? exp_of_bits(b) : 0);
}

// ---------------------------------------------------------------- scan
__global__ void k_gemv_init(unsigned long long* rowbits, uint32_t* flagsA, int mp, int m, int* counters,
                            int* listA, int keepA, int force, unsigned long long* colbits,
                            uint32_t* flagsB, int nrb) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) counters[1] = 0;
  if (i < nrb) {
    colbits[i] = 0;
    flagsB[i] = 0;
  }
  if (keepA) return;
  if (i == 0) counters[0] = force ? m : 0;
  if (i < mp) {
    rowbits[i] = 0;
    flagsA[i] = 0;
  }
  if (force && i < m) listA[i] = i;
}

// the largest of the workgroup's 256 values
__device__ __forceinline__ unsigned long long block_max(unsigned long long mx, unsigned long long* red) {
  const int t = threadIdx.x;
  for (int off = 32; off; off >>= 1) mx = max(mx, (unsigned long long)__shfl_xor((long long)mx, off));
  if ((t & 63) == 0) red[t >> 6] = mx;
  __syncthreads();
  return max(max(red[0], red[1]), max(red[2], red[3]));
}

// Workgroups 0 .. nrb-1: column b of X, its maximum, scale, flags and
// reversed digits: 8 bytes per (l, b) at [l/2][b][l%2], zeros for b >= nrhs and
// l >= k.  The others: the row maxima of A, 512 rows x kchunk columns each
// (hidden under them, one workgroup per column is enough for X).
// xs > 1 workgroups per column where they are not hidden (see the launch): only
// their parts' maxima here, the rest in k_gemv_digits.
__global__ void __launch_bounds__(256)
k_gemv_scan(const double* __restrict__ A, int lda, int m, int k, int kchunk, unsigned vec, int gx,
            unsigned long long* rowbits, const double* __restrict__ X, int ldx, int nrhs, int nrb,
            int kp, int width, unsigned tz, int force, int32_t* tB, uint32_t* flagsB, int* countB,
            int* listB, uint64_t* __restrict__ xd, int xs, unsigned long long* colbits) {
  const int blk = (int)blockIdx.x - nrb * xs;
  if (blk >= 0) {
    scan_rows_block(A, lda, m, k, kchunk, vec, rowbits, blk % gx, blk / gx);
    return;
  }
  __shared__ unsigned long long red[4];
  __shared__ unsigned flagged;
  const int b = blockIdx.x % nrb, t = threadIdx.x;
  const double* x = X + (size_t)b * ldx;
  unsigned long long mx = 0;
  if (xs > 1) {
    const int part = blockIdx.x / nrb, per = (k + xs - 1) / xs;
    const int l1 = min((long long)k, (long long)per * (part + 1));
    if (b < nrhs)
      for (long long l = (long long)per * part + t; l < l1; l += 256) mx = max(mx, abs_bits(x[l]));
    mx = block_max(mx, red);
    if (t == 0) atomicMax(colbits + b, mx);
    return;
  }
  if (b < nrhs)
    for (int l = t; l < k; l += 256) mx = max(mx, abs_bits(x[l]));
  if (t == 0) flagged = 0;
  mx = block_max(mx, red);
  const bool t1 = mx >= kInfBits;
  const int sc = row_scale(mx, width);
  bool any = false;
  for (int l = t; l < kp; l += 256) {
    bool t2 = false;
    const uint64_t v = (b < nrhs && l < k && !t1) ? digits(x[l], sc, tz, t2) : 0ull;
    any |= t2;
    xd[((size_t)(l >> 1) * nrb + b) * 2 + (l & 1)] = __builtin_bswap64(v);
  }
  if (any) atomicOr(&flagged, 1u);
  __syncthreads();
  if (t == 0 && b < nrhs) {
    const uint32_t f = (t1 ? OZ2_T1 : 0u) | (flagged ? OZ2_T2 : 0u);
    tB[b] = sc;
    flagsB[b] = f;
    if (f && !force) listB[atomicAdd(countB, 1)] = b;
  }
}

// The digits, scales and flags of X from the columns' maxima, GD rows l and all
// columns per workgroup (consecutive threads write consecutive bytes).
constexpr int GD = 512;
__global__ void __launch_bounds__(256)
k_gemv_digits(const double* __restrict__ X, int ldx, int k, int nrhs, int nrb, int kp, int width,
              unsigned tz, int force, const unsigned long long* __restrict__ colbits, int32_t* tB,
              uint32_t* flagsB, int* countB, int* listB, uint64_t* __restrict__ xd) {
  const int t = threadIdx.x, b = (t >> 1) & (nrb - 1);   // 2 nrb divides 256
  const unsigned long long mx = colbits[b];
  const bool t1 = mx >= kInfBits;
  const int sc = row_scale(mx, width);
  const int l0 = (int)blockIdx.x * GD, l1 = min(kp, l0 + GD);
  bool any = false;
  for (int l = l0 + 2 * (t / (2 * nrb)) + (t & 1); l < l1; l += 256 / nrb) {
    bool t2 = false;
    const uint64_t v = (b < nrhs && l < k && !t1) ? digits(X[(size_t)b * ldx + l], sc, tz, t2) : 0ull;
    any |= t2;
    xd[((size_t)(l >> 1) * nrb + b) * 2 + (l & 1)] = __builtin_bswap64(v);
  }
  const bool first = blockIdx.x == 0 && t < 2 * nrb && !(t & 1) && b < nrhs;
  if (first) tB[b] = sc;
  // a T1 column by the first workgroup, a T2 one by the first to flag it
  const uint32_t f = t1 ? (first ? OZ2_T1 : 0u) : (any ? OZ2_T2 : 0u);
  if (f && !(atomicOr(flagsB + b, f) & (OZ2_T1 | OZ2_T2)) && !force) listB[atomicAdd(countB, 1)] = b;
}

// ---------------------------------------------------------------- product
// The exact integer of weights' sums Y_w (from LDS, stride st), in NW words.
template <int NW>
__device__ __forceinline__ void carry(const long long* y, int nw, int nrb, uint32_t (&o)[NW]) {
  uint32_t byte[4 * NW];
  long long acc = 0;
  const int per = 16 / nrb;
#pragma unroll
  for (int w = 0; w < 4 * NW; ++w) {
    if (w < nw) acc += y[(w / per) * 16 + (w % per) * nrb];
    byte[w] = (uint32_t)acc & 0xFFu;
    acc >>= 8;
  }
#pragma unroll
  for (int q = 0; q < NW; ++q)
    o[q] = byte[4 * q] | (byte[4 * q + 1] << 8) | (byte[4 * q + 2] << 16) | (byte[4 * q + 3] << 24);
}

// grid (blocks of 16 RB rows, splits of k).  Lane L = (g, i) of a wave: rows
// row0 + RB i + q (q < RB, contiguous: 16-byte loads when aligned) and elements
// l = 8 c + 2 g, + 1 of every chunk c of 8; the wave takes chunks c0 + wave,
// + 4, .... NRB: columns of X rounded up to a power of two; NT tiles of 16
// columns (w, b), 16 / NRB weights each.
template <int NRB, int NT, int RB, int NW>
__global__ void __launch_bounds__(GT, 2)
k_gemv(const double* __restrict__ A, int lda, int m, int k, int cps, int width, unsigned vec,
       unsigned tz, int nweights, const unsigned long long* __restrict__ rowbits, uint32_t* flagsA,
       int* countA, int* listA, int listed, const uint4* __restrict__ xd, int nrhs,
       const int32_t* __restrict__ tB, uint32_t* __restrict__ part, int mp, double* Y, int ldy) {
  constexpr int PER = 16 / NRB, ROWS = 16 * RB;
  __shared__ unsigned long long sums[ROWS * NT * 16];
  const int t = threadIdx.x, lane = t & 63, i = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int row0 = (int)blockIdx.x * ROWS, rl = row0 + RB * i;
  for (int e = t; e < ROWS * NT * 16; e += GT) sums[e] = 0;
  __syncthreads();
  int sc[RB];
  unsigned t1 = 0;        // bit q: row rl + q is T1 or beyond m
#pragma unroll
  for (int q = 0; q < RB; ++q) {
    const unsigned long long b = rowbits[min(rl + q, m - 1)];
    sc[q] = row_scale(b, width);
    if (b >= kInfBits || rl + q >= m) t1 |= 1u << q;
  }
  const bool special = __any(t1 != 0);
  const int chunks = (k + 7) >> 3;
  const int c0 = (int)blockIdx.y * cps, c1 = min(chunks, c0 + cps);
  const bool wide = vec && row0 + ROWS <= m;   // uniform
  v4i acc[RB][NT];
#pragma unroll
  for (int q = 0; q < RB; ++q)
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[q][n] = v4i{0, 0, 0, 0};
  unsigned t2 = 0;
  // columns beyond k are clamped (X's digits are zeros there)
  auto load = [&](int c, double (&x)[2][RB], uint4& xr) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const double* p = A + (size_t)min(8 * c + 2 * g + u, k - 1) * lda;
      if (wide) {
#pragma unroll
        for (int q = 0; q < RB; q += 2) {
          const double2 v = *reinterpret_cast<const double2*>(p + rl + q);
          x[u][q] = v.x;
          x[u][q + 1] = v.y;
        }
      } else {
#pragma unroll
        for (int q = 0; q < RB; ++q) x[u][q] = p[min(rl + q, m - 1)];
      }
    }
    xr = xd[(size_t)(c * 4 + g) * NRB + (i & (NRB - 1))];
  };
  const int wl = i / NRB;   // the lane's weight within a tile
  double x[2][RB];
  uint4 xr;
  if (c0 + w < c1) load(c0 + w, x, xr);
  for (int c = c0 + w; c < c1; c += 4) {
    double xn[2][RB];
    uint4 xrn = xr;
    if (c + 4 < c1) load(c + 4, xn, xrn);
    const bool tail = 8 * c + 8 > k;   // uniform
    if (special || tail) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int q = 0; q < RB; ++q)
          if (((t1 >> q) & 1) || 8 * c + 2 * g + u >= k) x[u][q] = 0.0;
    }
    v4i fa[RB];
#pragma unroll
    for (int q = 0; q < RB; ++q)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        bool z;
        const uint64_t v = digits(x[u][q], sc[q], tz, z);
        t2 |= z ? 1u << q : 0u;
        fa[q][2 * u] = (int)(uint32_t)v;
        fa[q][2 * u + 1] = (int)(uint32_t)(v >> 32);
      }
    const uint64_t r0 = ((uint64_t)xr.y << 32) | xr.x, r1 = ((uint64_t)xr.w << 32) | xr.z;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      // byte p of column (wt, b) is digit wt - p: the reversed digits (byte p
      // holds digit 7 - p) moved down by 7 - wt bytes, up where negative
      const int sh = 8 * (7 - n * PER - (NRB == 16 ? 0 : wl));
      const int dn = max(sh, 0), up = max(-sh, 0) & 63;   // (a 16th weight is not used)
      const uint64_t b0 = (r0 >> dn) << up, b1 = (r1 >> dn) << up;
      const v4i fb{(int)(uint32_t)b0, (int)(uint32_t)(b0 >> 32), (int)(uint32_t)b1,
                   (int)(uint32_t)(b1 >> 32)};
#pragma unroll
      for (int q = 0; q < RB; ++q)
        acc[q][n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[q], fb, acc[q][n], 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int q = 0; q < RB; ++q) x[u][q] = xn[u][q];
    xr = xrn;
  }
  // flags and the fallback list: T1 rows once, T2 rows by the first to flag them
#pragma unroll
  for (int q = 0; q < RB; ++q) {
    const int row = rl + q;
    if (row >= m) continue;
    const bool is1 = (t1 >> q) & 1;
    const uint32_t f = is1 ? (g == 0 && w == 0 && blockIdx.y == 0 ? OZ2_T1 : 0u)
                           : (((t2 >> q) & 1) ? OZ2_T2 : 0u);
    if (f && !(atomicOr(flagsA + row, f) & (OZ2_T1 | OZ2_T2)) && !listed)
      listA[atomicAdd(countA, 1)] = row;
  }
  // the four waves' sums in 64 bits; lane (g, i) holds column i of tile n, rows
  // RB (4 g + e) + q
#pragma unroll
  for (int q = 0; q < RB; ++q)
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        atomicAdd(&sums[(RB * (4 * g + e) + q) * (NT * 16) + n * 16 + i],
                  (unsigned long long)(long long)acc[q][n][e]);
  __syncthreads();
  for (int o = t; o < ROWS * NRB; o += GT) {
    const int rr = o / NRB, b = o % NRB, row = row0 + rr;
    if (row >= m || b >= nrhs) continue;
    uint32_t v[NW];
    carry<NW>(reinterpret_cast<const long long*>(sums) + rr * (NT * 16) + b, nweights, NRB, v);
    if (gridDim.y == 1) {   // flagged entries are overwritten by the fallback
      Y[(size_t)row + (size_t)b * ldy] = round_scaled<NW>(v, row_scale(rowbits[row], width) + tB[b]);
    } else {
      uint32_t* dst = part + (((size_t)blockIdx.y * mp + row) * NRB + b) * NW;
#pragma unroll
      for (int q = 0; q < NW; ++q) dst[q] = v[q];
    }
  }
}

// the splits' integers summed and rounded once
template <int NW>
__global__ void __launch_bounds__(256)
k_gemv_sum(const uint32_t* __restrict__ part, int splits, int mp, int nrb, int m, int nrhs, int width,
           const unsigned long long* __restrict__ rowbits, const int32_t* __restrict__ tB, double* Y,
           int ldy) {
  const size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int row = (int)(o / nrb), b = (int)(o % nrb);
  if (row >= m || b >= nrhs) return;
  uint32_t v[NW];
#pragma unroll
  for (int q = 0; q < NW; ++q) v[q] = 0;
  for (int s = 0; s < splits; ++s) {
    const uint32_t* p = part + (((size_t)s * mp + row) * nrb + b) * NW;
    uint64_t cy = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      cy += (uint64_t)v[q] + p[q];
      v[q] = (uint32_t)cy;
      cy >>= 32;
    }
  }
  Y[(size_t)row + (size_t)b * ldy] = round_scaled<NW>(v, row_scale(rowbits[row], width) + tB[b]);
}

struct GemvArgs {
  const double* A;
  int lda, m, k, nrhs, splits, widthA, nweights, mp, listed, ldy;
  unsigned tz;
  const unsigned long long* rowbits;
  uint32_t* flagsA;
  int* countA;
  int* listA;
  const uint4* xd;
  const int32_t* tB;
  uint32_t* part;
  double* Y;
};

template <int NRB, int NT, int RB, int NW>
hipError_t launch_product(const GemvArgs& a, hipStream_t s) {
  const int chunks = (a.k + 7) / 8, cps = (chunks + a.splits - 1) / a.splits;
  const unsigned vec = ((uintptr_t)a.A % 16 == 0 && a.lda % 2 == 0) ? 1u : 0u;
  hipLaunchKernelGGL((k_gemv<NRB, NT, RB, NW>), dim3((a.m + 16 * RB - 1) / (16 * RB), a.splits),
                     dim3(GT), 0, s, a.A, a.lda, a.m, a.k, cps, a.widthA, vec, a.tz, a.nweights,
                     a.rowbits, a.flagsA, a.countA, a.listA, a.listed, a.xd, a.nrhs, a.tB, a.part,
                     a.mp, a.Y, a.ldy);
  return hipGetLastError();
}

// tiles for 2 D - 1 <= 9, 13, 15 weights
template <int NW>
hipError_t launch_columns(int nrb, const GemvArgs& a, hipStream_t s) {
  const int w = a.nweights;
  switch (nrb) {
    case 1: return launch_product<1, 1, 4, NW>(a, s);
    case 2: return launch_product<2, 2, 4, NW>(a, s);
    case 4: return launch_product<4, 4, 4, NW>(a, s);
    case 8:
      return w <= 10 ? launch_product<8, 5, 4, NW>(a, s)
           : w <= 14 ? launch_product<8, 7, 4, NW>(a, s) : launch_product<8, 8, 4, NW>(a, s);
    default:
      return w <= 9 ? launch_product<16, 9, 2, NW>(a, s)
           : w <= 13 ? launch_product<16, 13, 2, NW>(a, s) : launch_product<16, 15, 2, NW>(a, s);
  }
}

}  // namespace

// columns of X rounded up to a power of two
static int gemv_columns(int nrhs) {
  int b = 1;
  while (b < nrhs) b *= 2;
  return b;
}

hipError_t oz2_launch_gemv(const Oz2Const& c, const Oz2Dims& d, const Oz2Layout& L, uint8_t* ws,
                           const double* A, int lda, const double* X, int ldx, double* Y, int ldy,
                           int splits, bool reuse, hipStream_t s) {
  const int nrb = gemv_columns(d.n);
  const int force = (d.flags & 16u) ? 1 : 0;     // OZ2_FORCE_FALLBACK
  const unsigned tz = (d.flags & 4u) ? 1u : 0u;   // OZ2_QUANT_TZ
  // the fixed rule: ceil(log2(256 k)) halved (rounded up) off each budget
  int ell = 0;
  while ((1ull << ell) < 256ull * (unsigned long long)d.k) ++ell;
  const int wa = std::min(62, c.cA - ((ell + 1) >> 1)), wb = std::min(62, c.cB - ((ell + 1) >> 1));
  // |a| <= 2^w takes D balanced base-256 digits: 2^w <= 127/255 256^D
  const int da = (wa + 9) / 8, db = (wb + 9) / 8;
  auto* rowbits = (unsigned long long*)(ws + L.rowbits);
  auto* flagsA = (uint32_t*)(ws + L.flagsA);
  auto* counters = (int*)(ws + L.counters);
  auto* listA = (int*)(ws + L.listA);
  auto* tB = (int32_t*)(ws + L.tB);
  auto* colbits = (unsigned long long*)(ws + L.colbits);
  auto* flagsB = (uint32_t*)(ws + L.flagsB);
  hipLaunchKernelGGL(k_gemv_init, dim3((d.mp + 255) / 256), dim3(256), 0, s, rowbits, flagsA, d.mp,
                     d.m, counters, listA, reuse ? 1 : 0, force, colbits, flagsB, nrb);
  // rows: 512 per workgroup; k chunks sized for at most about 4096 workgroups
  const int gx = (d.m + 511) / 512;
  int kchunk = 32;
  while ((long long)gx * ((d.k + kchunk - 1) / kchunk) > 4096 && kchunk < 4096) kchunk *= 2;
  const int gy = (d.k + kchunk - 1) / kchunk;
  const unsigned vec = ((uintptr_t)A % 16 == 0 && lda % 2 == 0) ? 1u : 0u;
  // One workgroup per column of X takes 3 us per 1000 k.  It lies under the row
  // maxima of A where those are as long (16384^2 x 8: 781 us, 778 split); else,
  // from the k on where a launch more costs less, X is split over the chip (us, one
  // workgroup -> split: 1000 x 8000 x 8 69 -> 64, 1000 x 4000 x 8 49 -> 51; 16384 x
  // 16384 x 8 with A's scales kept 427 -> 409; 64 x 10^6 x 16 3484 -> 516).
  const bool hidden = !reuse && d.m >= 8192;
  const int xs = !hidden && d.k > 8192 ? std::min(256, (d.k + 2047) / 2048) : 1;
  hipLaunchKernelGGL(k_gemv_scan, dim3((unsigned)(nrb * xs + (reuse ? 0 : gx * gy))), dim3(256), 0, s, A,
                     lda, d.m, d.k, kchunk, vec, gx, rowbits, X, ldx, d.n, nrb, d.kp, wb, tz, force, tB,
                     flagsB, counters + 1, (int*)(ws + L.listB), (uint64_t*)(ws + L.xfrag), xs, colbits);
  if (xs > 1)
    hipLaunchKernelGGL(k_gemv_digits, dim3((d.kp + GD - 1) / GD), dim3(256), 0, s, X, ldx, d.k, d.n, nrb,
                       d.kp, wb, tz, force, colbits, tB, flagsB, counters + 1, (int*)(ws + L.listB),
                       (uint64_t*)(ws + L.xfrag));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const GemvArgs a{A, lda, d.m, d.k, d.n, splits, wa, da + db - 1, d.mp, force, ldy, tz, rowbits,
                   flagsA, counters, listA, (const uint4*)(ws + L.xfrag), tB,
                   (uint32_t*)(ws + L.part), Y};
  const unsigned blocks = (unsigned)(((size_t)d.m * nrb + 255) / 256);
#define OZ2_GV_WORDS(NW)                                                                          \
  {                                                                                               \
    e = launch_columns<NW>(nrb, a, s);                                                            \
    if (e == hipSuccess && splits > 1) {                                                          \
      hipLaunchKernelGGL(k_gemv_sum<NW>, dim3(blocks), dim3(256), 0, s, a.part, splits, d.mp, nrb, \
                         d.m, d.n, wa, rowbits, tB, Y, ldy);                                      \
      e = hipGetLastError();                                                                      \
    }                                                                                             \
  }
  if (c.nw == 3) OZ2_GV_WORDS(3) else if (c.nw == 4) OZ2_GV_WORDS(4) else OZ2_GV_WORDS(5)
  return e;
}
