// Phases 1 (last step) and 3 of Alg. 1 on byte residues: the quantise ->
// residue split of A and B, and the CRT reconstruction of C, of the one-call
// products (bytegemm.hip is the GEMM between them; Oz2Byte the residue
// system).  The quantised integers A~, B~ (Eq. (scale)), the flags and the
// integer C~ are those of the plane route, so C is the same bit for bit.
#include <algorithm>

#include "oz2_device.h"
#include "oz2_fallback.h"
#include "oz2_tile.h"

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------- split
// One workgroup of 256 threads per 64 x 64 tile: thread t quantises row t/4,
// k 16 (t%4) .. +15, and writes its 16 bytes of every modulus's plane (1 KiB
// contiguous per wave store).  The row's scale (Eq. (scale)'s width less the
// exponent) is formed here from the maxima; the tiles of k block 0 also leave
// scales, T1 flags and the fallback list.  Tiles wholly beyond the matrix are
// not written: their bytes reach padded outputs only.
//
// The residue of the quantised integer a (|a| <= 2^62): its eight balanced
// base-256 digits (bytes of a + 0x0080..80, each minus 128) against the
// centred residues of 256^j, two dot4 instructions on top of tof = 128 + K m
// (K m >= 2^17 > |sum|): t' >= 0 and below 2^19, so floor(t'/m) is one exact
// high multiply with ceil(2^32/m), and t' - m floor(t'/m) - 128 lies in
// [-128, m - 129]: an int8 congruent to a.  Six instructions per element and
// modulus, packing included, and no table: the split stays bound by its
// stores.
struct ByteSide {
  const double* X;
  int ld, rows, rows_pad, ntiles;
  const unsigned long long* bits;   // row maxima
  const uint32_t* rmax;             // code products' maxima, [cslabs][rows_pad]
  int cslabs, budget;
  unsigned long long fixedR;        // OZ2_SCALE_FIXED: 256 k, else 0
  int32_t* scale;
  uint32_t* flags;
  uint8_t* planes;
  unsigned vec;
  int* count;
  int* list;
  int listed, all;     // FORCE_FALLBACK: no row is listed by its flags; all rows are (A)
  long long stride;    // elements between the problems of a batch
};

template <bool TRANS>
__device__ __forceinline__ void byte_tile(const Oz2Byte& c, const ByteSide& S, int tl, int k, int kp,
                                          unsigned quant_tz, size_t z, int i0, int i1) {
  const int nrb = (S.rows + 63) / 64;
  const int t = threadIdx.x;
  const int row = (tl % nrb) * 64 + (t >> 2), l0 = (tl / nrb) * 64 + (t & 3) * 16;
  const bool inrow = row < S.rows;
  uint32_t* flags = zws(S.flags, z);
  const unsigned long long top = inrow ? zws(S.bits, z)[row] : 0ull;
  const bool t1 = top >= kInfBits, zero = !inrow || t1;
  int sc = 0;
  if (!zero) {
    unsigned long long R = S.fixedR;
    if (!R)
      for (int sl = 0; sl < S.cslabs; ++sl) R += zws(S.rmax, z)[(size_t)sl * S.rows_pad + row];
    sc = width_of(R, S.budget) - (top ? exp_of_bits(top) : 0);
  }
  if (tl < nrb && i0 == 0 && (t & 3) == 0 && inrow) {
    zws(S.scale, z)[row] = sc;
    if (t1) atomicOr(flags + row, OZ2_T1);
    if (S.all || (t1 && !S.listed)) zws(S.list, z)[atomicAdd(zws(S.count, z), 1)] = row;
  }
  const double* X = S.X + (size_t)blockIdx.z * S.stride;
  double x[16];
  if (!TRANS && S.vec && !zero && l0 + 16 <= k) {
    const double2* p = reinterpret_cast<const double2*>(X + (size_t)row * S.ld + l0);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const double2 v = p[j];
      x[2 * j] = v.x;
      x[2 * j + 1] = v.y;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int l = l0 + j;
      const size_t off = TRANS ? ((size_t)row + (size_t)l * S.ld) : ((size_t)l + (size_t)row * S.ld);
      x[j] = (!zero && l < k) ? X[off] : 0.0;
    }
  }
  uint32_t lo[16], hi[16];
  bool t2 = false;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const double y = ldexp(x[j], sc);
    const double a = quant_tz ? trunc(y) : rint(y);
    t2 |= (x[j] != 0.0) && (a == 0.0);
    const uint64_t v = digit_bytes(a);
    lo[j] = (uint32_t)v ^ 0x80808080u;
    hi[j] = (uint32_t)(v >> 32) ^ 0x00808080u;
  }
  // the first tile to flag a row adds it to the fallback list (unless every
  // row is listed already)
  if (t2 && i0 == 0 && !(atomicOr(flags + row, OZ2_T2) & (OZ2_T1 | OZ2_T2)) && !S.listed)
    zws(S.list, z)[atomicAdd(zws(S.count, z), 1)] = row;
  uint8_t* dst = zws(S.planes, z) + ((size_t)(l0 >> 6) * S.rows_pad + row) * OZ2_KBLK + (l0 & 63);
  const size_t pstride = (size_t)S.rows_pad * kp;
  dst += i0 * pstride;
  for (int i = i0; i < i1; ++i) {
    const int w0 = c.dot[i][0], w1 = c.dot[i][1], tof = c.tof[i];
    const uint32_t mg = c.mg0[i], nm = c.nm[i];
    uint32_t u[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      int s = __builtin_amdgcn_sdot4((int)lo[j], w0, tof, false);
      s = __builtin_amdgcn_sdot4((int)hi[j], w1, s, false);
      u[j] = __umul24(__umulhi((uint32_t)s, mg), nm) + (uint32_t)s;
    }
    u32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      v[q] = low4(u[4 * q], u[4 * q + 1], u[4 * q + 2], u[4 * q + 3]) ^ 0x80808080u;
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(dst));
    dst += pstride;
  }
}

// B's tiles first (B was read last by the scans and may still be in the
// memory-side cache), then A's; y: a share of the moduli
__global__ void __launch_bounds__(256)
k_byte_split(Oz2Byte c, ByteSide SA, ByteSide SB, int k, int kp, unsigned quant_tz, int share,
             size_t wsz) {
  const int t = blockIdx.x, i0 = blockIdx.y * share, i1 = min(c.n, i0 + share);
  const size_t z = (size_t)blockIdx.z * wsz;
  if (t < SB.ntiles) byte_tile<false>(c, SB, t, k, kp, quant_tz, z, i0, i1);
  else byte_tile<true>(c, SA, t - SB.ntiles, k, kp, quant_tz, z, i0, i1);
}

// ---------------------------------------------------------------- reconstruction
// X = sum_i u_i W_i - q M over the N moduli, with W_i the representative of
// smallest magnitude, in radix-2^38 fp64 limbs (NB of them; the top limb
// signed).  Exact: u_i <= 255 and at most 16 moduli with |W_i| top limbs
// below 2^41 (NB = 3) or 19 with lower limbs below 2^38: every sum is an
// integer below 2^53.  |X| <= 0.41 M (the host's choice of moduli), so the
// quotient estimate (error below 2^-24) is never ambiguous.
//
// A workgroup of 256 threads takes 128 rows x 16 columns: thread t the 8
// outputs of column t%64/4%16.. held by half a lane's 16 bytes of a unit
// (see bytegemm.hip); moduli outermost, so that each is loaded and used once
// and its weights stay in scalar registers.  The results go through LDS, so
// that a store instruction writes 512 contiguous bytes of a column.
//
// FB: the workgroups from ncrt on are the native fallback's, which write
// the flagged entries that the others leave (A read directly, no panel).
template <int N, bool ACC, bool FB>
__global__ void __launch_bounds__(256)
k_byte_crt(Oz2Byte c, Oz2Dims d, const uint8_t* __restrict__ res, const int32_t* __restrict__ sA,
           const int32_t* __restrict__ tB, const uint32_t* __restrict__ fA,
           const uint32_t* __restrict__ fB, double* C, int ldc, const double* __restrict__ A,
           int lda, const int* __restrict__ counters, const int* __restrict__ listA,
           double* __restrict__ panel, int cap, int nrow, const double* __restrict__ B, int ldb,
           const int* __restrict__ listB, int ncrt, Oz2Batch bt) {
  if constexpr (FB) {
    if ((int)blockIdx.x >= ncrt) {
      __shared__ FbShared fs;
      const size_t z = (size_t)blockIdx.z * bt.ws;
      const int na = zws(counters, z)[0], nb = zws(counters, z)[1];
      fallback_tiles<32>(fs, d, A + (size_t)blockIdx.z * bt.sA, lda, B + (size_t)blockIdx.z * bt.sB, ldb,
                         C + (size_t)blockIdx.z * bt.sC, ldc, na, nb, zws(listA, z), zws(listB, z),
                         zws(fA, z), nullptr, 0, (int)blockIdx.x - ncrt, (int)gridDim.x - ncrt);
      return;
    }
  }
  constexpr int NB = N <= 15 ? 3 : 4;
  __shared__ double tr[16][129];
  const size_t z = (size_t)blockIdx.z * bt.ws;
  counters = zws(counters, z);
  sA = zws(sA, z);
  tB = zws(tB, z);
  fA = zws(fA, z);
  fB = zws(fB, z);
  C += (size_t)blockIdx.z * bt.sC;
  const int nflag = panel ? counters[0] : 0;   // used at the end; loaded early
  const int t = threadIdx.x;
  const int rb = (int)(blockIdx.x % (unsigned)nrow), cb = (int)(blockIdx.x / (unsigned)nrow);
  // store phase: row t%128, columns t/128 + 2 j
  const int srow = rb * 128 + (t & 127);
  double cin[8];
  if constexpr (ACC) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int col = cb * 16 + (t >> 7) + 2 * j;
      cin[j] = (srow < d.m && col < d.n) ? __builtin_nontemporal_load(C + (size_t)col * ldc + srow) : 0.0;
    }
  }
  {
    // unit u = t / 128 (rows 64 u ..), lane L = (t % 128) / 2, half h = t % 2
    const int u = t >> 7, L = (t & 127) >> 1, h = t & 1;
    const uint8_t* q = res + z + ((size_t)cb * (d.mp / 64) + rb * 2 + u) * 1024 + 16 * L + 8 * h;
    const size_t plane = (size_t)d.mp * d.np;
    double S[8][NB];
#pragma unroll
    for (int I = 0; I < 8; ++I)
#pragma unroll
      for (int l = 0; l < NB; ++l) S[I][l] = 0.0;
    u32x2 x[N];
#pragma unroll
    for (int i = 0; i < N; ++i)
      x[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(q + (size_t)i * plane));
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
      for (int I = 0; I < 8; ++I) {
        const double v = (double)(float)((x[i][I >> 2] >> (8 * (I & 3))) & 0xFFu);
#pragma unroll
        for (int l = 0; l < NB; ++l) S[I][l] = fma(v, c.W38[i][l], S[I][l]);
      }
    }
    const int col = cb * 16 + (L & 15);
    const int tj = col < d.n ? tB[col] : 0;
#pragma unroll
    for (int I = 0; I < 8; ++I) {
      const int rr = 64 * u + 16 * (2 * h + (I >> 2)) + 4 * (L >> 4) + (I & 3);
      const int row = rb * 128 + rr;
      const int si = row < d.m ? sA[row] : 0;
      const double f = fma(S[I][NB - 2], 0x1p-38, S[I][NB - 1]) * c.mtop;
      const double qq = rint(f);
#pragma unroll
      for (int l = 0; l < NB; ++l) S[I][l] = fma(-qq, c.M38[l], S[I][l]);
      normalise38<NB>(S[I]);
      tr[L & 15][rr] = round38<NB>(S[I], si + tj);
    }
  }
  __syncthreads();
  const bool nofb = (d.flags & 8u) != 0;       // OZ2_NO_FALLBACK
  const bool force = (d.flags & 16u) != 0;     // OZ2_FORCE_FALLBACK
  if (srow < d.m && !(!nofb && (force || (fA[srow] & (OZ2_T1 | OZ2_T2))))) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int cc = (t >> 7) + 2 * j, col = cb * 16 + cc;
      if (col < d.n && (nofb || !(fB[col] & (OZ2_T1 | OZ2_T2)))) {
        const double v = tr[cc][t & 127];
        __builtin_nontemporal_store(ACC ? cin[j] + v : v, C + (size_t)col * ldc + srow);
      }
    }
  }
  // the fallback's panel: the first `cap` flagged rows of A, gathered once
  // (grid-stride over (row of the list, k); nothing to do without flags)
  if (nflag > 0) {
    panel = zws(panel, z);
    listA = zws(listA, z);
    A += (size_t)blockIdx.z * bt.sA;
    const int na = min(nflag, cap);
    const size_t total = (size_t)na * d.k, step = (size_t)gridDim.x * blockDim.x;
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + t; idx < total; idx += step) {
      const size_t l = idx / na;
      const int r = (int)(idx - l * na);
      panel[r + l * cap] = A[(size_t)listA[r] + l * lda];
    }
  }
}

int crt_blocks(const Oz2Dims& d) { return ((d.m + 127) / 128) * ((d.n + 15) / 16); }

template <int N>
void launch_crt_n(const Oz2Dims& d, const Oz2Layout& L, const Oz2Byte& c, uint8_t* ws,
                  const double* A, int lda, const double* B, int ldb, double* C, int ldc,
                  const Oz2Batch& bt, hipStream_t s) {
  const int nrow = (d.m + 127) / 128, ncrt = crt_blocks(d);
  const bool fb = oz2_byte_crt_takes_fallback(d, bt);
  // OZ2_NO_FALLBACK: no fallback, no panel
  const bool gather = !(d.flags & 8u) && !fb;
  const bool acc = (d.flags & 1u) != 0;
  auto kern = fb ? (acc ? k_byte_crt<N, true, true> : k_byte_crt<N, false, true>)
                 : (acc ? k_byte_crt<N, true, false> : k_byte_crt<N, false, false>);
  const int nfb = fb ? std::max(1, std::min(2 * ((d.m + 63) / 64) * ((d.n + 31) / 32), 256 / bt.count)) : 0;
  hipLaunchKernelGGL(kern, dim3((unsigned)(ncrt + nfb), 1, bt.count), dim3(256), 0, s, c, d,
                     ws + L.res, (const int32_t*)(ws + L.sA), (const int32_t*)(ws + L.tB),
                     (const uint32_t*)(ws + L.flagsA), (const uint32_t*)(ws + L.flagsB), C, ldc, A,
                     lda, (const int*)(ws + L.counters), (const int*)(ws + L.listA),
                     gather ? (double*)(ws + L.panel) : nullptr, d.mp < OZ2_FBCAP ? d.mp : OZ2_FBCAP,
                     nrow, B, ldb, (const int*)(ws + L.listB), ncrt, bt);
}

}  // namespace

hipError_t oz2_launch_byte_split(const Oz2Dims& d, const Oz2Layout& L, const Oz2Const& c,
                                 const Oz2Byte& b, uint8_t* ws, const double* A, int lda,
                                 const double* B, int ldb, const Oz2Batch& bt, hipStream_t s) {
  const unsigned tz = (d.flags & 4u) ? 1u : 0u;   // OZ2_QUANT_TZ
  const int force = (d.flags & 16u) ? 1 : 0;      // OZ2_FORCE_FALLBACK
  const unsigned long long fixedR = (d.flags & 2u) ? 256ull * (unsigned long long)d.k : 0ull;
  const bool vec = (uintptr_t)B % 16 == 0 && ldb % 2 == 0 && bt.sB % 2 == 0;
  const int nkb = d.kp / 64;
  const ByteSide SA{A, lda, d.m, d.mp, (d.m + 63) / 64 * nkb, (const unsigned long long*)(ws + L.rowbits),
                    (const uint32_t*)(ws + L.Rmax), d.cslabs, c.cA, fixedR, (int32_t*)(ws + L.sA),
                    (uint32_t*)(ws + L.flagsA), ws + L.planesA, 0u, (int*)(ws + L.counters),
                    (int*)(ws + L.listA), force, force, bt.sA};
  const ByteSide SB{B, ldb, d.n, d.np, (d.n + 63) / 64 * nkb, (const unsigned long long*)(ws + L.colbits),
                    (const uint32_t*)(ws + L.Kmax), d.cslabs, c.cB, fixedR, (int32_t*)(ws + L.tB),
                    (uint32_t*)(ws + L.flagsB), ws + L.planesB, vec ? 1u : 0u,
                    (int*)(ws + L.counters) + 1, (int*)(ws + L.listB), force, 0, bt.sB};
  // Few tiles: the moduli in up to five shares, each reading the tile again, so that
  // the chain of a tile's 15 to 19 residues does not set the time (256^3: 32
  // tiles, 9.0 us in one share).
  const long long tiles = (long long)(SA.ntiles + SB.ntiles) * bt.count;
  const int shares = (int)std::max(1ll, std::min(5ll, 2ll * oz2_device_cus() / tiles));
  const int share = (b.n + shares - 1) / shares;
  hipLaunchKernelGGL(k_byte_split, dim3(SA.ntiles + SB.ntiles, (b.n + share - 1) / share, bt.count),
                     dim3(256), 0, s, b, SA, SB, d.k, d.kp, tz, share, bt.ws);
  return hipGetLastError();
}

// One launch less where few workgroups reconstruct (us per product: 256^3 29.2 -> 28.1,
// 24 x (200 x 136 x 300), 432 workgroups, 63.9 -> 61.1); the fallback's registers and LDS
// cost the others more once they share CUs (777 x 1301 x 995, 574: 77.8 -> 78.5).
bool oz2_byte_crt_takes_fallback(const Oz2Dims& d, const Oz2Batch& bt) {
  return !(d.flags & 8u) && (long long)crt_blocks(d) * bt.count <= 2ll * oz2_device_cus();
}

hipError_t oz2_launch_byte_crt(const Oz2Dims& d, const Oz2Layout& L, const Oz2Byte& c, uint8_t* ws,
                               const double* A, int lda, const double* B, int ldb, double* C, int ldc,
                               const Oz2Batch& bt, hipStream_t s) {
  switch (c.n) {
    case 10: launch_crt_n<10>(d, L, c, ws, A, lda, B, ldb, C, ldc, bt, s); break;
    case 11: launch_crt_n<11>(d, L, c, ws, A, lda, B, ldb, C, ldc, bt, s); break;
    case 12: launch_crt_n<12>(d, L, c, ws, A, lda, B, ldb, C, ldc, bt, s); break;
    case 13: launch_crt_n<13>(d, L, c, ws, A, lda, B, ldb, C, ldc, bt, s); break;
    case 15: launch_crt_n<15>(d, L, c, ws, A, lda, B, ldb, C, ldc, bt, s); break;
    case 16: launch_crt_n<16>(d, L, c, ws, A, lda, B, ldb, C, ldc, bt, s); break;
    case 17: launch_crt_n<17>(d, L, c, ws, A, lda, B, ldb, C, ldc, bt, s); break;
    case 18: launch_crt_n<18>(d, L, c, ws, A, lda, B, ldb, C, ldc, bt, s); break;
    case 19: launch_crt_n<19>(d, L, c, ws, A, lda, B, ldb, C, ldc, bt, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
