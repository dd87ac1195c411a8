// The byte-residue products and their CRT reconstruction in one kernel, for
// short k: residues never leave the chip.
//
// At k = 256 the staged route writes and reads 15 bytes of residues per output
// beside the 16 bytes of C that C += A B has to move, and its two kernels take
// 6.7 and 6.2 ms of a rank-256 update of 32768^2.  Here a workgroup walks all
// moduli of its 128 x 128 tile; each output's residues stay packed in four
// registers (16 bytes), 256 KiB of a CU's 512 KiB of registers, which is what
// sets the tile.  The tiles of an XCD go in 4 x 8 groups that share panels in
// its L2, and a persistent workgroup has the next tile's first stages in
// flight while it reconstructs.  Measured (staged -> fused, us, r = 12):
// 32768^2 x 256 (C += A B) 12490 -> 11070, 16384^2 x 64 2550 -> 1960,
// 4096^2 x 256 270 -> 202; 16384^2 x 512 3930 -> 4070, where the staged
// products' 256 x 256 tiles win.  What bounds it: vector issue (144
// instructions per output and lane, 60% of the slots at k = 64) and the
// products' stages, one after the other within a workgroup.  Two workgroups of
// 128 x 64 per CU (half as much operand traffic more) took 12290 at k = 256, and
// reading the next stage's fragments under a stage's products 11780.
//
// Reconstruction on the matrix units: the sums sum_i u_i W_i of all byte limbs
// of W_i are int8 products too.  Output (row 4 g + e, column c) of a 16 x 16
// block sits in lane (g, c), its 16 residue bytes being exactly that lane's 16
// k-bytes of a B operand; with an A operand that holds the limbs of W (row r:
// byte limb r of each W_i) in lane group g' only, one 16x16x64 product gives
// the byte-limb sums of the outputs of group g'.  Four products, five vector
// instructions to join four byte limbs into a radix-2^32 limb and a 4 x 4
// transposition of lane groups (permlane swaps) replace 75 conversions and
// fmas per output.
#include "oz2_tile.h"
#include "oz2_device.h"

namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int KS = OZ2_KBLK;
constexpr int FT = 128, FNT = 512, FNB = 8;    // tile, threads, ring depth
constexpr int FOP = FT * KS, FST = 2 * FOP;    // 8 KiB per operand and stage

// swap the upper half of a's lanes (odd 16-lane rows) with the lower half
// (even rows) of b's
__device__ __forceinline__ void swap32(double& a, double& b) {
  const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
  const u32x2 lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
  const u32x2 hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  a = __longlong_as_double((long long)(((uint64_t)hi.x << 32) | lo.x));
  b = __longlong_as_double((long long)(((uint64_t)hi.y << 32) | lo.y));
}
__device__ __forceinline__ void swap16(double& a, double& b) {
  const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
  const u32x2 lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
  const u32x2 hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  a = __longlong_as_double((long long)(((uint64_t)hi.x << 32) | lo.x));
  b = __longlong_as_double((long long)(((uint64_t)hi.y << 32) | lo.y));
}

// RN-even binary64 value of X 2^-e for X = sum_j S_j 2^(32 j), |S_j| < 2^49, |X| <
// 2^112.  X = H 2^64 + mid 2^32 + lo with |mid| <= 2^31, 0 <= lo < 2^32 (every step
// exact).  Where |H| >= 8 a rounding boundary is at 2^13 or above, so lo may
// be rounded to odd at bit 11: mid 2^32 + lo is then exact (53 bits) and one
// fma rounds X itself; below, H 2^32 + mid is exact and one fma adds lo.
// Subnormal results (|X| 2^-e < 2^-1022 with X an integer: e above 1022, tiny
// inputs) go through 32-bit words, out of line: the caller's code is unrolled
// over many outputs and has to stay in the instruction cache.
__device__ __attribute__((noinline)) double round_words(double H, double mid, double lo, int e) {
  const uint64_t b0 = ((uint64_t)(long long)mid << 32) + (uint64_t)lo;
  const uint64_t b1 = (uint64_t)((long long)H - (mid < 0.0 ? 1 : 0));
  const uint32_t w[4] = {(uint32_t)b0, (uint32_t)(b0 >> 32), (uint32_t)b1, (uint32_t)(b1 >> 32)};
  return round_scaled<4>(w, e);
}

// the exact parts of X, for round_words
struct Parts {
  double H, mid, lo;
};
__device__ __forceinline__ double round_limbs32(const double (&S)[4], int e, Parts& P) {
  const double c0 = floor(S[0] * 0x1p-32);
  const double lo = fma(-c0, 0x1p32, S[0]);
  const double s1 = S[1] + c0;
  const double c1 = rint(s1 * 0x1p-32);
  const double mid = fma(-c1, 0x1p32, s1);
  const double H = fma(S[3], 0x1p32, S[2]) + c1;
  const uint32_t l = (uint32_t)lo;
  const uint32_t odd = (l & 0xFFFFF800u) | ((l & 0x7FFu) ? 0x800u : 0u);
  const double big = fma(H, 0x1p64, fma(mid, 0x1p32, (double)odd));
  const double small = fma(fma(H, 0x1p32, mid), 0x1p32, lo);
  const double v = (fabs(H) < 8.0 ? small : big) + 0.0;   // an exact zero is +0.0
  P.H = H;
  P.mid = mid;
  P.lo = lo;
  return ldexp(v, -e);
}

// as bytegemm.hip's for k <= 256: 0 <= a < 2^24; the low byte is a mod m
__device__ __forceinline__ uint32_t reduce(uint32_t a, uint32_t mg, uint32_t nm) {
  return __umul24(__umulhi(a, mg), nm) + a;
}

struct Stream {
  const uint8_t* pa;
  const uint8_t* pb;
  const uint8_t* na;   // the next tile's panels
  const uint8_t* nb;
  int left;        // stages left in the tile
  uint32_t vo, mw;
};

// tile of the workgroup's t-th turn: its XCD's contiguous share of the tiles,
// taken by the XCD's workgroups in turn; tiles in strips of four tile rows
__device__ __forceinline__ bool tile_at(int t, int tiles, int ntm, int ntn, int& tm, int& tn) {
  const int per = (tiles + 7) >> 3, slots = (int)gridDim.x >> 3;
  const int in = ((int)blockIdx.x >> 3) + t * slots;
  const int p = ((int)blockIdx.x & 7) * per + in;
  if (in >= per || p >= tiles) return false;
  const int strip = p / (4 * ntn), q = p - strip * 4 * ntn;
  const int h = min(4, ntm - 4 * strip);
  tn = q / h;
  tm = 4 * strip + (q - tn * h);
  return true;
}

template <int N, bool ACC>
__global__ void __launch_bounds__(FNT, 1)
k_byte_fused(Oz2Byte c, Oz2Dims d, const uint8_t* __restrict__ PA, const uint8_t* __restrict__ PB,
             const int32_t* __restrict__ sA, const int32_t* __restrict__ tB,
             const uint32_t* __restrict__ fA, const uint32_t* __restrict__ fB, double* C, int ldc,
             int ntm, int ntn, int turns, unsigned vecC) {
  __shared__ __attribute__((aligned(16))) uint8_t LB[FNB * FST];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)LB;
  const int tiles = ntm * ntn;
  const size_t kbA = (size_t)d.mp * KS, kbB = (size_t)d.np * KS;
  const int nk = d.kp / KS, T = N * nk;
  const int lane = threadIdx.x & 63, g = lane >> 4, cl = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Stream s;
  {
    const int rb = lane >> 2;
    s.vo = (uint32_t)(rb * KS + 16 * ((lane & 3) ^ swz16(rb))) + (uint32_t)w * 1024u;
    s.mw = (uint32_t)w * 1024u;
    s.left = 0;
  }
  int tm, tn, mine = 0;
  while (mine < turns && tile_at(mine, tiles, ntm, ntn, tm, tn)) ++mine;
  const int total = mine * T;
  auto issue = [&](int slot) {
    if (s.left == 0) {
      s.pa = s.na;
      s.pb = s.nb;
      s.left = T;
    }
    dma16(s.pa, s.vo, lds0 + slot * FST + s.mw);
    dma16(s.pb, s.vo, lds0 + slot * FST + FOP + s.mw);
    s.pa += kbA;
    s.pb += kbB;
    --s.left;
  };
  // panels of the workgroup's tile t (the stream enters a tile at most seven
  // stages before the products do, so one tile's panels are known ahead)
  auto next = [&](int t) {
    int a = 0, b = 0;
    (void)tile_at(min(t, mine - 1), tiles, ntm, ntn, a, b);
    s.na = PA + (size_t)a * FT * KS;
    s.nb = PB + (size_t)b * FT * KS;
  };
  if (mine == 0) return;
  next(0);
#pragma unroll 1
  for (int q = 0; q < FNB - 1; ++q)
    if (q < total) issue(q);

  // the wave's 64 x 32 outputs
  const int wr = w & 1, wc = w >> 1;
  const int fo = cl * KS + 16 * (g ^ swz16(cl));
  const uint8_t* fa0 = LB + wr * 64 * KS + fo;
  const uint8_t* fb0 = LB + FOP + wc * 32 * KS + fo;
  // byte limb cl of every W_i, in this lane's group only; their sums times 128
  // (the residues enter as u - 128) for byte limbs 4 g .. + 3
  v4i wv = v4i{0, 0, 0, 0}, w0 = v4i{0, 0, 0, 0};
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (cl == r) wv = v4i{c.wb[r][0], c.wb[r][1], c.wb[r][2], c.wb[r][3]};
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (g == r) w0 = v4i{c.woff[4 * r], c.woff[4 * r + 1], c.woff[4 * r + 2], c.woff[4 * r + 3]};
  const bool nofb = (d.flags & 8u) != 0;       // OZ2_NO_FALLBACK
  const bool force = (d.flags & 16u) != 0;     // OZ2_FORCE_FALLBACK

  int it = 0, landed = 0;
  for (int turn = 0; turn < mine; ++turn) {
    next(turn + 1);
    uint32_t pk[4][2][4][4];   // [row block][column block][output][word]
    // (the word of pk is static, the byte within it is not: code for four moduli
    // instead of N, which with the reconstruction below fits the instruction cache)
#pragma unroll
    for (int wd = 0; wd < 4; ++wd) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) pk[i][j][e][wd] = 0;
#pragma unroll 1
      for (int mi = 4 * wd; mi < min(N, 4 * wd + 4); ++mi) {
        const uint32_t mg = c.mg0[mi], nm = c.nm[mi];
        const int off = (int)c.off0[mi];
        v4i acc[4][2];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = v4i{off, off, off, off};
        for (int st = 0; st < nk; ++st, ++it) {
          // this wave's share of stage `it` (two DMA instructions, up to seven
          // stages ahead) has landed; after the barrier every share has, and
          // stage it - 1 has been read by all
          if (it >= landed) {
            if (it + FNB - 2 < total) wait_vm<2 * (FNB - 2)>();
            else wait_vm<0>();
          }
          bar();
          if (it + FNB - 1 < total) issue((it + FNB - 1) & (FNB - 1));
          const int so = (it & (FNB - 1)) * FST;
          v4i fa[4], fb[2];
#pragma unroll
          for (int i = 0; i < 4; ++i) fa[i] = frag(fa0 + so + i * 16 * KS);
#pragma unroll
          for (int j = 0; j < 2; ++j) fb[j] = frag(fb0 + so + j * 16 * KS);
          wait_lgkm0();
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the residue's byte into place
        const int by = 8 * (mi & 3);
        const uint32_t sel = (0x03020100u & ~(0xFFu << by)) | (0x04u << by);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const uint32_t u = reduce((uint32_t)acc[i][j][e], mg, nm);
              uint32_t& p = pk[i][j][e][wd];
              p = __builtin_amdgcn_perm(u, p, sel);
              // formed here: sunk to its use it would keep the accumulators instead
              asm volatile("" : "+v"(p));
            }
      }
    }
    // the stages in flight (the next tile's first seven) land before the loads
    // and stores of C share their counter
    wait_vm<0>();
    landed = it + FNB - 1;
    (void)tile_at(turn, tiles, ntm, ntn, tm, tn);
    const int row0 = tm * FT + wr * 64 + 4 * g, col0 = tn * FT + wc * 32 + cl;
    // scales and flags of the lane's 16 rows and 2 columns (padded arrays);
    // skip: entries left to the fallback or outside C
    int si[4][4], tj[2];
    uint32_t rskip = 0, cskip = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int4 a = *reinterpret_cast<const int4*>(sA + row0 + 16 * i);
      const uint4 f = *reinterpret_cast<const uint4*>(fA + row0 + 16 * i);
      const uint32_t fe[4] = {f.x, f.y, f.z, f.w};
      si[i][0] = a.x;
      si[i][1] = a.y;
      si[i][2] = a.z;
      si[i][3] = a.w;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (row0 + 16 * i + e >= d.m || (!nofb && (force || (fe[e] & (OZ2_T1 | OZ2_T2)))))
          rskip |= 1u << (4 * i + e);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = col0 + 16 * j;
      tj[j] = tB[col];
      if (col >= d.n || (!nofb && (fB[col] & (OZ2_T1 | OZ2_T2)))) cskip |= 1u << j;
    }
    int smax = si[0][0];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) smax = max(smax, si[i][e]);
    const bool tiny = __any(smax + max(tj[0], tj[1]) > 1022);
    auto wide_at = [&](int i, int j) { return vecC && !((rskip >> (4 * i)) & 15u) && !((cskip >> j) & 1u); };
    auto load_c = [&](int i, int j, double (&o)[4]) {
      if (!ACC) return;
      const double* p = C + (size_t)(col0 + 16 * j) * ldc + row0 + 16 * i;
      if (wide_at(i, j)) {
        const double2 a = *reinterpret_cast<const double2*>(p), b = *reinterpret_cast<const double2*>(p + 2);
        o[0] = a.x;
        o[1] = a.y;
        o[2] = b.x;
        o[3] = b.y;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o[e] = (((rskip >> (4 * i + e)) | (cskip >> j)) & 1u) ? 0.0 : p[e];
      }
    };
    double cin[4], cnx[4];
    load_c(0, 0, cin);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // C of the next block is on its way while this one is formed
        if (i < 3 || j < 1) load_c((i + 1) & 3, i < 3 ? j : j + 1, cnx);
        double v[4];
        Parts P[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (e == 0) __builtin_amdgcn_sched_barrier(0);   // one block's registers at a time
          const uint32_t* p = pk[i][j][e];
          const v4i u = v4i{(int)(p[0] ^ 0x80808080u), (int)(p[1] ^ 0x80808080u),
                            (int)((N > 8 ? p[2] : 0u) ^ 0x80808080u),
                            (int)((N > 12 ? p[3] : 0u) ^ 0x80808080u)};
          double S[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const v4i wq = g == q ? wv : v4i{0, 0, 0, 0};
            const v4i b = __builtin_amdgcn_mfma_i32_16x16x64_i8(wq, u, w0, 0, 0, 0);
            S[q] = fma((double)(b[2] + (b[3] << 8)), 0x1p16, (double)(b[0] + (b[1] << 8)));
          }
          // S[q]: limb g of the output of group q -> limb q of this lane's output
          swap32(S[0], S[2]);
          swap32(S[1], S[3]);
          swap16(S[0], S[1]);
          swap16(S[2], S[3]);
          const double qq = rint(fma(S[2], 0x1p-32, S[3]) * c.mtop32);
#pragma unroll
          for (int l = 0; l < 4; ++l) S[l] = fma(-qq, c.M32[l], S[l]);
          v[e] = round_limbs32(S, si[i][e] + tj[j], P[e]);
        }
        if (__builtin_expect(tiny, 0)) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = round_words(P[e].H, P[e].mid, P[e].lo, si[i][e] + tj[j]);
        }
        if (ACC) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = cin[e] + v[e];
        }
        double* p = C + (size_t)(col0 + 16 * j) * ldc + row0 + 16 * i;
        if (wide_at(i, j)) {
          reinterpret_cast<double2*>(p)[0] = make_double2(v[0], v[1]);
          reinterpret_cast<double2*>(p)[1] = make_double2(v[2], v[3]);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (!(((rskip >> (4 * i + e)) | (cskip >> j)) & 1u)) p[e] = v[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) cin[e] = cnx[e];
      }
    }
  }
  wait_vm<0>();
}

template <int N>
void launch_n(const Oz2Dims& d, const Oz2Layout& L, const Oz2Byte& c, uint8_t* ws, double* C, int ldc,
              hipStream_t s) {
  const int ntm = (d.m + FT - 1) / FT, ntn = (d.n + FT - 1) / FT;
  const int per = (ntm * ntn + 7) / 8, slots = (oz2_device_cus() + 7) / 8;
  const int turns = (per + slots - 1) / slots;
  auto kern = (d.flags & 1u) ? k_byte_fused<N, true> : k_byte_fused<N, false>;
  const unsigned vecC = ((uintptr_t)C % 16 == 0 && ldc % 2 == 0) ? 1u : 0u;
  hipLaunchKernelGGL(kern, dim3((unsigned)(8 * (slots < per ? slots : per))), dim3(FNT), 0, s, c, d,
                     ws + L.planesA, ws + L.planesB, (const int32_t*)(ws + L.sA),
                     (const int32_t*)(ws + L.tB), (const uint32_t*)(ws + L.flagsA),
                     (const uint32_t*)(ws + L.flagsB), C, ldc, ntm, ntn, turns, vecC);
}

}  // namespace

// At most 15 moduli (16 residue bytes, |X| < 2^112), which is r <= 12; k up to 256
// (above); and tiles that fill the CUs, in whole turns while there are few (2048^2:
// 256 tiles, 97 -> 91; 1500^2: 144 tiles, 78 -> 90; 3000^2: 576 tiles in three turns,
// 163 -> 168).  With the fewest moduli too (us, staged -> fused, r = 8: 2048^2 x 64 55 ->
// 47, 4096^2 x 256 187 -> 162, 20000^2 x 64 2469 -> 2163, 30000^2 x 16 5570 -> 4792; r = 9:
// 16384^2 x 256 2238 -> 2178).
bool oz2_byte_fused_fits(const Oz2Dims& d, const Oz2Byte& c) {
  if (c.n > 15 || d.kp > 256) return false;
  const long long cus = oz2_device_cus();
  const long long tiles = (long long)((d.m + FT - 1) / FT) * ((d.n + FT - 1) / FT);
  const long long turns = (tiles + cus - 1) / cus;
  return tiles * 5 >= turns * cus * 4;
}

hipError_t oz2_launch_byte_fused(const Oz2Dims& d, const Oz2Layout& L, const Oz2Byte& c, uint8_t* ws,
                                 double* C, int ldc, hipStream_t s) {
  switch (c.n) {
    case 10: launch_n<10>(d, L, c, ws, C, ldc, s); break;
    case 11: launch_n<11>(d, L, c, ws, C, ldc, s); break;
    case 12: launch_n<12>(d, L, c, ws, C, ldc, s); break;
    case 13: launch_n<13>(d, L, c, ws, C, ldc, s); break;
    case 15: launch_n<15>(d, L, c, ws, C, ldc, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
