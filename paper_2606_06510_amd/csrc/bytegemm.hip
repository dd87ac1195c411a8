// Phase 2 of Alg. 1 on byte residues: the route of the one-call products
// (ozaki2_dgemm and its variants).
//
// The exact integer C~ = A~ B~ is bounded by the scales (|C~| <= M/4 up to
// rounding, M the product of the r moduli the caller chose), so any residue
// number system of at least that range gives the same integer.  E4M3 holds
// consecutive integers only up to 16, so a nine-bit modulus takes three plane
// products there; gfx950 multiplies int8 at the same rate as E4M3, and a
// modulus of at most 256 is ONE product with exact int32 sums: 15 products
// instead of 36 at r = 12, 18 instead of 45 at r = 15 (Oz2Byte).  Measured on
// operands uniform over their range, read from LDS, the 16x16x64 instruction
// sustains 3.5 POP/s and the 32x32x32 one 3.0 (the E4M3 digits 3.6): the chip
// is power-limited, and the smaller tile toggles less.
//
// Operands are K-blocked byte planes ([k/64][rows][64 B], one per modulus, the
// planes of consecutive moduli adjacent), so that a workgroup's whole run --
// all k of one modulus, then the next modulus -- is one linear DMA stream.
// Accumulators start at a multiple of m large enough to make every sum
// non-negative; the residue is then sum - m floor(sum / m), one high multiply,
// a shift and one multiply-add (exact: see reduce()), of which the low byte is
// stored.
//
// Residue layout: 1 KiB units of 64 rows x 16 columns per modulus, unit
// (column block) * (rows_pad / 64) + row block; lane L of a unit holds
// column L%16, rows 16 i + 4 (L/16) + e as byte e of its 32-bit word i (the
// accumulator order of the 16x16 instruction).
#include <algorithm>
#include <cmath>

#include "oz2_tile.h"

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int KS = OZ2_KBLK;

// The residue of a modulus-m accumulator.  a = sum + (a multiple of m) >= 0;
// floor(a / m) by a high multiply with mg = ceil(2^(32+s)/m): the estimate
// exceeds a/m by less than a 2^-(32+s), below 1/m (so the floor is exact) for
//   s = 7: a < 2^30 + 2^9 (k up to 32768 between reductions: |sum| <= 2^29),
//   s = 0: a < 2^24       (k up to 256: |sum| <= 2^22).
// nm = 2^24 - m: the low byte of a + q nm is that of a - q m, a value in
// [0, m).  q < 2^23 fits the 24-bit multiply.
template <bool SHORT>
__device__ __forceinline__ uint32_t reduce(uint32_t a, uint32_t mg, uint32_t nm) {
  uint32_t q = __umulhi(a, mg);
  if (!SHORT) q >>= 7;
  return __umul24(q, nm) + a;
}

// mid-stream reduction (k beyond one exact slab): back to [0, m) plus the offset
template <int NI, int NJ>
__device__ __forceinline__ void fold(v4i (&acc)[NI][NJ], uint32_t mg, uint32_t nm, uint32_t off) {
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc[i][j][e] = (int)((reduce<false>((uint32_t)acc[i][j][e], mg, nm) & 0xFFu) + off);
}

template <int NI, int NJ>
__device__ __forceinline__ void start(v4i (&acc)[NI][NJ], uint32_t off) {
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = v4i{(int)off, (int)off, (int)off, (int)off};
}

// the words of acc (NI row blocks of 16) for column block j, stored as 16-byte
// pieces: unit rows 64 h .. of the wave's rows at dst + 1024 h
template <bool SHORT, int NI, int NJ>
__device__ __forceinline__ void pack(const v4i (&acc)[NI][NJ], uint32_t mg, uint32_t nm,
                                     uint32_t (&w)[NJ][NI]) {
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      uint32_t v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = reduce<SHORT>((uint32_t)acc[i][j][e], mg, nm);
      w[j][i] = low4(v[0], v[1], v[2], v[3]);
    }
}

template <int NI, int NJ>
__device__ __forceinline__ void store(uint8_t* dst, size_t cbs, const uint32_t (&w)[NJ][NI]) {
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int h = 0; h < NI / 4; ++h)
      __builtin_nontemporal_store(
          u32x4{w[j][4 * h], w[j][4 * h + 1], w[j][4 * h + 2], w[j][4 * h + 3]},
          reinterpret_cast<u32x4*>(dst + j * cbs + h * 1024));
}

// ------------------------------------------------ 256 x 256 tiles, ping-pong
// 8 waves (2 per SIMD), each 128 x 64 outputs; a 4-deep ring of 32 KiB stages
// (K = 64), three stages in flight; the two waves of a SIMD run a phase
// apart, so that one's fragment reads and DMA issue lie under the other's 32
// MFMAs.  Barriers and waits as in k_resgemm (gemm.hip), whose operands are
// laid out alike.
constexpr int BT = 256, BNT = 512, BNB = 4;
constexpr int BOP = BT * KS, BST = 2 * BOP;

// The (tile, modulus group) pair of workgroup b of `pairs`, tiles fastest.
// Workgroups go round-robin over the 8 XCDs, each with its own L2: XCD x takes
// a contiguous eighth of the pairs, so that the workgroups sharing a modulus's
// operand panels share an L2.  False: no pair left (the last XCD's share).
__device__ __forceinline__ bool pair_of(int b, int pairs, int tiles, int& tile, int& group) {
  const int per = (pairs + 7) >> 3;
  const int p = (b & 7) * per + (b >> 3);
  if (p >= pairs) return false;
  group = p / tiles;
  tile = p - group * tiles;
  return true;
}

struct Stream {
  const uint8_t* pa;
  const uint8_t* pb;
  uint32_t vo;   // lane offset of block w (VGPR)
  uint32_t mw;   // w KiB (uniform)
};

__device__ __forceinline__ void big_issue(Stream& d, size_t kbA, size_t kbB, uint32_t lbase) {
  dma16(d.pa, d.vo, lbase + d.mw);
  dma16(d.pa + 8192, d.vo, lbase + d.mw + 8192u);
  dma16(d.pb, d.vo, lbase + BOP + d.mw);
  dma16(d.pb + 8192, d.vo, lbase + BOP + d.mw + 8192u);
  d.pa += kbA;
  d.pb += kbB;
}

// this wave's share of stage s has landed (it has issued stages up to
// min(s + 2, T - 1), four DMA instructions each, returning in order; stages
// below `landed` are known to be in LDS)
__device__ __forceinline__ void big_wait(int s, int T, int landed) {
  if (s >= T || s < landed) return;
  if (s + 2 < T) wait_vm<8>();
  else if (s + 1 < T) wait_vm<4>();
  else wait_vm<0>();
}

__global__ void __launch_bounds__(BNT, 1)
k_bytegemm(Oz2Byte c, const uint8_t* __restrict__ PA, const uint8_t* __restrict__ PB, int mp, int np,
           int kp, int mpw, int pairs, int mgroup, int tbase, uint8_t* __restrict__ res, size_t wsz) {
  __shared__ __attribute__((aligned(16))) uint8_t LB[BNB * BST];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)LB;
  const int ntm = mp / BT, ntn = np / BT;
  int tile, group = mgroup;
  if (pairs) {
    if (!pair_of(blockIdx.x, pairs, ntm * ntn, tile, group)) return;
  } else {
    tile = tile_of(tbase + blockIdx.x, ntm, ntn);
  }
  const int mi0 = group * mpw, mi1 = min(c.n, mi0 + mpw);
  const int tm = tile % ntm, tn = tile / ntm;
  const size_t kbA = (size_t)mp * KS, kbB = (size_t)np * KS;
  const int nk = kp / KS, T = nk * (mi1 - mi0);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = w >> 2;
  Stream d;
  {
    const int rb = lane >> 2;
    d.vo = (uint32_t)(rb * KS + 16 * ((lane & 3) ^ swz16(rb))) + (uint32_t)w * 1024u;
    d.mw = (uint32_t)w * 1024u;
    const size_t z = (size_t)blockIdx.z * wsz;
    d.pa = PA + z + (size_t)tm * BT * KS + (size_t)mi0 * nk * kbA;
    d.pb = PB + z + (size_t)tn * BT * KS + (size_t)mi0 * nk * kbB;
    res += z;
  }
#pragma unroll
  for (int t = 0; t < BNB - 1; ++t)
    if (t < T) big_issue(d, kbA, kbB, lds0 + t * BST);
  big_wait(0, T, 0);
  bar();
  if (g) bar();

  const int wr = w >> 2, wc = w & 3;
  const int fo = (lane & 15) * KS + 16 * ((lane >> 4) ^ swz16(lane & 15));
  const uint8_t* fa0 = LB + wr * 128 * KS + fo;
  const uint8_t* fb0 = LB + BOP + wc * 64 * KS + fo;
  // first unit of the wave's outputs: column block 4 wc (of 16 columns), row block 2 wr (of 64)
  const size_t cbs = (size_t)(mp / 64) * 1024;
  const size_t unit = ((size_t)(tn * 16 + wc * 4) * (mp / 64) + tm * 4 + wr * 2) * 1024;
  int it = 0, landed = 0;
  for (int mi = mi0; mi < mi1; ++mi) {
    const uint32_t mg = c.mg7[mi], nm = c.nm[mi], off = c.off7[mi];
    v4i acc[8][4];
    start(acc, off);
    for (int k0 = 0; k0 < nk; k0 += OZ2_KSLAB / KS) {
      if (k0) fold(acc, mg, nm, off);
      const int end = it + min(nk - k0, OZ2_KSLAB / KS);
      for (; it < end; ++it) {
        if (it + 3 < T) big_issue(d, kbA, kbB, lds0 + ((it + 3) & 3) * BST);
        const int so = (it & 3) * BST;
        v4i fa[8], fb[4];
#pragma unroll
        for (int i = 0; i < 8; ++i) fa[i] = frag(fa0 + so + i * 16 * KS);
#pragma unroll
        for (int j = 0; j < 4; ++j) fb[j] = frag(fb0 + so + j * 16 * KS);
        wait_lgkm0();
        if (g) big_wait(it + 1, T, landed);
        bar();
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[i], fb[j], acc[i][j], 0, 0, 0);
        if (!g) big_wait(it + 1, T, landed);
        bar();
      }
    }
    uint32_t wd[4][8];
    pack<false>(acc, mg, nm, wd);
    // the DMAs issued so far (up to three stages of the next modulus) land
    // before the stores go out, which share their counter
    wait_vm<0>();
    landed = it + 3;
    store(res + (size_t)mi * mp * np + unit + lane * 16, cbs, wd);
  }
  if (!g) bar();
  wait_vm<0>();
}

// ------------------------------------------------ 128 x 128 tiles
// For products with too few 256 x 256 tiles to fill the chip, and for the
// shortest k, where a tile's start, residue epilogue and stores are long beside
// its MFMAs: one modulus per workgroup, 256 threads (4 waves, 64 x 64 outputs each), a 3-deep ring of 16 KiB
// stages, one barrier per stage, three independent workgroups per CU, so that
// one's epilogue lies under the others' MFMAs.
constexpr int ST = 128, SNT = 256, SNB = 3;
constexpr int SOP = ST * KS, SST = 2 * SOP;

__device__ __forceinline__ void small_issue(Stream& d, size_t kbA, size_t kbB, uint32_t lbase) {
  dma16(d.pa, d.vo, lbase + d.mw);
  dma16(d.pa + 4096, d.vo, lbase + d.mw + 4096u);
  dma16(d.pb, d.vo, lbase + SOP + d.mw);
  dma16(d.pb + 4096, d.vo, lbase + SOP + d.mw + 4096u);
  d.pa += kbA;
  d.pb += kbB;
}

// stages it0 .. it0 + n - 1 of T into acc.  A wave's share of stage `it` is four
// DMA instructions, issued two stages ahead; after the barrier every share has
// landed and stage it - 1 has been read by all, so its slot takes stage it + 2.
__device__ __forceinline__ void small_stages(Stream& d, size_t kbA, size_t kbB, const uint8_t* fa0,
                                             const uint8_t* fb0, uint32_t lds0, int T, int it0, int n,
                                             v4i (&acc)[4][4]) {
  int slot = it0 % SNB;
  for (int it = it0; it < it0 + n; ++it) {
    if (it + 1 < T) wait_vm<4>();
    else wait_vm<0>();
    bar();
    if (it + SNB - 1 < T) small_issue(d, kbA, kbB, lds0 + (slot == 0 ? SNB - 1 : slot - 1) * SST);
    const int so = slot * SST;
    slot = slot == SNB - 1 ? 0 : slot + 1;
    v4i fa[4], fb[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) fa[i] = frag(fa0 + so + i * 16 * KS);
#pragma unroll
    for (int j = 0; j < 4; ++j) fb[j] = frag(fb0 + so + j * 16 * KS);
    wait_lgkm0();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[i], fb[j], acc[i][j], 0, 0, 0);
  }
}

template <bool SHORT>
__global__ void __launch_bounds__(SNT, 3)
k_bytegemm128(Oz2Byte c, const uint8_t* __restrict__ PA, const uint8_t* __restrict__ PB, int mp,
              int np, int kp, int ntm, int ntn, int pairs, uint8_t* __restrict__ res, size_t wsz) {
  __shared__ __attribute__((aligned(16))) uint8_t LB[SNB * SST];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)LB;
  int tile, mi;
  if (!pair_of(blockIdx.x, pairs, ntm * ntn, tile, mi)) return;
  const int tm = tile % ntm, tn = tile / ntm;
  const size_t kbA = (size_t)mp * KS, kbB = (size_t)np * KS;
  const int T = kp / KS;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Stream d;
  {
    const int rb = lane >> 2;
    d.vo = (uint32_t)(rb * KS + 16 * ((lane & 3) ^ swz16(rb))) + (uint32_t)w * 1024u;
    d.mw = (uint32_t)w * 1024u;
    const size_t z = (size_t)blockIdx.z * wsz;
    d.pa = PA + z + (size_t)tm * ST * KS + (size_t)mi * T * kbA;
    d.pb = PB + z + (size_t)tn * ST * KS + (size_t)mi * T * kbB;
    res += z;
  }
#pragma unroll
  for (int t = 0; t < SNB - 1; ++t)
    if (t < T) small_issue(d, kbA, kbB, lds0 + t * SST);
  const int wr = w >> 1, wc = w & 1;
  const int fo = (lane & 15) * KS + 16 * ((lane >> 4) ^ swz16(lane & 15));
  const uint8_t* fa0 = LB + wr * 64 * KS + fo;
  const uint8_t* fb0 = LB + SOP + wc * 64 * KS + fo;
  const size_t cbs = (size_t)(mp / 64) * 1024;
  const size_t unit = ((size_t)(tn * 8 + wc * 4) * (mp / 64) + tm * 2 + wr) * 1024;
  const uint32_t mg = SHORT ? c.mg0[mi] : c.mg7[mi], nm = c.nm[mi];
  const uint32_t off = SHORT ? c.off0[mi] : c.off7[mi];
  v4i acc[4][4];
  start(acc, off);
  for (int k0 = 0; k0 < T; k0 += OZ2_KSLAB / KS) {
    if (k0) fold(acc, mg, nm, off);
    small_stages(d, kbA, kbB, fa0, fb0, lds0, T, k0, min(T - k0, OZ2_KSLAB / KS), acc);
  }
  uint32_t wd[4][4];
  pack<SHORT>(acc, mg, nm, wd);
  store(res + (size_t)mi * mp * np + unit + lane * 16, cbs, wd);
}

// ------------------------------------------------ code products, 128 x 128 tiles
// The max-magnitude pass on integer code bytes (0..16), where the E4M3 kernel's
// 256 x 256 tiles are too few: the loop above for one "modulus", the
// epilogue row and column maxima.  Exact: |sums| <= 256 k, one code slab.

// One halving step of a maximum over lanes L and L^B: of the first 2 N entries of
// u, lane L keeps the half selected by bit B of L.
template <int N, int B>
__device__ __forceinline__ void halve(int (&u)[16], int lane) {
  const bool up = (lane & B) != 0;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int keep = up ? u[k + N] : u[k], send = up ? u[k] : u[k + N];
    u[k] = max(keep, __shfl_xor(send, B));
  }
}

__global__ void __launch_bounds__(SNT, 3)
k_codegemm128(const uint8_t* __restrict__ PA, const uint8_t* __restrict__ PB, int mp, int np, int kp,
              int ntm, uint32_t* Rmax, uint32_t* Kmax, size_t wsz) {
  __shared__ __attribute__((aligned(16))) uint8_t LB[SNB * SST];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)LB;
  const int tm = (int)blockIdx.x % ntm, tn = (int)blockIdx.x / ntm;
  const size_t kbA = (size_t)mp * KS, kbB = (size_t)np * KS, z = (size_t)blockIdx.z * wsz;
  const int T = kp / KS;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Stream d;
  {
    const int rb = lane >> 2;
    d.vo = (uint32_t)(rb * KS + 16 * ((lane & 3) ^ swz16(rb))) + (uint32_t)w * 1024u;
    d.mw = (uint32_t)w * 1024u;
    d.pa = PA + z + (size_t)tm * ST * KS;
    d.pb = PB + z + (size_t)tn * ST * KS;
  }
#pragma unroll
  for (int t = 0; t < SNB - 1; ++t)
    if (t < T) small_issue(d, kbA, kbB, lds0 + t * SST);
  const int wr = w >> 1, wc = w & 1;
  const int fo = (lane & 15) * KS + 16 * ((lane >> 4) ^ swz16(lane & 15));
  v4i acc[4][4];
  start(acc, 0);
  small_stages(d, kbA, kbB, LB + wr * 64 * KS + fo, LB + SOP + wc * 64 * KS + fo, lds0, T, 0, T, acc);
  // lane (g, c): rows 16 i + 4 g + e, columns 16 j + c of the wave's 64 x 64
  const int g = lane >> 4, c = lane & 15;
  int u[16], v[16];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      u[4 * i + e] = max(max(acc[i][0][e], acc[i][1][e]), max(acc[i][2][e], acc[i][3][e]));
  halve<8, 8>(u, lane);
  halve<4, 4>(u, lane);
  halve<2, 2>(u, lane);
  halve<1, 1>(u, lane);
  // entry c of the 16: i = c / 4, e = c % 4
  uint32_t* R = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(Rmax) + z) + tm * ST + wr * 64;
  atomicMax(R + 16 * (c >> 2) + 4 * g + (c & 3), (uint32_t)u[0]);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int x = acc[0][j][0];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) x = max(x, acc[i][j][e]);
    v[j] = x;
  }
  halve<2, 32>(v, lane);
  halve<1, 16>(v, lane);
  uint32_t* K = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(Kmax) + z) + tn * ST + wc * 64;
  atomicMax(K + 16 * g + c, (uint32_t)v[0]);
}

}  // namespace

// One code slab, and by the times below: 0.37 us per stage + 4 for a 128-tile
// workgroup alone on its CU (0.80 with two beside it) against 0.82 + 6 for a
// 256-tile one of the E4M3 kernel.
bool oz2_codegemm128_fits(const Oz2Dims& d, const Oz2Batch& bt) {
  if (d.cslabs != 1) return false;
  const double cus = oz2_device_cus(), nk = d.kp / KS;
  const double small = (double)((d.m + ST - 1) / ST) * ((d.n + ST - 1) / ST) * bt.count;
  const double big = (double)(d.mp / BT) * (d.np / BT) * bt.count;
  const double t_small = small <= cus ? 0.37 * nk + 4.0
                                      : std::max(1.0, small / (3.0 * cus)) * (0.80 * nk + 1.8) + 3.0;
  return t_small < std::ceil(big / cus) * (0.82 * nk + 6.0);
}

hipError_t oz2_launch_codegemm128(const Oz2Dims& d, const Oz2Layout& L, uint8_t* ws,
                                  const Oz2Batch& bt, hipStream_t s) {
  const int ntm = (d.m + ST - 1) / ST, ntn = (d.n + ST - 1) / ST;
  hipLaunchKernelGGL(k_codegemm128, dim3(ntm * ntn, 1, bt.count), dim3(SNT), 0, s, ws + L.codesA,
                     ws + L.codesB, d.mp, d.np, d.kp, ntm, (uint32_t*)(ws + L.Rmax),
                     (uint32_t*)(ws + L.Kmax), bt.ws);
  return hipGetLastError();
}

// Which kernel, and how many moduli a workgroup walks.  Measured times (us,
// one MI355X) fit: a 256-tile workgroup 0.82 per K-stage + 3.3 per modulus
// (+ 3 a round of one workgroup per CU); a 128-tile workgroup 0.37 per stage
// + 4 alone on its CU, 0.80 per stage + 1.8 with two more beside it, one
// modulus each (more never won).  For instance (128-tile / 256-tile kernel):
// 256^3 5.2 / 9.8, 512^3 7.8 / 13.6, 300 x 300 x 8192 50 / 90,
// 1024 x 1024 x 8192 143 / 102, 2048^3 126 / 116, 4096^2 x 1024 261 / 244,
// 16384^2 x 128 1123 / 1186, 4096^3 1088 / 785 (r = 12).
hipError_t oz2_launch_bytegemm(const Oz2Dims& d, const Oz2Layout& L, const Oz2Byte& c, uint8_t* ws,
                               const Oz2Batch& bt, hipStream_t s) {
  const double cus = oz2_device_cus();
  const int nk = d.kp / KS, n = c.n;
  const long long tb = (long long)(d.mp / BT) * (d.np / BT);
  const int ntm = (d.m + ST - 1) / ST, ntn = (d.n + ST - 1) / ST;
  const long long ts = (long long)ntm * ntn;
  const uint8_t *pa = ws + L.planesA, *pb = ws + L.planesB;
  uint8_t* res = ws + L.res;

  const double ws_small = (double)ts * n * bt.count;
  const double t_small = ws_small <= cus ? 0.37 * nk + 4.0
                                         : std::max(1.0, ws_small / (3.0 * cus)) * (0.80 * nk + 1.8) + 3.0;
  int mpw = 1;
  double t_big = -1.0;
  for (int q = 1; q <= n; ++q) {
    const double wgs = (double)tb * bt.count * ((n + q - 1) / q);
    const double rounds = wgs <= 4.0 * cus ? std::ceil(wgs / cus) : wgs / cus;
    const double t = rounds * (q * (0.82 * nk + 3.3) + (rounds > 4.0 ? 0.0 : 3.0));
    if (t_big < 0.0 || t < t_big) {
      t_big = t;
      mpw = q;
    }
  }
  if (t_small < t_big) {
    const long long pairs = ts * n;
    auto kern = d.kp <= 256 ? k_bytegemm128<true> : k_bytegemm128<false>;
    hipLaunchKernelGGL(kern, dim3((unsigned)((pairs + 7) / 8 * 8), 1, bt.count), dim3(SNT), 0, s, c,
                       pa, pb, d.mp, d.np, d.kp, ntm, ntn, (int)pairs, res, bt.ws);
    return hipGetLastError();
  }
  // Many tiles: whole rounds of tiles per launch, one modulus group at a time,
  // so that the workgroups sharing operand panels start together and meet in
  // L2 (16384^3, r = 15: 60 ms against 71-73 in one launch; 8192^3, r = 12:
  // 6.4 against 6.8-7.6).  Not where the last launch would leave the chip
  // mostly idle (300 tiles: 44 of 256).
  const int round = (int)((cus + 255) / 256) * 256;
  const long long full = (tb + round - 1) / round * round;
  if (tb > round && (double)full <= 1.15 * (double)tb) {
    mpw = std::min(n, std::max(1, 768 / nk));
    const int groups = (n + mpw - 1) / mpw;
    mpw = (n + groups - 1) / groups;
    const int chunk = nk * mpw >= 384 ? round : 4 * round;
    for (int g = 0; g < groups; ++g)
      for (long long t0 = 0; t0 < tb; t0 += chunk) {
        hipLaunchKernelGGL(k_bytegemm, dim3((unsigned)std::min<long long>(chunk, tb - t0), 1, bt.count),
                           dim3(BNT), 0, s, c, pa, pb, d.mp, d.np, d.kp, mpw, 0, g, (int)t0, res, bt.ws);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
    return hipSuccess;
  }
  const long long pairs = tb * ((n + mpw - 1) / mpw);
  hipLaunchKernelGGL(k_bytegemm, dim3((unsigned)((pairs + 7) / 8 * 8), 1, bt.count), dim3(BNT), 0, s, c,
                     pa, pb, d.mp, d.np, d.kp, mpw, (int)pairs, 0, 0, res, bt.ws);
  return hipGetLastError();
}
