// Phase 3 of Alg. 1 on gfx950: CRT reconstruction of the exact integer,
// removal of the power-of-two scaling with ONE rounding of the multi-limb
// integer (App. B), and the native-FP64 fallback for flagged rows of A /
// columns of B (Alg. 1, fallback step: rows the scaling cannot certify are
// recomputed in plain FP64; the numerical contract's item (vi)).
//
// Reconstruction.  The integer C~ in [-M/2, M/2) is unique given its r
// residues (Eq. (M-bound)), so any exact CRT algorithm yields the same bits
// as Garner's Eq. (garner).  On this VALU the direct CRT sum is cheaper than
// Garner's r(r-1)/2 dependent modular steps:
//     X = sum_i x_i W_i - q M,  W_i = (M/m_i) ((M/m_i)^-1 mod m_i),
// evaluated exactly in radix-2^38 fp64 limbs (three for r <= 12, four
// above), with q = rint(sum_i x_i W_i/M) estimated from the top limbs (error
// < 2^-24; an exact range check fixes the rare ambiguous case).  The x_i are
// any representatives of the residues with |x_i| <= m_i/2 + 32 <= 577 (what
// the residue GEMM stores): every partial limb sum is then an integer below
// 2^52, and the quotient estimate is as good for them as for centred
// residues.  The residue GEMMs store them offset (u = x + floor(m/2) + 32,
// 12 bits per output): the sums start at minus the offsets' share and add the
// u_i, which gives the same integers.
// The normalised limbs are rounded once to binary64 with the exponent shift
// -(s_i + t_j), including gradual underflow (through 32-bit words) and
// overflow.
#include "oz2_device.h"
#include "oz2_fallback.h"

namespace {

// Thread mapping shared by the reconstruction kernels.  The residue GEMM
// leaves, per modulus, each 32x32 output block (wave w of a 256x256 tile,
// sub-block x, y) as 1024 12-bit slots in its accumulator order: lane L holds
// 16 outputs of column L%32, rows 4(L/32) + 8(e/4) + e%4, e = 0..15, as two
// 96-bit records (e = 0..7, e = 8..15), six words w = 0..5 per lane, stored
// lane-major or pair-major (oz2_pair_records).  Here two threads share a
// lane's 16 (t = 2L + h takes record h: words 3h .. 3h + 2), so the 128
// threads of a block read its 1.5 KiB per modulus; a workgroup of 256 takes
// two blocks.
struct BlockMap {
  size_t roff;      // word offset of the block in a modulus plane
  int lane, h;      // the record: lane L's record h
  int row0, col0;   // block origin in C
  int cl;           // column within the block
  int rb;           // row within the block of output i: rb + 8(i/4) + i%4
  int hb, tt;       // block of the pair, thread within the block
};

__device__ __forceinline__ BlockMap block_map(int mp) {
  BlockMap b;
  const int t = threadIdx.x;
  b.hb = t >> 7;
  b.tt = t & 127;
  const size_t G = (size_t)blockIdx.x * 2 + b.hb;
  const size_t tile = G >> 6;
  const int blk = (int)(G & 63);
  const int ntm = mp / OZ2_TILE;
  const int tm = (int)(tile % ntm), tn = (int)(tile / ntm);
  const int y = blk & 1, x = (blk >> 1) & 3, w = blk >> 3;
  b.row0 = tm * OZ2_TILE + (w >> 2) * 128 + x * 32;
  b.col0 = tn * OZ2_TILE + (w & 3) * 64 + y * 32;
  const int lane = b.tt >> 1, h = b.tt & 1;
  b.cl = lane & 31;
  b.rb = 4 * (lane >> 5) + 16 * h;
  b.roff = tile * (OZ2_TILE * OZ2_TILE / 8 * 3) + (size_t)blk * 384;
  b.lane = lane;
  b.h = h;
  return b;
}

// the thread's record of each modulus (plane: words per modulus).
// Lane-major: words 6 L + 3 h .. + 2, one 12-byte load.  Pair-major: record
// 0 is words 0, 1 (8 bytes at 2 L) and 2 (at 128 + 2 L), record 1 words 3
// (at 129 + 2 L) and 4, 5 (8 bytes at 256 + 2 L).  The residues, C_in and C
// are each touched once: non-temporal loads and stores (3-4% faster
// reconstruction on the 16384^3 and rank-256 workloads).
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
template <int R, bool PAIR>
__device__ __forceinline__ void load_residues(const uint32_t* __restrict__ res, size_t plane,
                                              const BlockMap& b, uint3 (&x)[R]) {
  if constexpr (PAIR) {
    const int o2 = b.h ? 256 + 2 * b.lane : 2 * b.lane, o1 = 128 + 2 * b.lane + b.h;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const uint32_t* q = res + (size_t)i * plane + b.roff;
      const u32x2 p = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(q + o2));
      const uint32_t w = __builtin_nontemporal_load(q + o1);
      x[i] = b.h ? make_uint3(w, p.x, p.y) : make_uint3(p.x, p.y, w);
    }
  } else {
    const int o = 6 * b.lane + 3 * b.h;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const uint32_t* q = res + (size_t)i * plane + b.roff + o;
      x[i] = make_uint3(__builtin_nontemporal_load(q), __builtin_nontemporal_load(q + 1),
                        __builtin_nontemporal_load(q + 2));
    }
  }
}

template <int R, int I>
struct Outputs {
  __device__ __forceinline__ static void run(const Oz2Const& c, const Oz2Dims& d,
                                             const uint3 (&x)[R], const BlockMap& b, int tj,
                                             const int32_t* __restrict__ sA, double (*tr)[33]) {
    const int rr = b.rb + 8 * (I >> 2) + (I & 3);
    const int row = b.row0 + rr;
    const int si = row < d.m ? sA[row] : 0;
    tr[b.cl][rr] = crt38_rounded<R, I>(c, x, si + tj);
    Outputs<R, I + 1>::run(c, d, x, b, tj, sA, tr);
  }
};
template <int R>
struct Outputs<R, 8> {
  __device__ __forceinline__ static void run(const Oz2Const&, const Oz2Dims&, const uint3 (&)[R],
                                             const BlockMap&, int, const int32_t* __restrict__,
                                             double (*)[33]) {}
};

// Reconstruct, rescale and store: the block's 32x32 results go through LDS so
// that each store instruction writes whole 256-byte column segments of C.
// Entries of flagged rows / columns are left to the fallback kernel, which
// follows on the same stream; for it the grid also gathers the first `cap`
// flagged rows of A into a contiguous panel (row r at panel[r + l cap]), read
// once here instead of once per column tile there (nothing to do on inputs
// without flagged rows).  ACC (OZ2_ACCUMULATE): C_in is loaded before the
// CRT work, so that its latency hides behind it.  PAIR: the records are
// pair-major (oz2_pair_records; a separate instantiation, which measured
// 0.4 ms faster on the rank-256 update than one kernel reading both).
template <int R, bool ACC, bool PAIR>
__global__ void __launch_bounds__(256)
k_reconstruct(Oz2Const c, Oz2Dims d, const uint32_t* __restrict__ res,
              const int32_t* __restrict__ sA, const int32_t* __restrict__ tB,
              const uint32_t* __restrict__ fA, const uint32_t* __restrict__ fB, double* C, int ldc,
              const double* __restrict__ A, int lda, const int* __restrict__ counters,
              const int* __restrict__ listA, double* __restrict__ panel, int cap) {
  __shared__ double tr[2][32][33];
  const int nflag = panel ? counters[0] : 0;   // used at the end; loaded early
  const BlockMap b = block_map(d.mp);
  const int rr = b.tt & 31;
  const int row = b.row0 + rr;
  // the thread's outputs in the store phase: row, columns col0 + 4 j + tt/32
  double cin[8];
  if constexpr (ACC) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int col = b.col0 + j * 4 + (b.tt >> 5);
      cin[j] = (row < d.m && col < d.n) ? __builtin_nontemporal_load(C + (size_t)col * ldc + row) : 0.0;
    }
  }
  {
    uint3 x[R];
    load_residues<R, PAIR>(res, (size_t)d.mp * d.np / 8 * 3, b, x);
    const int col = b.col0 + b.cl;
    const int tj = col < d.n ? tB[col] : 0;
    Outputs<R, 0>::run(c, d, x, b, tj, sA, tr[b.hb]);
  }
  __syncthreads();
  const bool nofb = (d.flags & 8u) != 0;       // OZ2_NO_FALLBACK
  const bool force = (d.flags & 16u) != 0;     // OZ2_FORCE_FALLBACK
  if (row < d.m && !(!nofb && (force || (fA[row] & (OZ2_T1 | OZ2_T2))))) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int cc = j * 4 + (b.tt >> 5);
      const int col = b.col0 + cc;
      if (col < d.n && (nofb || !(fB[col] & (OZ2_T1 | OZ2_T2)))) {
        const double v = tr[b.hb][cc][rr];
        __builtin_nontemporal_store(ACC ? cin[j] + v : v, C + (size_t)col * ldc + row);
      }
    }
  }
  // the fallback's panel: grid-stride over (row of the list, k)
  const int na = min(nflag, cap);
  const size_t total = (size_t)na * d.k, step = (size_t)gridDim.x * blockDim.x;
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += step) {
    const size_t l = idx / na;
    const int r = (int)(idx - l * na);
    panel[r + l * cap] = A[(size_t)listA[r] + l * lda];
  }
}

// The exact integer of output I of a thread as NL 32-bit words (two's
// complement, little endian), formed by the routine the reconstruction
// itself uses: radix-2^38 limbs (three for R <= 12, four above).
template <int R, int I, class X>
__device__ __forceinline__ void store_integer(const Oz2Const& c, const X (&x)[R], uint32_t* o) {
  constexpr int NB = Limbs38<R>::value, NW = NB + 1;
  static_assert(NW <= NL, "the exported words hold the limbs");
  uint32_t w[NW];
  double S[NB];
  crt38_limbs<R, I, NB>(c, x, S);
  limbs38_words<NB>(S, w);
  const uint32_t ext = (uint32_t)((int32_t)w[NW - 1] >> 31);
#pragma unroll
  for (int q = 0; q < NL; ++q) o[q] = q < NW ? w[q < NW ? q : 0] : ext;
}

// The rounded value of output I exactly as the reconstruction forms it.
template <int R, int I, class X>
__device__ __forceinline__ double rounded_value(const Oz2Const& c, const X (&x)[R], int e) {
  return crt38_rounded<R, I>(c, x, e);
}

template <int R, int I>
struct IntOut {
  __device__ __forceinline__ static void run(const Oz2Const& c, const Oz2Dims& d,
                                             const uint3 (&x)[R], const BlockMap& b,
                                             uint32_t* out) {
    const int row = b.row0 + b.rb + 8 * (I >> 2) + (I & 3);
    const int col = b.col0 + b.cl;
    if (row < d.m && col < d.n) {
      uint32_t* o = out + ((size_t)col * d.m + row) * NL;
      store_integer<R, I>(c, x, o);
    }
    IntOut<R, I + 1>::run(c, d, x, b, out);
  }
};
template <int R>
struct IntOut<R, 8> {
  __device__ __forceinline__ static void run(const Oz2Const&, const Oz2Dims&, const uint3 (&)[R],
                                             const BlockMap&, uint32_t*) {}
};

// the exact integers themselves, [n][m][5] words (a diagnostic query)
template <int R>
__global__ void __launch_bounds__(256)
k_integers(Oz2Const c, Oz2Dims d, const uint32_t* __restrict__ res, uint32_t* out) {
  const BlockMap b = block_map(d.mp);
  uint3 x[R];
  if (oz2_pair_records(d)) load_residues<R, true>(res, (size_t)d.mp * d.np / 8 * 3, b, x);
  else load_residues<R, false>(res, (size_t)d.mp * d.np / 8 * 3, b, x);
  IntOut<R, 0>::run(c, d, x, b, out);
}

// The reconstruction's integer and rounding routines on given residues (a
// probe): thread t takes residue t of each modulus (res[i n + t], any
// representative x with -(floor(m/2) + 32) <= x <= m/2 + 32, what the residue
// GEMMs store), puts it into a stored record as the residue GEMMs do, and
// writes the exact integer as 5 words and its value rounded with the shift e[t].
template <int R>
__global__ void __launch_bounds__(256)
k_crt_probe(Oz2Const c, const int16_t* __restrict__ res, const int* __restrict__ e, int n,
            uint32_t* __restrict__ words, double* __restrict__ rounded) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  uint3 x[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int u = (int)res[(size_t)i * n + t] + c.m[i] / 2 + 32;   // slot 0 of the record
    x[i] = make_uint3((uint32_t)u & 0xFFFu, 0u, 0u);
  }
  store_integer<R, 0>(c, x, words + (size_t)t * NL);
  rounded[t] = rounded_value<R, 0>(c, x, e[t]);
}

__global__ void __launch_bounds__(256)
k_fallback(Oz2Dims d, const double* __restrict__ A, int lda, const double* __restrict__ B, int ldb,
           double* C, int ldc, const int* __restrict__ counters, const int* __restrict__ listA,
           const int* __restrict__ listB, const uint32_t* __restrict__ fA,
           const double* __restrict__ panel, int cap, Oz2Batch bt) {
  __shared__ FbShared S;
  // The problem of the batch varies fastest: with few tiles each, the busy
  // workgroups are the first of the grid and get a CU of their own (problem
  // after problem, 40 x (300 x 300 x 2000) with three flagged rows each took 1195
  // us, now 1066)
  {
    const size_t z = (size_t)blockIdx.x * bt.ws;
    counters = zws(counters, z);
    listA = zws(listA, z);
    listB = zws(listB, z);
    fA = zws(fA, z);
    if (panel) panel = zws(panel, z);
    A += (size_t)blockIdx.x * bt.sA;
    B += (size_t)blockIdx.x * bt.sB;
    C += (size_t)blockIdx.x * bt.sC;
  }
  const int na = counters[0], nb = counters[1];
  // 64 x 32 tiles where 64 x 64 ones would leave half of the chip idle (the
  // sums' order within an entry does not depend on the tile)
  const long long wide = (long long)((na + FB_T - 1) / FB_T) * ((d.n + FB_T - 1) / FB_T) +
                         (long long)((d.m + FB_T - 1) / FB_T) * ((nb + FB_T - 1) / FB_T);
  const int first = blockIdx.y, stride = gridDim.y;
  if (wide <= 128)
    fallback_tiles<32>(S, d, A, lda, B, ldb, C, ldc, na, nb, listA, listB, fA, panel, cap, first, stride);
  else
    fallback_tiles<64>(S, d, A, lda, B, ldb, C, ldc, na, nb, listA, listB, fA, panel, cap, first, stride);
}

__global__ void k_fill(double* C, int m, int n, int ldc) {
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)m * n) return;
  const size_t j = idx / m, i = idx % m;
  C[i + j * ldc] = 0.0;
}

// one workgroup of 256 threads per two 32x32 output blocks
template <int R>
void launch_reconstruct_r(const Oz2Dims& d, const Oz2Layout& L, const Oz2Const& c, uint8_t* ws,
                          const double* A, int lda, double* C, int ldc, hipStream_t s) {
  const size_t blocks = (size_t)d.mp * d.np / 2048;
  const bool gather = !(d.flags & 8u);   // OZ2_NO_FALLBACK: no fallback, no panel
  const bool pair = oz2_pair_records(d);
  auto kern = (d.flags & 1u) ? (pair ? k_reconstruct<R, true, true> : k_reconstruct<R, true, false>)
                             : (pair ? k_reconstruct<R, false, true> : k_reconstruct<R, false, false>);
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, c, d,
                     (const uint32_t*)(ws + L.res), (const int32_t*)(ws + L.sA),
                     (const int32_t*)(ws + L.tB), (const uint32_t*)(ws + L.flagsA),
                     (const uint32_t*)(ws + L.flagsB), C, ldc, A, lda,
                     (const int*)(ws + L.counters), (const int*)(ws + L.listA),
                     gather ? (double*)(ws + L.panel) : nullptr, std::min(d.mp, OZ2_FBCAP));
}

template <int R>
void launch_integers_r(const Oz2Dims& d, const Oz2Layout& L, const Oz2Const& c, uint8_t* ws,
                       uint32_t* out, hipStream_t s) {
  const size_t blocks = (size_t)d.mp * d.np / 2048;
  hipLaunchKernelGGL(k_integers<R>, dim3((unsigned)blocks), dim3(256), 0, s, c, d,
                     (const uint32_t*)(ws + L.res), out);
}

template <int R>
void launch_crt_probe_r(const Oz2Const& c, const int16_t* res, const int* e, int n,
                        uint32_t* words, double* rounded, hipStream_t s) {
  hipLaunchKernelGGL(k_crt_probe<R>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, c, res, e,
                     n, words, rounded);
}

#define OZ2_R_SWITCH(FN, ...)                 \
  switch (c.r) {                              \
    case 8: FN<8>(__VA_ARGS__); break;        \
    case 9: FN<9>(__VA_ARGS__); break;        \
    case 10: FN<10>(__VA_ARGS__); break;      \
    case 11: FN<11>(__VA_ARGS__); break;      \
    case 12: FN<12>(__VA_ARGS__); break;      \
    case 13: FN<13>(__VA_ARGS__); break;      \
    case 14: FN<14>(__VA_ARGS__); break;      \
    case 15: FN<15>(__VA_ARGS__); break;      \
    case 16: FN<16>(__VA_ARGS__); break;      \
    default: return hipErrorInvalidValue;     \
  }

}  // namespace

hipError_t oz2_launch_reconstruct(const Oz2Dims& d, const Oz2Layout& L, const Oz2Const& c,
                                  uint8_t* ws, const double* A, int lda, double* C, int ldc,
                                  hipStream_t s) {
  OZ2_R_SWITCH(launch_reconstruct_r, d, L, c, ws, A, lda, C, ldc, s)
  return hipGetLastError();
}

hipError_t oz2_launch_integers(const Oz2Dims& d, const Oz2Layout& L, const Oz2Const& c,
                               uint8_t* ws, uint32_t* out, hipStream_t s) {
  OZ2_R_SWITCH(launch_integers_r, d, L, c, ws, out, s)
  return hipGetLastError();
}


hipError_t oz2_launch_crt_probe(const Oz2Const& c, const int16_t* res, const int* e, int n,
                                uint32_t* words, double* rounded, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  OZ2_R_SWITCH(launch_crt_probe_r, c, res, e, n, words, rounded, s)
  return hipGetLastError();
}

// workgroups of each problem: two per CU over the batch, which are resident
// together, and no more than the tiles there can be (an empty launch of 1024 takes
// 2.4-4.6 us, one of 32 under 2)
static unsigned fallback_grid(const Oz2Dims& d, int count) {
  const long long tiles = 2ll * ((d.m + FB_T - 1) / FB_T) * ((d.n + 31) / 32);
  return (unsigned)std::max(1ll, std::min<long long>(tiles, 2 * oz2_device_cus() / count));
}

hipError_t oz2_launch_fallback(const Oz2Dims& d, const Oz2Layout& L, uint8_t* ws, const double* A,
                               int lda, const double* B, int ldb, double* C, int ldc,
                               const Oz2Batch& bt, hipStream_t s) {
  // the lists were filled by the deconstruction (k_scales: T1, k_split: T2;
  // k_byte_split: both), the panel of flagged rows by the reconstruction launch
  hipLaunchKernelGGL(k_fallback, dim3(bt.count, fallback_grid(d, bt.count)), dim3(256), 0, s, d,
                     A, lda, B, ldb, C, ldc, (const int*)(ws + L.counters),
                     (const int*)(ws + L.listA), (const int*)(ws + L.listB),
                     (const uint32_t*)(ws + L.flagsA), (const double*)(ws + L.panel),
                     std::min(d.mp, OZ2_FBCAP), bt);
  return hipGetLastError();
}

hipError_t oz2_launch_fallback_direct(const Oz2Dims& d, const Oz2Layout& L, uint8_t* ws,
                                      const double* A, int lda, const double* B, int ldb,
                                      double* C, int ldc, hipStream_t s) {
  hipLaunchKernelGGL(k_fallback, dim3(1, fallback_grid(d, 1)), dim3(256), 0, s, d, A, lda, B, ldb, C, ldc,
                     (const int*)(ws + L.counters), (const int*)(ws + L.listA),
                     (const int*)(ws + L.listB), (const uint32_t*)(ws + L.flagsA),
                     (const double*)nullptr, 0, Oz2Batch{1, 0, 0, 0, 0});
  return hipGetLastError();
}

hipError_t oz2_launch_fill(double* C, int m, int n, int ldc, hipStream_t s) {
  const size_t total = (size_t)m * n;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, C, m, n, ldc);
  return hipGetLastError();
}
