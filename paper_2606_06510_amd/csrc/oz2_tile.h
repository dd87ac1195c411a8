// Device helpers shared by the LDS-ring GEMMs of gemm.hip (E4M3 planes),
// bytegemm.hip and bytefused.hip (byte residues), and by the other byte kernels:
// pinned barriers and waits, the LDS DMA and its chunk swizzle, int8 fragments,
// byte packing, and the block -> tile mapping.
#pragma once
#include "oz2_internal.h"

namespace {

typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef int v4i __attribute__((ext_vector_type(4)));

// s_barrier pinned in the instruction stream: the scheduler moves nothing
// (not even register-only MFMAs) across it, so the phases below stay phases
__device__ __forceinline__ void bar() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
__device__ __forceinline__ void wait_lgkm0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// chunk swizzle of LDS row r: conflict free for 16 consecutive rows
__device__ __forceinline__ int swz(int r) { return ((r >> 1) & 3) ^ ((r >> 3) & 1); }

// The same for fragments of 16 rows x 64 k bytes (lane L: row L%16, chunk L/16):
// a 16-byte LDS read serves lanes 0-3, 12-15 and 20-27 together (likewise the
// complements), rows 0-3, 12-15 of one chunk and 4-11 of the next; the swizzle
// of 32-row fragments above is two-way conflicted there (four extra cycles
// per read, the matrix unit busy 60% of the cycles at 4096^3).
__device__ __forceinline__ int swz16(int r) { return (-(r >> 2)) & 3; }

// operand fragment of 16 rows x 64 k: lane L holds row L%16, k 16 (L/16) .. +15
// (the logical chunk L/16 of the row at its swizzled place)
__device__ __forceinline__ v4i frag(const uint8_t* p) {
  const uint4 v = *reinterpret_cast<const uint4*>(p);
  return v4i{(int)v.x, (int)v.y, (int)v.z, (int)v.w};
}

// the low bytes of four words, packed
__device__ __forceinline__ uint32_t low4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const uint32_t lo = __builtin_amdgcn_perm(b, a, 0x0c0c0400u);
  const uint32_t hi = __builtin_amdgcn_perm(d, c, 0x04000c0cu);
  return lo | hi;
}

// global_load_lds_dwordx4: lane L's 16 bytes land at M0 + 16 L.  The sc1
// cache policy (streaming operands with no reuse inside the CU's vector L1)
// measured 10-12% faster than the default policy on the 4096^3 residue GEMMs.
__device__ __forceinline__ void dma16(const uint8_t* sbase, uint32_t voff, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 sc1" ::"v"(voff), "s"(sbase),
               "s"(m0)
               : "memory");
}

// Tile of block b.  Blocks are dispatched round-robin over the 8 XCDs (each
// with its own L2); when the grid allows it each XCD gets a 4x8 group of
// tiles per 256-block round (4 A row panels, 8 B column panels).
__device__ __forceinline__ int tile_of(int b, int ntm, int ntn) {
  if ((ntm % 4) || (ntn % 8) || ((ntm * ntn) % 256)) return b;
  const int xcd = b & 7, slot = b >> 3;
  const int grp = slot >> 5, in = slot & 31;
  const int gid = grp * 8 + xcd, ngx = ntm / 4;
  const int gm = gid % ngx, gn = gid / ngx;
  return (gm * 4 + (in & 3)) + (gn * 8 + (in >> 2)) * ntm;
}

}  // namespace
