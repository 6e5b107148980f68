// Device code that the matrix-core products of gsi_mfma.hip, gsi_wide.hip and gsi_basis.hip share.
#pragma once
#include "gsi_device.h"
#include "gsi_mfma.h"

namespace gsi {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // a native vector: loads and stores of it are
                                                              // instructions, not aggregate copies
constexpr int BK = 64;           // the host's unit of the contraction (K is a multiple of it)

// Parts of the contraction of a product over `rows` rows (a device-side count).  It is sized for row_tiles tiles of
// tile_rows rows.  With fewer, the same number of workgroups: each tile is cut into more parts (the workgroups of the row tiles that
// are not there take them).  With more, fewer parts, down to min_parts, as long as they fill the chip: what is cut for
// nothing writes partial sums for nothing.  Tiles of tile_rows rows (gemm_nt: 128, wide_scatter_kernel: 256, whatever the launch's tile): the
// order of a sum is the product's and the count's own.  W r beside the image term, us a call, parts fixed / following the count: 16384 x 4096, 102 of 2048
// rows 137 / 102, all of 512 rows 167 / 106; 4096 x 16384, 51 of 1024 rows 75 / 52; a block, 2048 tokens that all fire
// 1480 / 1414, 102 fired 644 / 632.  A product whose expected rows take one part has the launch of the sums all the same:
// 16384 x 4096, 410 of 2048 rows 139 / 143.
constexpr int kUnits = 256;      // compute units: one workgroup each
constexpr int kMaxDepth = 64;    // k-tiles of 64 columns per workgroup, where a product has fewer tiles than the chip units
constexpr int kFewParts = 8;
constexpr int kMinDepth = 8;     // k-tiles that a split keeps at least
__device__ __forceinline__ int parts_for(const GemmProb& g, int rows) {
  if (!g.row_tiles) return g.splits;
  const int tiles = (rows + g.tile_rows - 1) / g.tile_rows, want = g.splits * g.row_tiles;
  if (tiles <= g.row_tiles) return min(max(g.splits, min(kFewParts, g.K / (BK * kMinDepth))), want / tiles);
  const int fit = max(want, (g.row_tiles > 1 ? kUnits / 2 : kUnits) / g.col_tiles) / tiles;
  return min(g.splits, max(g.min_parts, fit));
}

// ONCE: how many of the rows of a launch go past the caches.  1: R and Y as they are written, the fired rows of Y and the partial
// sums of a scatter product as they are read again; 2: x of a residual as well.  The calls that ask for it read and write
// more than the memory-side cache has room for (passes_caches), and what the rows displaced were the operands of the tiles beside
// them.  us a call, through the caches / past them: a block of 2048 tokens at rank 512, 410 fired 730 / 683; the pair 4096 / 16384, 200
// tokens, 30 fired 129 / 114, 333 tokens, 50 fired 148 / 129.  Where all of it fits, the products of the fired rows find R and Y there:
// 4096 x 4096, 1024 tokens that fire 112 / 124, a block of 1024 / 4096, 1000 tokens 126 / 138.  x goes past them where products of the
// fired rows follow (the pair at 333 tokens 133 / 129, none fired 69 / 72), not in a projection by itself (16384 x 256, 4096 tokens 182 /
// 193), and so do the partial sums of such a call's coefficients, as they are added (the same 126.1 / 123.7, rank 512 149.7 / 146.2; a block of
// 2048 tokens, none fired, 408 / 411); those of images of more than 2^19 elements are read through the caches, weights that no cache
// holds: 11008 x 1024 x 512 41.5 / 48.7, 16384 x 1024 x 128 22.4 / 25.1, 3072 x 3072 x 256 24.1 / 24.3; smaller ones past them: 2048 x 2048 x
// 256 18.7 / 16.7, 3072 x 3072 x 128 23.7 / 22.6, 1024 x 4096 x 256 17.8 / 17.1, 8192 x 4096 x 64 28.8 / 28.7.
// (A property of the launch and not of a problem: chosen at run time per row it took 1 to 2 %.)
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <bool PAST>
__device__ __forceinline__ void store_row(float* p, const float4& v) {
  if constexpr (PAST) __builtin_nontemporal_store(f32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<f32x4*>(p));
  else *reinterpret_cast<f32x4*>(p) = f32x4{v.x, v.y, v.z, v.w};
}
template <bool PAST>
__device__ __forceinline__ float4 load_row(const float* p) {
  if constexpr (!PAST) return *reinterpret_cast<const float4*>(p);
  const f32x4 v = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p));
  return float4{v[0], v[1], v[2], v[3]};
}
template <bool PAST>
__device__ __forceinline__ uint2 load_row(const uint16_t* p) {
  if constexpr (!PAST) return *reinterpret_cast<const uint2*>(p);
  const u32x2 v = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p));
  return uint2{v[0], v[1]};
}

__device__ __forceinline__ float4 widen_row(const float4& v) { return v; }
__device__ __forceinline__ float4 widen_row(const uint2& v) { return float4{bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y)}; }

// four columns of a row of k (a multiple of 64) in two bf16 terms: of 32 columns the heads, then the tails
__device__ __forceinline__ void store_two_terms(uint16_t* Ht, int64_t row, int k, int col, const float4& v) {
  uint16_t* const p = Ht + row * (2 * k) + col / 32 * 64 + col % 32;
  const float x[4] = {v.x, v.y, v.z, v.w};
  uint32_t h[4], l[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const __bf16 hb = (__bf16)x[e];
    h[e] = __builtin_bit_cast(uint16_t, hb);
    const __bf16 lb = (__bf16)(x[e] - __uint_as_float(h[e] << 16));
    l[e] = __builtin_bit_cast(uint16_t, lb);
  }
  *reinterpret_cast<u32x2*>(p) = u32x2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
  *reinterpret_cast<u32x2*>(p + 32) = u32x2{l[0] | (l[1] << 16), l[2] | (l[3] << 16)};
}

// Loads from memory straight to LDS are inline assembly: they write no register, and the compiler, which would wait for all of them
// before every read of LDS, does not see them.  Every wait for them is written out; the compiler's own counts can only wait
// for more.
typedef __attribute__((address_space(3))) char lds_char;
// a buffer resource over `bytes` bytes: what lies behind them reads as zero
__device__ __forceinline__ u32x4 buffer_of(const void* p, uint64_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a), (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu),
               (uint32_t)__builtin_amdgcn_readfirstlane(bytes > 0xffffffffull ? 0xffffffffu : (uint32_t)bytes), 0x00020000u};
}
// 16 bytes per lane from buffer + voff + soff to LDS at lds + 16 * lane
__device__ __forceinline__ void load_to_lds(uint32_t lds, const u32x4& buffer, uint32_t voff, uint32_t soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(buffer), "s"(soff)
               : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads() {  // all but the N requested last
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

}  // namespace
}  // namespace gsi
