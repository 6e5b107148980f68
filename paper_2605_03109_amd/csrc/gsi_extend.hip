// Online basis maintenance of libgsi: one DGKS rank-1 extension of a basis of fixed capacity, with the matching
// append to the cached images (Section 5.3 "The cascade initialization", Section 5.4 "Time-dimension tracking",
// Section 7 "Online basis adaptation").
//
// The basis lives in U[d, K] whose columns from k on are zero (a zero column changes neither c, r nor y, so every
// other kernel of the library runs on it unchanged at rank K).  Given the residual r = x - U U^T x of a token and
// its norms (what the projection of the layer already produced), the step is
//     candidate   iff  |x| > 0, |r| / |x| >= tau, k < K
//     s = U^T r,  r2 = r - U s                    (the re-orthogonalisation pass of classical Gram-Schmidt)
//     u = r2 / |r2| rounded to the basis' storage type  ->  column k of U
//     M[:, k] = W u   for every map that reads this basis, from the STORED u, so that M = W U keeps holding
//     E[:, k] = E[k, :] = U^T u - e_k             (when the caller keeps E = U^T U - I for the single-pass gate)
//     k <- k + 1
// Everything is decided on the device (k is a device counter): every kernel below starts by reading (or, the
// first one, forming) the verdict and leaves at once when there is nothing to do, so a token that does not extend
// the basis costs a handful of empty launches and no pass over U or W.  All sums have a fixed order.
//
// Launches: s partials (+ the candidate verdict) | s, r2 and shares of |r2|^2 | final verdict, the stored column, the image
// columns of all maps and the partials of U^T u | E's row and column.  The three jobs of the third launch need the stored
// column u = r2 / |r2| rounded, and each workgroup forms the part it reads from r2 and the shares itself (the same
// arithmetic everywhere), so none waits for another; the workgroup that reads the new column of U takes u for it.  An
// extension moves U three times and every W once; operands whose rows are 16-byte aligned are read with 16-byte loads,
// several in flight per lane.  Large bases have s added up by a launch of its own (own_sums).  (s, the column and U^T u in
// launches of their own for every basis: seven launches of 4 to 5 us around one of 24 us; three maps 4096 x 4096 on a
// basis of 4096 x 384, 256 columns in use: 46.7 us, 34.9 us with these four, calls replayed from a graph.)
//
// Every launch covers ALL bases of a call (one grid dimension is the basis, or the map): a token's pass over the
// bases of a whole model is these launches, not as many per basis, and what it costs when no basis grows is
// four or five nearly empty ones.  The records of a call with several bases sit in a table in the workspace (copied
// there by the call); a call with one basis carries its record in the kernel arguments.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "gsi_decode.h"
#include "gsi_device.h"
#include "gsi_extend.h"

namespace gsi {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / kWave;
constexpr int kCols = 64;       // columns of U per workgroup in the projections
constexpr int kRowsPerWg = 32;  // rows of U per workgroup in the residual
constexpr int kImgPerWave = 2;    // rows of W per wave and turn in the image rows
constexpr int kImgRows = kWaves * kImgPerWave;
constexpr int kLdsK = 2048;       // ranks whose s the residual workgroups can add up themselves (in LDS)
constexpr int kUBytes = 16384;    // block of the stored column that the image workgroups hold in LDS
constexpr int kFewMaps = 8;     // maps whose records fit the kernel arguments
constexpr int kSumBlock = 64;   // a wave per workgroup in the slab sums

struct ExtArg {  // the bases of a launch: a device table, or (tab == null) the one record
  const ExtIn* tab;
  ExtIn one;
};
// Where the record is, is known at compile time: chosen at run time, every field of it would be a flat load of its own, and
// so every load through its pointers.
template <bool TAB>
__device__ __forceinline__ ExtIn ext_record(const ExtArg& a, int i) {
  if constexpr (TAB) return a.tab[i];
  else return a.one;
}
struct ExtMapArg {  // the maps of an image launch: a device table, or up to kFewMaps records
  const ExtMapRec* tab;
  ExtMapRec few[kFewMaps];
};

// Loads through pointers that a record holds.  The record comes from the table or from the kernel arguments, so that these
// pointers are generic to the compiler, and a plain load would be a flat one: it counts as an LDS access as well, and
// every wait is a wait for all of them.
__device__ __forceinline__ uint4 load_global16(const void* p) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = *(const __attribute__((address_space(1))) u32x4*)p;
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint4 load_global16_once(const void* p) {  // (non-temporal)
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float load_global(const float* p) { return *(const __attribute__((address_space(1))) float*)p; }
__device__ __forceinline__ float2 load_global2(const float* p) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  const f32x2 v = *(const __attribute__((address_space(1))) f32x2*)p;
  return float2{v.x, v.y};
}
__device__ __forceinline__ float4 load_global4(const float* p) {
  const uint4 v = load_global16(p);
  return float4{__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)};
}

struct ExtWs {
  ExtState* st;
  float *part, *sv, *r2, *pn;
};
__host__ __device__ __forceinline__ size_t a256(size_t b) { return (b + 255) / 256 * 256; }
__host__ __device__ __forceinline__ ExtWs ext_ws(const ExtIn& in) {
  ExtWs w;
  char* p = in.ws;
  w.st = reinterpret_cast<ExtState*>(p);
  p += a256(sizeof(ExtState));
  w.part = reinterpret_cast<float*>(p);
  p += a256((size_t)in.slabs * in.K * 4);
  w.sv = reinterpret_cast<float*>(p);
  p += a256((size_t)in.K * 4);
  w.r2 = reinterpret_cast<float*>(p);
  p += a256((size_t)in.d * 4);
  w.pn = reinterpret_cast<float*>(p);
  return w;
}

// the candidate's norm: every workgroup of a basis adds the shares of |r2|^2 in the same fixed order; 1 / |r2|, or 0 when
// the basis does not grow.  first: the thread's first share (ext_first_share), requested earlier.
__device__ __forceinline__ float ext_first_share(const ExtIn& in, const ExtWs& w) {
  return load_global(w.pn + min((int)threadIdx.x, in.wgs - 1));
}
__device__ __forceinline__ float ext_inverse(const ExtIn& in, const ExtWs& w, float* sh, float first) {
  const int cand = w.st->cand;  // (the shares are not used if it is zero)
  float t = (int)threadIdx.x < in.wgs ? first : 0.f;
  for (int q = threadIdx.x + kBlock; q < in.wgs; q += kBlock) t += load_global(w.pn + q);
  t = group_sum<kWave>(t);
  if (threadIdx.x % kWave == 0) sh[threadIdx.x / kWave] = t;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) tot += sh[q];
  const float n2 = sqrtf(tot);
  return cand && n2 > 0.f ? 1.f / n2 : 0.f;
}
// element of the stored column, widened
template <class T>
__device__ __forceinline__ float stored(float v) {
  typename T::storage t;
  T::store(&t, 0, v);
  return T::load(&t, 0);
}

// part[slab][j] = sum over the rows of slabs slab0, slab0 + step, ... of U[i, j] v[i] for the 64 columns of block cb.
// v: the residual r (inv == 0), or the stored column u = r2 inv, which stands in for column kc of U as well (another
// workgroup of the launch is writing it).
template <class T>
__device__ __forceinline__ void proj_block(const ExtIn& in, const ExtWs& w, const float* __restrict__ v, float inv, int kc, int cb,
                                           int slab0, int step) {
  using S = typename T::storage;
  const int64_t d = in.d, K = in.K;
  const S* U = static_cast<const S*>(in.U);
  float* part = w.part;
  constexpr int V = T::kVec;
  constexpr int TPR = kCols / V;        // threads per row segment of 64 columns
  constexpr int RG = kBlock / TPR;      // rows in flight per pass of the workgroup
  __shared__ float sh[RG][kCols + 1];
  const bool use_u = inv != 0.f;
  auto value = [&](int64_t i) { return use_u ? stored<T>(load_global(v + i) * inv) : load_global(v + i); };
  // (a call with many bases launches fewer workgroups per basis than it has slabs: the workgroup takes several)
  for (int slab = slab0; slab < in.slabs; slab += step) {
    const int64_t r0 = (int64_t)slab * in.rows_per_slab;
    const int64_t r1 = r0 + in.rows_per_slab < d ? r0 + in.rows_per_slab : d;
    if (in.uvec) {
      const int rg = threadIdx.x / TPR, cv = threadIdx.x % TPR;
      const int64_t col0 = (int64_t)cb * kCols + cv * V;
      const int own = use_u ? (int)(kc - col0) : -1;  // the element that is column kc
      float acc[V];
#pragma unroll
      for (int e = 0; e < V; ++e) acc[e] = 0.f;
      if (col0 < K) {  // K is a multiple of V here: whole vectors
        for (int64_t i = r0 + rg; i < r1; i += 4 * RG) {
          float f[4][V], wt[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {  // four rows requested before the first is used; rows past the slab repeat
            const int64_t ii = i + q * RG;  // the last one with weight zero
            const int64_t ic = ii < r1 ? ii : r1 - 1;
            T::widen(load_global16(U + ic * K + col0), f[q]);
            wt[q] = ii < r1 ? value(ic) : 0.f;
          }
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < V; ++e) acc[e] = fmaf(e == own ? wt[q] : f[q][e], wt[q], acc[e]);
        }
      }
#pragma unroll
      for (int e = 0; e < V; ++e) sh[rg][cv * V + e] = acc[e];
      __syncthreads();
      const int64_t col = (int64_t)cb * kCols + threadIdx.x;
      if (threadIdx.x < kCols && col < K) {
        float s = 0.f;
        for (int q = 0; q < RG; ++q) s += sh[q][threadIdx.x];
        part[(int64_t)slab * K + col] = s;
      }
    } else {
      constexpr int RL = kBlock / kCols;
      const int64_t col = (int64_t)cb * kCols + threadIdx.x % kCols;
      const int rl = threadIdx.x / kCols;
      float acc = 0.f;
      if (col < K)
        for (int64_t i = r0 + rl; i < r1; i += RL) {
          const float x = value(i);
          acc = fmaf(use_u && col == kc ? x : T::load(U, i * K + col), x, acc);
        }
      sh[rl][threadIdx.x % kCols] = acc;
      __syncthreads();
      if (rl == 0 && col < K) {
        float s = 0.f;
        for (int q = 0; q < RL; ++q) s += sh[q][threadIdx.x];
        part[(int64_t)slab * K + col] = s;
      }
    }
    __syncthreads();  // the sums have been read before the next slab's are written
  }
}

// Partials of s = U^T r (grid: column blocks x slabs x bases); every workgroup forms the candidate verdict from the
// token's norms and the column counter, the first one of a basis records it.
template <class T, bool TAB>
__global__ __launch_bounds__(kBlock) void ext_proj(const ExtArg a, float tau) {
  const ExtIn in = ext_record<TAB>(a, blockIdx.z);
  const ExtWs w = ext_ws(in);
  if ((int64_t)blockIdx.x * kCols >= in.K || (int)blockIdx.y >= in.slabs) return;  // (the grid is sized for the largest basis)
  const int k = in.k_cur[0];
  const bool cand = k >= 0 && k < in.K && gate_fires(in.rnorm[0], in.xnorm[0], tau);
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    w.st->kc = k;
    w.st->cand = cand ? 1 : 0;
    w.st->ext = 0;
    w.st->inv = 0.f;
  }
  if (!cand) return;
  proj_block<T>(in, w, in.R, 0.f, k, blockIdx.x, blockIdx.y, gridDim.y);
}

// sum over the slabs, in slab order, of part[slab][j]; sixteen requests in flight
__device__ __forceinline__ float slab_sum(const float* __restrict__ part, int slabs, int64_t K, int64_t j) {
  float t = 0.f;
  for (int q0 = 0; q0 < slabs; q0 += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = load_global(part + (int64_t)min(q0 + u, slabs - 1) * K + j);
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (q0 + u < slabs) t += v[u];
  }
  return t;
}

// ... of columns j and j + 1 (K even, the partials 8-byte aligned), N slabs requested at once (past the last, that one again: up to
// 16 slabs are asked for as 16: bases of up to 1024 rows, 768 x 64 without maps 13.5 us with 32, 12.8)
template <int N>
__device__ __forceinline__ float2 slab_sum2(const float* __restrict__ part, int slabs, int64_t K, int64_t j) {
  float2 t = float2{0.f, 0.f};
  for (int q0 = 0; q0 < slabs; q0 += N) {
    float2 v[N];
#pragma unroll
    for (int u = 0; u < N; ++u) v[u] = load_global2(part + (int64_t)min(q0 + u, slabs - 1) * K + j);
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (q0 + u < slabs) {
        t.x += v[u].x;
        t.y += v[u].y;
      }
  }
  return t;
}

// Is s added up by a launch of its own?  Else every residual workgroup adds all slab partials itself: a launch less, but the
// sums stand before its first product, and slabs x K x 4 bytes come from L2 for every workgroup.  us per extension of a
// basis with one map, together / in a launch of their own: 16384 x 256 62.0 / 63.8; 4096 x 512 27.8 / 27.5; 16384 x 512
// 65.6 / 65.0; 65536 x 512 197 / 191; 4096 x 2048 50.2 / 41.0; 16384 x 2048 109 / 100.  The line: 64 KB per
// workgroup, 64 MB in all.
__host__ __device__ __forceinline__ bool own_sums(const ExtIn& in) {
  const int64_t per = in.K * in.slabs;
  return in.K > kLdsK || per > 16384 || per * in.wgs > (1 << 24);
}

// s of the bases whose residual workgroups do not add it up themselves
template <bool TAB>
__global__ __launch_bounds__(kSumBlock) void ext_sum(const ExtArg a) {
  const ExtIn in = ext_record<TAB>(a, blockIdx.y);
  const ExtWs w = ext_ws(in);
  if (!own_sums(in) || !w.st->cand) return;
  const int64_t j = (int64_t)blockIdx.x * kSumBlock + threadIdx.x;
  if (j >= in.K) return;
  w.sv[j] = slab_sum(w.part, in.slabs, in.K, j);
}

// r2[i] = r[i] - sum_j U[i, j] s[j], a wave per row (two rows at a time); pn[workgroup] = the workgroup's share
// of |r2|^2
template <class T, bool TAB>
__global__ __launch_bounds__(kBlock) void ext_resid(const ExtArg a) {
  using S = typename T::storage;
  const ExtIn in = ext_record<TAB>(a, blockIdx.y);
  const ExtWs w = ext_ws(in);
  if ((int)blockIdx.x >= in.wgs || !w.st->cand) return;
  const int64_t d = in.d, K = in.K;
  const S* U = static_cast<const S*>(in.U);
  const float* v = in.R;
  float* r2 = w.r2;
  constexpr int V = T::kVec;
  __shared__ float shn[kWaves];
  __shared__ __align__(16) float ss[kLdsK];
  const float* s = w.sv;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  // rows r0 + wave, + 4, ... of a workgroup's 32: a wave's eight are requested together (rows past the end repeat the last)
  constexpr int NR = kRowsPerWg / kWaves;
  uint4 raw[NR];
  const int64_t chunks = K / V;
  auto request = [&](int64_t r0, int64_t c) {
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int64_t i = r0 + wave + q * kWaves;
      raw[q] = load_global16(U + (i < d ? i : d - 1) * K + (c < chunks ? c : chunks - 1) * V);
    }
  };
  if (in.uvec) request((int64_t)blockIdx.x * kRowsPerWg, lane);  // ahead of the sums below
  if (!own_sums(in)) {  // uniform
    if (K % 2 == 0) {
      auto sums = [&](auto sum) {
        for (int64_t j = 2 * threadIdx.x; j < K; j += 2 * kBlock)
          *reinterpret_cast<float2*>(ss + j) = sum(w.part, in.slabs, K, j);
      };
      if (in.slabs <= 16) sums(slab_sum2<16>);
      else sums(slab_sum2<32>);
    } else {
      for (int64_t j = threadIdx.x; j < K; j += kBlock) ss[j] = slab_sum(w.part, in.slabs, K, j);
    }
    __syncthreads();
    s = ss;
  }
  for (int blk = blockIdx.x; blk < in.wgs; blk += gridDim.x) {
  const int64_t r0 = (int64_t)blk * kRowsPerWg;
  const int64_t r1 = r0 + kRowsPerWg < d ? r0 + kRowsPerWg : d;
  float nn = 0.f;
  if (in.uvec) {
    float acc[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) acc[q] = 0.f;
    for (int64_t c = lane; c - lane < chunks; c += kWave) {  // (whole waves)
      if (c != lane || blk != (int)blockIdx.x) request(r0, c);
      const bool live = c < chunks;
      const float* sp = s + (live ? c : chunks - 1) * V;
      float sv[V];
#pragma unroll
      for (int q = 0; q < V / 4; ++q) {
        const float4 x = *reinterpret_cast<const float4*>(sp + 4 * q);
        sv[4 * q] = x.x; sv[4 * q + 1] = x.y; sv[4 * q + 2] = x.z; sv[4 * q + 3] = x.w;
      }
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        float f[V];
        T::widen(raw[q], f);
        float t = acc[q];
#pragma unroll
        for (int e = 0; e < V; ++e) t = fmaf(f[e], sv[e], t);
        acc[q] = live ? t : acc[q];
      }
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const float t = group_sum<kWave>(acc[q]);
      const int64_t i = r0 + wave + q * kWaves;
      if (i < r1) {  // uniform
        const float ra = load_global(v + i) - t;
        if (lane == 0) r2[i] = ra;
        nn = fmaf(ra, ra, nn);  // (every lane holds the same value)
      }
    }
  } else {
    for (int64_t i = r0 + wave; i < r1; i += kWaves) {
      float acc = 0.f;
      for (int64_t j = lane; j < K; j += kWave) acc = fmaf(T::load(U, i * K + j), s[j], acc);
      acc = group_sum<kWave>(acc);
      const float r = v[i] - acc;
      if (lane == 0) r2[i] = r;
      nn = fmaf(r, r, nn);
    }
  }
  if (lane == 0) shn[wave] = nn;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
    for (int q = 0; q < kWaves; ++q) t += shn[q];
    w.pn[blk] = t;
  }
  __syncthreads();
  }
}

// Column kc of U <- r2 / |r2| rounded to storage; the first workgroup of a basis records the verdict, the column counter
// and the caller's flag.
template <class T>
__device__ __forceinline__ void column_block(const ExtIn& in, const ExtWs& w, float inv, int blk, int blocks) {
  using S = typename T::storage;
  const int kc = w.st->kc;
  if (blk == 0 && threadIdx.x == 0) {
    const int ext = inv != 0.f ? 1 : 0;
    w.st->ext = ext;
    w.st->inv = inv;
    if (ext) in.k_cur[0] = kc + 1;
    if (in.extended) in.extended[0] = ext;
  }
  if (inv == 0.f) return;  // uniform
  S* U = static_cast<S*>(in.U);
  for (int64_t i = (int64_t)blk * kBlock + threadIdx.x; i < in.d; i += (int64_t)blocks * kBlock)
    T::store(U, i * in.K + kc, w.r2[i] * inv);
}

// M[row, kc] = sum_i W[row, i] u[i]: a workgroup takes kImgRows rows of a map a turn, a wave kImgPerWave of them.  The
// workgroup keeps a block of u (8192 columns in bf16) in LDS, rounded as it is stored, from turn to turn if it is all of u;
// a wave streams its rows past it in steps of 128 pieces of 16 bytes, the next three steps' loads under way all the time:
// from row to row, along the rows and across blocks.
// Bound by how much a unit has in flight: 119 registers leave four waves per SIMD.  Three maps 4096 x 4096 beside the rest of
// the launch 25.1 us, 21.8 with the first block of r2 requested beside the norm's shares, the image workgroups first (the
// launch has 16 more than the chip has places, and they waited for the last) and one basis' record read as an argument.
// With four rows per wave and the
// lanes' share of u in registers (163, three waves per SIMD) nothing was under way from one block of columns to the next,
// and long rows lost.  us per extension, rank 512, so / here / as a launch of its own behind the stored column: three maps
// 4096 x 4096 39.6 / 39.4 / 46.5, one of 16384 x 4096 48.2 / 42.7 / 53.2, one of 4096 x 16384 65.5 / 56.0 / 60.5, one of
// 4096 x 65536 197 / 160 / 168.  Other shapes of the ring (rows per wave x loads per step): 2 x 4 and 4 x 2 lose a wave per
// SIMD (1 to 9 us), 1 x 2 reads u from LDS twice as often (three maps 46.0).
// (Requesting the first rows ahead of the verdict costs more in registers than it hides.)
template <class T>
__device__ __forceinline__ void image_rows_block(const ExtIn& in, const ExtWs& w, const ExtMapRec& p, int blk, int blocks, float* sh) {
  using S = typename T::storage;
  constexpr int V = T::kVec;
  constexpr int NL = 2;                   // loads per lane and step
  constexpr int kStep = kWave * NL;       // 16-byte pieces of a step
  constexpr int kUPieces = kUBytes / 16;  // ... of a block of u
  static_assert(kUPieces % kStep == 0, "a block is whole steps");
  __shared__ uint4 us[kUPieces];
  const int64_t d = in.d, K = in.K;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int kc = w.st->kc;
  const S* W = static_cast<const S*>(p.W);
  const int64_t chunks = d / V;
  const int steps = (int)((chunks + kStep - 1) / kStep);
  int64_t held = -1;  // first piece of the block of u in LDS
  // The first block of r2 is requested with the shares of its norm, so that the rows wait for one round trip, not two.
  constexpr int kUPer = kUPieces / kBlock;
  float4 head[kUPer][V / 4];
  const float first = ext_first_share(in, w);
  if (p.vec) {
#pragma unroll
    for (int e = 0; e < kUPer; ++e) {
      if (e > 0 && e * kBlock >= chunks) break;  // uniform
#pragma unroll
      for (int q = 0; q < V / 4; ++q)
        head[e][q] = load_global4(w.r2 + min((int64_t)(threadIdx.x + e * kBlock), chunks - 1) * V + 4 * q);
    }
  }
  const float inv = ext_inverse(in, w, sh, first);
  if (inv == 0.f) return;  // uniform
  if (p.vec) {
#pragma unroll
    for (int e = 0; e < kUPer; ++e) {
      if (e > 0 && e * kBlock >= chunks) break;
      __align__(16) S t[V];
#pragma unroll
      for (int q = 0; q < V / 4; ++q) {
        const float4 x = head[e][q];
        T::store(t, 4 * q, x.x * inv); T::store(t, 4 * q + 1, x.y * inv);
        T::store(t, 4 * q + 2, x.z * inv); T::store(t, 4 * q + 3, x.w * inv);
      }
      us[threadIdx.x + e * kBlock] = *reinterpret_cast<const uint4*>(t);
    }
    held = 0;
    __syncthreads();
  }
#pragma unroll 1
  for (int64_t row_begin = (int64_t)blk * kImgRows; row_begin < p.m; row_begin += (int64_t)blocks * kImgRows) {
    const int64_t row0 = row_begin + wave * kImgPerWave;
    float acc[kImgPerWave];
#pragma unroll
    for (int r = 0; r < kImgPerWave; ++r) acc[r] = 0.f;
    if (p.vec) {
      constexpr int kSlots = 4, kAhead = kSlots - 1;  // steps under way: slot f of the ring is row f % kImgPerWave
      static_assert(kSlots % kImgPerWave == 0, "a slot belongs to a row");
      uint4 raw[kSlots][NL];
      // rows past the matrix and pieces past the row repeat the last one (uniform base, 32-bit lane offsets)
      auto request = [&](int slot, int g, int r) {
        const char* base = reinterpret_cast<const char*>(W + (row0 + r < p.m ? row0 + r : p.m - 1) * d + (int64_t)g * kStep * V);
        const int left = (int)(chunks - (int64_t)g * kStep < kStep ? chunks - (int64_t)g * kStep : kStep);
#pragma unroll
        for (int q = 0; q < NL; ++q) raw[slot][q] = load_global16_once(base + 16u * (uint32_t)min(lane + q * kWave, left - 1));
      };
#pragma unroll
      for (int f = 0; f < kAhead; ++f)
        if (f / kImgPerWave < steps) request(f, f / kImgPerWave, f % kImgPerWave);
#pragma unroll 1
      for (int g0 = 0; g0 < steps; g0 += kSlots / kImgPerWave) {
#pragma unroll
        for (int f = 0; f < kSlots; ++f) {
          const int g = g0 + f / kImgPerWave, r = f % kImgPerWave;
          if (g < steps) {
            const int64_t c0 = (int64_t)g * kStep;
            const int in_block = (int)(c0 % kUPieces), left = (int)(chunks - c0 < kStep ? chunks - c0 : kStep);
            if (r == 0 && in_block == 0 && c0 != held) {
              held = c0;  // uniform: the next block of u
              __syncthreads();  // (the one before has been read)
#pragma unroll 1
              for (int e = threadIdx.x; e < kUPieces && c0 + e < chunks; e += kBlock) {
                __align__(16) S t[V];
#pragma unroll
                for (int q = 0; q < V; q += 4) {
                  const float4 x = load_global4(w.r2 + (c0 + e) * V + q);
                  T::store(t, q, x.x * inv); T::store(t, q + 1, x.y * inv);
                  T::store(t, q + 2, x.z * inv); T::store(t, q + 3, x.w * inv);
                }
                us[e] = *reinterpret_cast<const uint4*>(t);
              }
              __syncthreads();
            }
            const int nf = f + kAhead, ng = g0 + nf / kImgPerWave;
            if (ng < steps) request(nf % kSlots, ng, nf % kImgPerWave);
            __builtin_amdgcn_sched_barrier(0);  // later rows' requests stay ahead of this row's arithmetic
#pragma unroll
            for (int q = 0; q < NL; ++q) {
              float f32[V], u[V];
              T::widen(raw[f][q], f32);
              T::widen(us[in_block + lane + q * kWave], u);
              float t = 0.f;
#pragma unroll
              for (int e = 0; e < V; ++e) t = fmaf(f32[e], u[e], t);
              acc[r] += lane + q * kWave < left ? t : 0.f;
            }
          }
        }
      }
    } else {
      for (int64_t i = lane; i < d; i += kWave) {
        const float x = stored<T>(w.r2[i] * inv);
#pragma unroll
        for (int r = 0; r < kImgPerWave; ++r)
          acc[r] = fmaf(T::load(W, (row0 + r < p.m ? row0 + r : p.m - 1) * d + i), x, acc[r]);
      }
    }
#pragma unroll
    for (int r = 0; r < kImgPerWave; ++r) {
      const float t = group_sum<kWave>(acc[r]);
      if (lane == 0 && row0 + r < p.m) T::store(static_cast<S*>(p.M), (row0 + r) * K + kc, t);
    }
  }
}

// What needs the stored column: workgroups of three kinds, told apart by their index: maps x img_wgs image rows, n bases x
// col_wgs columns, n bases x (pcols x pslabs) partials of U^T u.  The images go first, the launch lasts as long as they do; but
// behind the others (images_last) where a basis whose rows are no whole 16-byte pieces has partials, which then take longest:
// 4096 x 250 with three maps of 4096 rows 51.0 us behind the images, 49.7 ahead of them.
struct ExtStore {
  int col_wgs, pcols, pslabs, img_wgs, n, n_maps, images_last;
};
template <class T, bool TAB>
__global__ __launch_bounds__(kBlock) void ext_store(const ExtArg a, const ExtMapArg ma, const ExtStore g) {
  __shared__ float sh[kWaves];
  const int images = g.n_maps * g.img_wgs;
  int b = blockIdx.x;
  if (g.images_last) b = b < (int)gridDim.x - images ? b + images : b - ((int)gridDim.x - images);
  if (b < images) {
    const ExtMapRec p = TAB ? ma.tab[b / g.img_wgs] : ma.few[b / g.img_wgs];
    const int blk = b % g.img_wgs;
    if ((int64_t)blk * kImgRows >= p.m) return;
    const ExtIn in = ext_record<TAB>(a, p.in);
    const ExtWs w = ext_ws(in);
    if (!w.st->cand) return;
    image_rows_block<T>(in, w, p, blk, g.img_wgs, sh);
    return;
  }
  b -= images;
  if (b < g.n * g.col_wgs) {
    const int blk = b % g.col_wgs;
    const ExtIn in = ext_record<TAB>(a, b / g.col_wgs);
    if (blk > 0 && (int64_t)blk * kBlock >= in.d) return;
    const ExtWs w = ext_ws(in);
    column_block<T>(in, w, ext_inverse(in, w, sh, ext_first_share(in, w)), blk, g.col_wgs);
    return;
  }
  b -= g.n * g.col_wgs;
  const int per = g.pcols * g.pslabs;
  const ExtIn in = ext_record<TAB>(a, b / per);
  const int cb = b % per % g.pcols, slab = b % per / g.pcols;
  if (!in.gram || (int64_t)cb * kCols >= in.K || slab >= in.slabs) return;
  const ExtWs w = ext_ws(in);
  if (!w.st->cand) return;
  const float inv = ext_inverse(in, w, sh, ext_first_share(in, w));
  if (inv != 0.f) proj_block<T>(in, w, w.r2, inv, w.st->kc, cb, slab, g.pslabs);
}

// E[j, kc] = E[kc, j] = (U^T u)[j] - (j == kc), the projection over the extended basis added over its slabs
template <bool TAB>
__global__ __launch_bounds__(kSumBlock) void ext_gram(const ExtArg a) {
  const ExtIn in = ext_record<TAB>(a, blockIdx.y);
  const ExtWs w = ext_ws(in);
  if (!in.gram || !w.st->ext) return;
  const int64_t K = in.K;
  const int64_t j = (int64_t)blockIdx.x * kSumBlock + threadIdx.x;
  if (j >= K) return;
  const float t = slab_sum(w.part, in.slabs, K, j);
  const int kc = w.st->kc;
  const float v = t - (j == kc ? 1.f : 0.f);
  in.gram[j * K + kc] = v;
  in.gram[(int64_t)kc * K + j] = v;
}

struct Geom {
  int slabs, rows_per_slab, wgs;
};
Geom geom(int64_t d) {
  Geom g;
  g.slabs = (int)(d < 64 * 32 ? ceil_div(d, 64) : 32);
  g.rows_per_slab = (int)ceil_div(d, g.slabs);
  g.slabs = (int)ceil_div(d, g.rows_per_slab);
  g.wgs = (int)ceil_div(d, kRowsPerWg);
  return g;
}

template <class T, bool TAB>
hipError_t launch_all(const ExtIn* in, int n, const ExtMapRec* maps, int n_maps, float tau, void* table, hipStream_t s) {
  ExtArg a;
  std::memset(&a, 0, sizeof(a));
  const ExtMapRec* mtab = nullptr;
  if (!TAB) {
    a.one = in[0];
  } else {  // the records go to the table in the workspace: bases first, then maps
    const size_t ib = align_up((size_t)n * sizeof(ExtIn), 256), mb = align_up((size_t)n_maps * sizeof(ExtMapRec), 256);
    std::vector<char> host(ib + mb, 0);
    std::memcpy(host.data(), in, (size_t)n * sizeof(ExtIn));
    if (n_maps) std::memcpy(host.data() + ib, maps, (size_t)n_maps * sizeof(ExtMapRec));
    if (hipError_t e = upload_launch(host.data(), host.size(), table, s); e != hipSuccess) return e;
    a.tab = static_cast<const ExtIn*>(table);
    mtab = reinterpret_cast<const ExtMapRec*>(static_cast<const char*>(table) + ib);
  }
  int64_t K_max = 0, d_max = 0, m_max = 0;
  int slabs_max = 0, wgs_max = 0, any_gram = 0, any_own = 0;
  for (int i = 0; i < n; ++i) {
    K_max = std::max<int64_t>(K_max, in[i].K);
    d_max = std::max<int64_t>(d_max, in[i].d);
    slabs_max = std::max(slabs_max, in[i].slabs);
    wgs_max = std::max(wgs_max, in[i].wgs);
    any_gram |= in[i].gram != nullptr;
    any_own |= own_sums(in[i]);
  }
  for (int j = 0; j < n_maps; ++j) m_max = std::max<int64_t>(m_max, maps[j].m);
  // A launch is about kGridCap workgroups at most: every workgroup of a basis that does not grow reads its record and
  // leaves, which is what a token costs nearly always, so a call with many bases gives each fewer workgroups (they
  // take several slabs, row blocks ... in turn; what a workgroup computes per slab or row does not change).
  constexpr int64_t kGridCap = 2048;
  // image workgroups: of one basis three per compute unit, resident beside the launch's other workgroups; of many, of
  // which few grow as a rule, up to twice the cap, so that the maps of a basis that grows alone get some of the chip
  // (48 maps, 85 workgroups each: 63 us when one of 32 bases grows, 173 us with 16 each)
  const int64_t img_cap = n > 1 ? 2 * kGridCap : 768;
  const int64_t pc = ceil_div(K_max, kCols);
  const dim3 pgrid((unsigned)pc, (unsigned)std::min<int64_t>(slabs_max, std::max<int64_t>(1, kGridCap / (pc * n))), (unsigned)n);
  const dim3 kgrid((unsigned)ceil_div(K_max, kSumBlock), (unsigned)n);
  const int64_t per_basis = std::max<int64_t>(8, kGridCap / n);
  ext_proj<T, TAB><<<pgrid, kBlock, 0, s>>>(a, tau);
  if (any_own) ext_sum<TAB><<<kgrid, kSumBlock, 0, s>>>(a);
  ext_resid<T, TAB><<<dim3((unsigned)std::min<int64_t>(wgs_max, per_basis), (unsigned)n), kBlock, 0, s>>>(a);
  ExtStore g;
  g.n = n;
  g.images_last = 0;
  for (int i = 0; i < n; ++i) g.images_last |= in[i].gram && !in[i].uvec;
  g.col_wgs = (int)std::min<int64_t>(ceil_div(d_max, kBlock), std::max<int64_t>(1, per_basis / 8));
  g.pcols = any_gram ? (int)pgrid.x : 0;
  g.pslabs = any_gram ? (int)pgrid.y : 0;
  // the maps of one basis travel in the kernel arguments, kFewMaps at a time: the first launch does the other jobs as well
  for (int j0 = 0; j0 == 0 || (!mtab && j0 < n_maps); j0 += kFewMaps) {
    ExtMapArg ma;
    std::memset(&ma, 0, sizeof(ma));
    ma.tab = mtab;
    g.n_maps = mtab ? n_maps : std::min(kFewMaps, n_maps - j0);
    int64_t mm = m_max;
    if (!mtab) {
      mm = 0;
      for (int q = 0; q < g.n_maps; ++q) {
        ma.few[q] = maps[j0 + q];
        mm = std::max<int64_t>(mm, maps[j0 + q].m);
      }
    }
    g.img_wgs = g.n_maps > 0 ? (int)std::min<int64_t>(ceil_div(mm, kImgRows), std::max<int64_t>(8, img_cap / g.n_maps)) : 0;
    if (j0 > 0) g.n = 0;
    const int64_t blocks = (int64_t)g.n * (g.col_wgs + (int64_t)g.pcols * g.pslabs) + (int64_t)g.n_maps * g.img_wgs;
    if (blocks > 0) ext_store<T, TAB><<<(unsigned)blocks, kBlock, 0, s>>>(a, ma, g);
  }
  if (any_gram) ext_gram<TAB><<<kgrid, kSumBlock, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace

size_t extend_ws_bytes(int64_t d, int64_t K) {
  const Geom g = geom(d);
  return align_up(sizeof(ExtState), 256) + align_up((size_t)g.slabs * K * 4, 256) + align_up((size_t)K * 4, 256) +
         align_up((size_t)d * 4, 256) + align_up((size_t)g.wgs * 4, 256);
}

size_t extend_table_bytes(int n, int n_maps) {
  return n > 1 ? align_up((size_t)n * sizeof(ExtIn), 256) + align_up((size_t)n_maps * sizeof(ExtMapRec), 256) : 0;
}

void extend_fill(ExtIn& in, int udtype) {
  const Geom g = geom(in.d);
  in.slabs = g.slabs;
  in.rows_per_slab = g.rows_per_slab;
  in.wgs = g.wgs;
  // 16-byte loads along the rows of U: whole vectors per row, rows that start on 16 bytes
  const int V = udtype == GSI_BF16 ? 8 : 4;
  in.uvec = in.K % V == 0 && reinterpret_cast<uintptr_t>(in.U) % 16 == 0;
}

void extend_fill_map(ExtMapRec& mp, int64_t d, int udtype) {
  const int V = udtype == GSI_BF16 ? 8 : 4;
  mp.vec = d % V == 0 && reinterpret_cast<uintptr_t>(mp.W) % 16 == 0;
}

hipError_t extend_many(const ExtIn* in, int n, const ExtMapRec* maps, int n_maps, int udtype, float tau, void* table,
                       hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (n == 1)
    return udtype == GSI_BF16 ? launch_all<BF16, false>(in, n, maps, n_maps, tau, table, s)
                              : launch_all<F32, false>(in, n, maps, n_maps, tau, table, s);
  return udtype == GSI_BF16 ? launch_all<BF16, true>(in, n, maps, n_maps, tau, table, s)
                            : launch_all<F32, true>(in, n, maps, n_maps, tau, table, s);
}

}  // namespace gsi
