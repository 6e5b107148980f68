// Decode batches (2..128 tokens per call) with fp32 storage: Algorithm 1 lines 1-7 on the fp32 matrix instructions.
//
// The operands are fp32 and stay fp32 (v_mfma_f32_16x16x4_f32: products and sums in 32 bits, as the FMA kernels that these
// replace).  A float4 of a matrix row and a float4 of a token's vector are the operands of four MFMAs: lane l holds row (or
// token) l % 16 and columns 4 (l / 16) .. + 3 of a 16-column step, MFMA e takes element e of both, so any 16 columns are
// covered once and both operands are read straight from memory in 16-byte pieces.
//
//   f32_rows        16 output rows per workgroup, the whole contraction: eight waves take its 16-column pieces in turn, their
//                   sums meet in LDS, in pairs.  The image term of every token, then the W term of the fired tokens (or
//                   W x), are added in LDS and written once: no partial sums, no second pass over Y.
//   f32_proj        c = U^T x over a slab of rows of U and 64 of its columns: float4s of U's rows are the operands of four
//                   column tiles (columns 4 j + e), so U is read along its rows.  Slab partials, added by tile_proj_reduce.
//   f32_residual    r = x - U c for 64 rows x 16 tokens per workgroup, the norms' shares, and, by the workgroup of an input
//                   that finishes last, norms, gate and the list of fired tokens (as tile_residual).
// What bounds them is latency: a layer of these sizes is a few MB.  The kernels before these went token by token through the
// same rows (a group of four tokens a time in the projection, one fired token a time in the W term).  Project, gate and map of
// 768 x 3072, rank 64: 64 tokens, 16 fired: 223 us of
// launches, 32 us here; 2048 x 8192, rank 128, 64 tokens: 391 us, 56 us.
#include <algorithm>

#include "gsi_decode.h"
#include "gsi_device.h"
#include "gsi_tile_common.h"

namespace gsi {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kFBlock = 512;                // f32_rows, f32_proj: eight waves
constexpr int kFWaves = kFBlock / kWave;
constexpr int kFRows = 16;                  // output rows per workgroup of f32_rows
constexpr int kGroupTiles = 4;              // f32_proj: token tiles (of 16) that share a pass
constexpr int kGroupTok = 16 * kGroupTiles;
constexpr int kRowTiles = 2;                // f32_rows: ditto
constexpr int kRowTok = 16 * kRowTiles;
constexpr int kPiece = 16;                  // columns a wave takes at a time: a step of four MFMAs
constexpr int kPCols = 64;                  // columns of U per workgroup of f32_proj
constexpr int kSlabRows = 16 * kFWaves;     // rows of U per workgroup of f32_proj, lower bound
constexpr int kRBlock = 256;                // f32_residual: four waves of 16 rows
constexpr int kRRows = 64;

// the four MFMAs of a step, each with a sum of its own: a chain of sums is then no longer than in a kernel that adds a
// row's products over its lanes (with one sum for all, y was 1.5e-7 off instead of 0.9e-7 at rank 64)
__device__ __forceinline__ void mma4(const float4& a, const float4& b, f32x4 (&acc)[4]) {
  acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc[0], 0, 0, 0);
  acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc[1], 0, 0, 0);
  acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, acc[2], 0, 0, 0);
  acc[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, acc[3], 0, 0, 0);
}
__device__ __forceinline__ f32x4 sum4(const f32x4 (&acc)[4]) { return (acc[0] + acc[1]) + (acc[2] + acc[3]); }
__device__ __forceinline__ float4 zero4() { return float4{0.f, 0.f, 0.f, 0.f}; }

// acc[t] += rows of A times the tokens of tile t over the pieces of this wave (pieces wave, wave + 8, ... of K columns, K a
// multiple of four; columns past the end are zero).  arow: this lane's row of A; tok: this lane's token of each tile.
// nt: tiles in use (uniform).
__device__ __forceinline__ void rows_pieces(const float* __restrict__ arow, const void* __restrict__ V, int vdt, int64_t ldv,
                                            const int (&tok)[kRowTiles], int nt, int K, int wave, int lq,
                                            f32x4 (&acc)[kRowTiles][4]) {
  const int pieces = (K + kPiece - 1) / kPiece;
  for (int p0 = wave; p0 < pieces; p0 += 4 * kFWaves) {  // four pieces requested together
    float4 a[4], b[kRowTiles][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = (p0 + q * kFWaves) * kPiece + 4 * lq;
      const bool live = c < K;
      const int cc = live ? c : 0;
      a[q] = *reinterpret_cast<const float4*>(arow + cc);
      if (!live) a[q] = zero4();
#pragma unroll
      for (int t = 0; t < kRowTiles; ++t)
        if (t < nt) {
          b[t][q] = load_act4<false>(V, vdt, tok[t] * ldv + cc);
          if (!live) b[t][q] = zero4();
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int t = 0; t < kRowTiles; ++t)
        if (t < nt) mma4(a[q], b[t][q], acc[t]);
  }
}

__global__ __launch_bounds__(kFBlock) void f32_rows(const LinBatch lb) {
  __shared__ float4 red[kFWaves][kRowTiles][kWave];
  __shared__ __align__(16) float y[kMaxTok][kFRows];
  int ti = 0;
#pragma unroll
  for (int i = 1; i < kMaxLinTasks; ++i)
    if (i < lb.n && (int)blockIdx.x >= lb.blk_begin[i]) ti = i;
  const LinTask& p = lb.t[ti];
  const LinGroup& g = lb.g[p.group];
  const int B = lb.B, m = p.m, row0 = ((int)blockIdx.x - lb.blk_begin[ti]) * kFRows;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int li = lane & 15, lq = lane >> 4;
  const int row = min(row0 + li, m - 1);  // rows past the matrix repeat the last one

  // one product: tokens 0 .. count - 1 (token j is row idx ? idx[j] : j of V) of A's rows, stored to or added to y
  auto product = [&](const void* A, int K, const void* V, int vdt, const int32_t* idx, int count, bool add) {
    for (int g0 = 0; g0 < count; g0 += kRowTok) {
      const int nt = min(kRowTiles, (count - g0 + 15) / 16);
      int tok[kRowTiles];
      f32x4 acc[kRowTiles][4];
#pragma unroll
      for (int t = 0; t < kRowTiles; ++t) {
        const int j = min(g0 + 16 * t + li, count - 1);
        tok[t] = idx ? min(max(idx[j], 0), B - 1) : j;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      rows_pieces(reinterpret_cast<const float*>(A) + (int64_t)row * K, V, vdt, K, tok, nt, K, wave, lq, acc);
#pragma unroll
      for (int t = 0; t < kRowTiles; ++t)
        if (t < nt) {
          const f32x4 q = sum4(acc[t]);
          red[wave][t][lane] = float4{q[0], q[1], q[2], q[3]};
        }
      __syncthreads();
      // tile t, lane l: token 16 t + l % 16, rows 4 (l / 16) .. + 3
      if (wave < nt) {
        float4 s[kFWaves];
#pragma unroll
        for (int w = 0; w < kFWaves; ++w) s[w] = red[w][wave][lane];
#pragma unroll
        for (int h = kFWaves / 2; h > 0; h /= 2)  // pairs, then pairs of pairs
#pragma unroll
          for (int w = 0; w < h; ++w) {
            s[w].x += s[w + h].x; s[w].y += s[w + h].y; s[w].z += s[w + h].z; s[w].w += s[w + h].w;
          }
        const int j = g0 + 16 * wave + li;
        if (j < count) {
          const int t = idx ? min(max(idx[j], 0), B - 1) : j;
          float4* yp = reinterpret_cast<float4*>(&y[t][4 * lq]);
          if (add) {
            const float4 o = *yp;
            s[0] = float4{o.x + s[0].x, o.y + s[0].y, o.z + s[0].z, o.w + s[0].w};
          }
          *yp = s[0];
        }
      }
      __syncthreads();
    }
  };
  if (lb.dense) {
    product(p.W, g.d, g.X, g.xdtype, nullptr, B, false);
  } else {
    int nf = g.n_fired[0];
    nf = nf < 0 ? 0 : (nf > B ? B : nf);
    product(p.M, g.k, g.C, GSI_F32, nullptr, B, false);
    if (nf > 0) product(p.W, g.d, g.wx ? g.X : g.R, g.wx ? g.xdtype : GSI_F32, g.fired_idx, nf, !g.wx);
  }
  for (int e = threadIdx.x; e < B * kFRows; e += kFBlock) {  // sixteen consecutive rows of a token per sixteen threads
    const int t = e / kFRows, r = e % kFRows;
    if (row0 + r < m) p.Y[(int64_t)t * m + row0 + r] = y[t][r];
  }
}

// part_c[slab][t][j] = sum over the slab's rows i of U[i][j] x_t[i]
__global__ __launch_bounds__(kFBlock) void f32_proj(const ProjBatch pb) {
  __shared__ float4 red[kFWaves][4][kWave];
  int ti = 0;
#pragma unroll
  for (int i = 1; i < kMaxTasks; ++i)
    if (i < pb.n && (int)blockIdx.x >= pb.a_begin[i]) ti = i;
  const ProjTask& p = pb.t[ti];
  const int local = blockIdx.x - pb.a_begin[ti];
  const int slab = local % p.a_slabs, cg = local / p.a_slabs;
  const int d = p.d, k = p.k, B = pb.B;
  if (local == 0 && threadIdx.x == 0) *p.sync = 0u;  // the residual launch counts its finished workgroups here
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int li = lane & 15, lq = lane >> 4;
  const int r_begin = slab * p.a_rows, r_end = min(d, r_begin + p.a_rows);
  const int col = min(cg * kPCols + 4 * li, k - 4);  // columns past the rank repeat the last four (not stored)
  const float* U = reinterpret_cast<const float*>(p.U) + col;
  for (int g0 = 0; g0 < B; g0 += kGroupTok) {
    const int nt = min(kGroupTiles, (B - g0 + 15) / 16);
    f32x4 acc[kGroupTiles][4];
#pragma unroll
    for (int t = 0; t < kGroupTiles; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int i0 = r_begin + 16 * wave; i0 < r_end; i0 += 16 * kFWaves) {
      const int i = i0 + 4 * lq;  // this lane's four rows of U, elements of the tokens' vectors (d is a multiple of four)
      const bool live = i < r_end;
      const int ic = live ? i : r_begin;
      float4 u[4], x[kGroupTiles];
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        u[f] = *reinterpret_cast<const float4*>(U + (int64_t)(ic + f) * k);
        if (!live) u[f] = zero4();
      }
#pragma unroll
      for (int t = 0; t < kGroupTiles; ++t)
        if (t < nt) {
          x[t] = load_act4<false>(p.X, p.xdtype, (int64_t)min(g0 + 16 * t + li, B - 1) * d + ic);
          if (!live) x[t] = zero4();
        }
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        const float uf[4] = {u[f].x, u[f].y, u[f].z, u[f].w};
#pragma unroll
        for (int t = 0; t < kGroupTiles; ++t)
          if (t < nt) {
            const float xf = f == 0 ? x[t].x : f == 1 ? x[t].y : f == 2 ? x[t].z : x[t].w;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[t][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(uf[e], xf, acc[t][e], 0, 0, 0);
          }
      }
    }
    // element v of column tile e: token l % 16, column 4 (4 (l / 16) + v) + e: sixteen consecutive columns per lane
#pragma unroll
    for (int t = 0; t < kGroupTiles; ++t) {
      if (t >= nt) break;  // uniform
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][v][lane] = float4{acc[t][0][v], acc[t][1][v], acc[t][2][v], acc[t][3][v]};
      __syncthreads();
      if (wave < 4) {
        float4 s = red[0][wave][lane];
#pragma unroll
        for (int w = 1; w < kFWaves; ++w) {
          const float4 q = red[w][wave][lane];
          s.x += q.x; s.y += q.y; s.z += q.z; s.w += q.w;
        }
        const int tok = g0 + 16 * t + li, j = cg * kPCols + 16 * lq + 4 * wave;
        if (tok < B && j < k) *reinterpret_cast<float4*>(p.part_c + ((int64_t)slab * B + tok) * k + j) = s;
      }
      __syncthreads();
    }
  }
}

__global__ __launch_bounds__(kRBlock) void f32_residual(const ProjBatch pb) {
  __shared__ float shares[kRBlock / kWave][16][2];
  __shared__ float2 red[kRBlock];
  __shared__ int wave_count[kMaxTok / kWave];
  __shared__ int s_last;
  int ti = 0;
#pragma unroll
  for (int i = 1; i < kMaxTasks; ++i)
    if (i < pb.n && (int)blockIdx.x >= pb.b_begin[i]) ti = i;
  const ProjTask& p = pb.t[ti];
  const int B = pb.B, tiles = (B + 15) / 16, item = blockIdx.x - pb.b_begin[ti];
  const int rb = item % p.b_slabs, g0 = (item / p.b_slabs) * 16;
  const int d = p.d, k = p.k;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int li = lane & 15, lq = lane >> 4;
  const int row0 = rb * kRRows + 16 * wave;
  const int tok = min(g0 + li, B - 1);
  const float* arow = reinterpret_cast<const float*>(p.U) + (int64_t)min(row0 + li, d - 1) * k;
  const float* c = p.C + (int64_t)tok * k;
  const int row = row0 + 4 * lq;          // the lane's four outputs (d is a multiple of four)
  const bool live = row < d;
  const float4 x = load_act4<false>(p.X, p.xdtype, (int64_t)tok * d + (live ? row : 0));
  f32x4 acc[4][4];  // (a sum per step of 64 columns as well: what is left of x is a few percent of the terms)
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[q][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < k; c0 += 64) {  // four steps requested together; columns past the rank are zero
    float4 a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int cc = c0 + 16 * q + 4 * lq;
      const bool in = cc < k;
      a[q] = *reinterpret_cast<const float4*>(arow + (in ? cc : 0));
      b[q] = *reinterpret_cast<const float4*>(c + (in ? cc : 0));
      if (!in) a[q] = b[q] = zero4();
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) mma4(a[q], b[q], acc[q]);
  }
  const f32x4 s = (sum4(acc[0]) + sum4(acc[1])) + (sum4(acc[2]) + sum4(acc[3]));
  const float4 r = float4{x.x - s[0], x.y - s[1], x.z - s[2], x.w - s[3]};
  float sr = 0.f, sx = 0.f;
  if (live && g0 + li < B) {
    *reinterpret_cast<float4*>(p.R + (int64_t)tok * d + row) = r;
    sr = fmaf(r.x, r.x, fmaf(r.y, r.y, fmaf(r.z, r.z, r.w * r.w)));
    sx = fmaf(x.x, x.x, fmaf(x.y, x.y, fmaf(x.z, x.z, x.w * x.w)));
  }
  sr += __shfl_xor(sr, 16); sr += __shfl_xor(sr, 32);
  sx += __shfl_xor(sx, 16); sx += __shfl_xor(sx, 32);
  if (lq == 0) {
    shares[wave][li][0] = sr;
    shares[wave][li][1] = sx;
  }
  __syncthreads();
  if (threadIdx.x < 32) {
    const int tl = threadIdx.x >> 1, q = threadIdx.x & 1;
    if (g0 + tl < B) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < kRBlock / kWave; ++w) sum += shares[w][tl][q];
      __hip_atomic_store(&p.part_n[((int64_t)rb * B + g0 + tl) * 2 + q], sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (!pb.norms) return;  // uniform
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the shares have reached memory ...
  __syncthreads();                                  // ... before the workgroup counts as done
  if (threadIdx.x == 0)
    s_last = __hip_atomic_fetch_add(p.sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == (unsigned)(p.b_slabs * tiles);
  __syncthreads();
  if (!s_last) return;  // uniform
  norms_and_gate<kRBlock>(p, B, pb.gate, pb.eps, red, wave_count);
}

}  // namespace

// ---- projection ---------------------------------------------------------------------------------
// (what the vector kernels take: k and d multiples of four)
static int slab_rows(int64_t d) { return (int)(ceil_div(std::max<int64_t>(ceil_div(d, kPartSlabs), kSlabRows), kSlabRows) * kSlabRows); }

bool f32_project_shape_ok(int64_t d, int64_t k, int64_t B, int udtype) {
  return udtype == GSI_F32 && B >= 2 && B <= kMaxTok && d % 4 == 0 && k % 4 == 0 && k <= kMaxK && d < (1 << 24);
}

size_t f32_project_ws(int64_t d, int64_t k, int64_t B) {
  return align_up((size_t)ceil_div(d, slab_rows(d)) * B * k * 4, 256) + align_up((size_t)ceil_div(d, kRRows) * B * 2 * 4, 256) + 256;
}

void f32_project_fill(ProjTask& t, int64_t d, int64_t k, int64_t B, void* ws) {
  t.d = (int)d;
  t.k = (int)k;
  t.a_rows = slab_rows(d);
  t.a_slabs = (int)ceil_div(d, t.a_rows);
  t.a_cblocks = (int)ceil_div(k, kPCols);
  t.b_rows = kRRows;
  t.b_slabs = (int)ceil_div(d, kRRows);
  t.part_c = reinterpret_cast<float*>(ws);
  t.part_n = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + align_up((size_t)t.a_slabs * B * k * 4, 256));
  t.sync = reinterpret_cast<unsigned*>(reinterpret_cast<char*>(t.part_n) + align_up((size_t)t.b_slabs * B * 2 * 4, 256));
}

hipError_t f32_project_launch(ProjBatch& pb, bool with_norms, bool with_gate, float eps, hipStream_t s) {
  if (pb.n == 0 || pb.B == 0) return hipSuccess;
  int ta = 0, tb = 0;
  for (int i = 0; i < pb.n; ++i) {
    pb.a_begin[i] = ta;
    pb.b_begin[i] = tb;
    ta += pb.t[i].a_slabs * pb.t[i].a_cblocks;
    tb += pb.t[i].b_slabs * (int)ceil_div(pb.B, 16);
  }
  pb.b_total = tb;
  pb.norms = with_norms ? 1 : 0;
  pb.gate = with_gate ? 1 : 0;
  pb.eps = eps;
  f32_proj<<<ta, kFBlock, 0, s>>>(pb);
  if (hipError_t e = tile_proj_reduce_launch(pb, s); e != hipSuccess) return e;
  f32_residual<<<tb, kRBlock, 0, s>>>(pb);
  return hipGetLastError();
}

// ---- linear maps --------------------------------------------------------------------------------
hipError_t f32_rows_launch(LinBatch& lb, hipStream_t s) {
  int total = 0;
  for (int i = 0; i < lb.n; ++i) {
    lb.blk_begin[i] = total;
    total += (int)ceil_div(lb.t[i].m, kFRows);
  }
  f32_rows<<<total, kFBlock, 0, s>>>(lb);
  return hipGetLastError();
}

}  // namespace gsi
