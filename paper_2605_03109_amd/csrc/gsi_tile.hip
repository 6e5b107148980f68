// Linear maps of a decode batch (2..128 tokens per call) on the matrix cores: Algorithm 1 lines 4-7 in
// the y = M c (+ W r when the gate fires) form of Eq. (exact), and the dense baseline y = W x.
//
// The work is a skinny GEMM bound by the one pass over the weights, so the kernel is organised around
// that pass.  A work item is 128 rows of one matrix by a slice of 512 contraction columns: each of the
// eight waves owns 16 rows and requests its whole share (16 loads of 16 bytes per lane) at once, straight
// from memory into A operands of v_mfma_f32_16x16x32_bf16 (lane l holds row l%16, columns 8*(l/16)..+8
// of a 32-column step).  The B operands are the same columns of up to 32 tokens' activation vectors,
// staged once per workgroup in LDS: fp32 activations are split into a bf16 head and a bf16
// tail (the rounded remainder) and take two MFMAs, so nothing is rounded to 8 bits.  More than 32 tokens
// take further rounds against the same A registers: the weights are read once whatever the token count.
// For the W term the tokens are the fired ones, taken from the device-side list in ascending order; with
// no fired token the kernel leaves before touching the weight matrix.
// Items of one matrix that cover different column slices write partial sums to the workspace, and a
// second kernel adds them in slice order, so results do not vary from run to run.
//
// Terms of an fp32 operand: two (relative remainder 2^-17) or three (2^-25, the fp32 value itself).  The projection and the
// residual take two for ranks of 64 * 2^j columns and fp32 activations, else three; image and weight rows take three only at
// ranks that are no multiple of 32 columns, or where the weight rows read bf16 activations.  What takes three ran on fp32
// FMAs before, and with two the residual, whose parts cancel to a few percent, was 2e-5 .. 5e-5 off instead of 3e-6 .. 2e-5.
// Three terms cost weight rows half of their places: 97.5 KB of LDS and 164 registers, one workgroup per unit, against 65 KB
// and 126, two per unit.
// Measured: a block of d = 2560, rank 128, 23 bf16 tokens 174 us on the FMA kernels, 64 us on these.
#include <algorithm>
#include <type_traits>

#include "gsi_decode.h"
#include "gsi_device.h"
#include "gsi_tile_common.h"

namespace gsi {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTBlock = 512;                       // threads per workgroup
constexpr int kTWaves = kTBlock / kWave;           // 8
constexpr int kItemRows = 16 * kTWaves;            // 128 rows per item
constexpr int kSteps = 16;                         // MFMA steps per item
constexpr int kStepCols = 32;                      // contraction columns per MFMA
constexpr int kSliceCols = kSteps * kStepCols;     // 512 columns per item
constexpr int kRoundTok = 32;                      // tokens staged per round (two MFMA token tiles)
constexpr int kMaxTokTiles = kMaxTok / 16;
constexpr int kVRow = kSliceCols + 8;              // bf16 per staged token row: 16 bytes of padding keep
                                                   // the 16 lanes of a 128-bit LDS read on distinct banks
constexpr int kHalfVec = 16 * kSliceCols / 4 / kTBlock;  // float4 per thread per 16 staged tokens (4)

template <int N>
__device__ __forceinline__ int find_task(const int (&begin)[N], int n, int b) {
  int t = 0;
#pragma unroll
  for (int i = 1; i < N; ++i)
    if (i < n && b >= begin[i]) t = i;
  return t;
}

// four fp32 values as T bf16 terms each: term 0 the rounded value, every further term the rounded remainder (exact
// differences).  Three terms: a value whose rounding overflows is cut instead, and an infinity or NaN has zero
// remainders, so that it travels through the products as itself, as it does through fp32 FMAs.
template <int T>
__device__ __forceinline__ void split4(const float4& v, uint2 (&out)[T]) {
  float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int t = 0; t < T; ++t) {
    uint32_t h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const __bf16 hb = (__bf16)x[e];
      h[e] = __builtin_bit_cast(uint16_t, hb);
      if (T == 3 && t == 0 && (h[e] & 0x7fffu) == 0x7f80u) h[e] = __float_as_uint(x[e]) >> 16;
      const float rem = x[e] - __uint_as_float(h[e] << 16);
      x[e] = T == 2 || fabsf(rem) <= 3.402823466e38f ? rem : 0.f;
    }
    out[t] = uint2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
  }
}

// Requests this thread's share of a staging round: tokens [g0, g0 + 32) of the phase (token j is row idx ? idx[j] : j of
// V, vdt its type), columns [c0, c0 + ncol), ncol a multiple of four; the second sixteen tokens only where two is set.  A
// wave pair covers one token row per pass.  Every load is unconditional: tokens past the count repeat the last one and
// columns past the slice its last four.  The second half goes out first: loads return in order, so a wait for the first
// half is the same number on both paths and never one for the weights that are requested next.  (Requested behind the
// weights, the second half waited for them too: 18.9 us instead of 17.8 for the residuals of 64 tokens.)
template <int T>
__device__ __forceinline__ void stage_issue(float4 (&v)[2][kHalfVec], bool two, const void* __restrict__ V, int vdt, int64_t ldv,
                                            const int32_t* __restrict__ idx, int g0, int count, int B, int c0, int ncol,
                                            int wave) {
  const int c4 = min((int)(threadIdx.x & 127), ncol / 4 - 1);
  const int j0 = g0 + (wave >> 1);
  int tok[2][kHalfVec];  // all token indices first (uniform across the wave), so that their loads overlap
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < kHalfVec; ++i) tok[h][i] = min(j0 + 16 * h + 4 * i, count - 1);
  if (idx) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h == 1 && !two) continue;
#pragma unroll
      for (int i = 0; i < kHalfVec; ++i) tok[h][i] = idx[tok[h][i]];
#pragma unroll
      for (int i = 0; i < kHalfVec; ++i) tok[h][i] = min(max(tok[h][i], 0), B - 1);
    }
  }
#pragma unroll
  for (int h = 1; h >= 0; --h) {
    if (h == 1 && !two) continue;  // uniform
#pragma unroll
    for (int i = 0; i < kHalfVec; ++i) v[h][i] = load_act4<T == 2>(V, vdt, (int64_t)tok[h][i] * ldv + c0 + 4 * c4);
  }
}

// what stage_issue requested, as T bf16 terms in LDS; columns past the slice are zero (three terms;
// with two, slices end with a step)
template <int T>
__device__ __forceinline__ void stage_commit(const float4 (&v)[2][kHalfVec], bool two, uint16_t* vt, int vrow, int ncol,
                                             int wave) {
  const int c4 = threadIdx.x & 127;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if ((h == 1 && !two) || 4 * c4 >= vrow - 8) continue;
#pragma unroll
    for (int i = 0; i < kHalfVec; ++i) {
      const int t = 16 * h + (wave >> 1) + 4 * i;
      uint2 term[T];
      split4<T>(T == 2 || 4 * c4 < ncol ? v[h][i] : float4{0.f, 0.f, 0.f, 0.f}, term);
#pragma unroll
      for (int q = 0; q < T; ++q) *reinterpret_cast<uint2*>(vt + (q * kRoundTok + t) * vrow + 4 * c4) = term[q];
    }
  }
}

// The weights of a wave's item: rows row (per lane), columns c0 + 32 s + 8 lq .. + 7 for step s.  base: first column of
// the slice; steps past the slice repeat its last one.  A slice that ends inside a step (a rank that is no multiple of
// 32, three terms only) has zeros past its end: those lanes read the step's first columns instead and are cleared.
template <int T, int N>
__device__ __forceinline__ void weights_issue(uint4 (&w)[N], const char* __restrict__ base, uint32_t row_off, int lq, int ncol,
                                              int ns) {
  const uint32_t voff = row_off + 16u * lq;
  if (ns == N && (T == 2 || (N < kSteps && ncol % kStepCols == 0))) {  // uniform: a whole slice, at constant offsets
#pragma unroll
    for (int s = 0; s < N; ++s) w[s] = *reinterpret_cast<const uint4*>(base + s * kStepCols * 2 + voff);
    return;
  }
  const uint32_t vlast = T == 2 || (ns - 1) * kStepCols + 8 * lq < ncol ? voff : row_off;
#pragma unroll
  for (int s = 0; s < N; ++s)
    w[s] = *reinterpret_cast<const uint4*>(base + (size_t)(min(s, ns - 1) * kStepCols * 2) + (s < ns - 1 ? voff : vlast));
}
template <int T, int N>
__device__ __forceinline__ void weights_clear_tail(uint4 (&w)[N], int lq, int ncol, int ns) {
  if (T == 2 || ncol % kStepCols == 0) return;  // uniform
  const bool dead = (ns - 1) * kStepCols + 8 * lq >= ncol;
#pragma unroll
  for (int s = 0; s < N; ++s)
    if (s == ns - 1 && dead) w[s] = uint4{0u, 0u, 0u, 0u};
}

// Sum of the head's products plus that of the remainders', which count only where the first is finite: an infinite weight
// times a remainder of either sign, or of zero, would make a NaN of the infinity that the fp32 product is.
__device__ __forceinline__ f32x4 add_tails(const f32x4& head, const f32x4& tails) {
  f32x4 s;
#pragma unroll
  for (int e = 0; e < 4; ++e) s[e] = head[e] + (fabsf(head[e]) <= 3.402823466e38f ? tails[e] : 0.f);
  return s;
}

// acc0 / acc1 = the item's weights times the staged tokens 0 .. 15 / 16 .. 31.  Three terms: the head's products of even
// and odd steps and those of the two remainders have accumulators of their own, so that fewer large partial sums are
// rounded (the residual's error against 64 bits is then the FMA kernel's, 2.7e-6 at rank 128; 3.6e-6 with one).
template <int T, int N>
__device__ __forceinline__ void item_mma(const uint4 (&w)[N], const uint16_t* vt, int vrow, int li, int lq,
                                         int ns, bool two, f32x4& acc0, f32x4& acc1) {
  constexpr int NA = T == 3 ? 3 : 1;
  f32x4 acc[2][NA];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int q = 0; q < NA; ++q) acc[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](int s, int t) {  // column step s of token tile t
    const bf16x8 a = __builtin_bit_cast(bf16x8, w[s]);
    const int col = s * kStepCols + 8 * lq;
#pragma unroll
    for (int q = 0; q < T; ++q) {
      f32x4& d = acc[t][NA == 1 ? 0 : (q > 0 ? 2 : s & 1)];
      d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          a, *reinterpret_cast<const bf16x8*>(vt + (q * kRoundTok + 16 * t + li) * vrow + col), d, 0, 0, 0);
    }
  };
  if ((T == 2 || N < kSteps) && ns == N) {
    // a whole slice: no branch per step, so the LDS reads run ahead of the products (the pair, 16 tokens: 72.5 -> 70.5 us
    // with the constant offsets of weights_issue, 32 tokens 77.2 -> 75.0)
    if (two) {
#pragma unroll
      for (int s = 0; s < N; ++s) {
        step(s, 0);
        step(s, 1);
      }
    } else {
#pragma unroll
      for (int s = 0; s < N; ++s) step(s, 0);
    }
  } else {
#pragma unroll
    for (int s = 0; s < N; ++s) {
      if (s < ns) {
        step(s, 0);
        if (two) step(s, 1);
      }
    }
  }
  acc0 = acc[0][0];
  acc1 = acc[1][0];
  if constexpr (NA == 3) {
    acc0 = add_tails(acc0 + acc[0][1], acc[0][2]);
    acc1 = add_tails(acc1 + acc[1][1], acc[1][2]);
  }
}

template <int T>
__global__ __launch_bounds__(kTBlock) void tile_rows(const LinBatch lb) {
  __shared__ __align__(16) uint16_t vt[T * kRoundTok * kVRow];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  const int li = lane & 15, lq = lane >> 4;
  const int B = lb.B;

  // item -> (map, kind, row block, column slice).  The image items come first: they are few and always have work,
  // and behind the weight items of a step in which nothing fired (which only read a count and leave) they would
  // wait for two rounds of empty workgroups to drain.
  const bool second = (int)blockIdx.x < lb.tile_split;
  const int ti = second ? find_task(lb.blk_begin2, lb.n, blockIdx.x) : find_task(lb.blk_begin, lb.n, blockIdx.x);
  const LinTask& p = lb.t[ti];
  const LinGroup& g = lb.g[p.group];
  const int m = p.m;
  const int item = blockIdx.x - (second ? lb.blk_begin2[ti] : lb.blk_begin[ti]);

  const uint16_t* A;
  const void* V;
  const int32_t* idx = nullptr;
  int K, count, slices, g_begin = 0, vdt = GSI_F32;
  bool to_part;
  if (second) {
    // image term over all tokens, whole rank in one slice, written straight to Y; one item per round of
    // 32 tokens, so that a large batch spreads over more workgroups instead of taking rounds in turn
    A = reinterpret_cast<const uint16_t*>(p.M); V = g.C; K = g.k; slices = (B + kRoundTok - 1) / kRoundTok;
    to_part = false;
    g_begin = (item % slices) * kRoundTok;
    count = min(B, g_begin + kRoundTok);
  } else if (lb.dense) {
    A = reinterpret_cast<const uint16_t*>(p.W); V = g.X; vdt = g.xdtype; K = g.d; count = B;
    slices = p.slices; to_part = true;
  } else {
    int nf = g.n_fired[0];
    nf = nf < 0 ? 0 : (nf > B ? B : nf);
    // the fired tokens' r (added to the image term), or their x (replacing it: Algorithm 1, line 7)
    A = reinterpret_cast<const uint16_t*>(p.W); V = g.wx ? g.X : g.R; K = g.d;
    if (g.wx) vdt = g.xdtype;
    count = nf; idx = g.fired_idx;
    slices = p.slices; to_part = true;
  }
  if (count == 0) return;  // uniform: no fired token, no weight byte is read
  const int rb = item / slices, ks = second ? 0 : item - rb * slices;
  const int c0 = ks * kSliceCols;
  const int ncol = min(kSliceCols, K - c0);
  const int ns = (ncol + kStepCols - 1) / kStepCols;
  const int row0 = rb * kItemRows + 16 * wave;

  // first round's activations, then the weights, so that the activations can be converted and staged while
  // the weights are still on their way
  float4 v[2][kHalfVec];
  const bool two0 = count - g_begin > 16;  // uniform
  stage_issue<T>(v, two0, V, vdt, K, idx, g_begin, count, B, c0, ncol, wave);
  __builtin_amdgcn_sched_barrier(0);
  uint4 w[kSteps];
  // uniform base + one 32-bit lane offset (the matrix is smaller than 2 GiB); rows past m repeat the last
  weights_issue<T>(w, reinterpret_cast<const char*>(A + c0), (uint32_t)min(row0 + li, m - 1) * (uint32_t)K * 2u, lq, ncol, ns);
  __builtin_amdgcn_sched_barrier(0);  // keep the weight requests ahead of the wait for the activations
  stage_commit<T>(v, two0, vt, kVRow, ncol, wave);
  weights_clear_tail<T>(w, lq, ncol, ns);

  for (int g0 = g_begin; g0 < count; g0 += kRoundTok) {
    if (g0 != g_begin) {
      __syncthreads();  // the previous round's operands have been read
      stage_issue<T>(v, count - g0 > 16, V, vdt, K, idx, g0, count, B, c0, ncol, wave);
      stage_commit<T>(v, count - g0 > 16, vt, kVRow, ncol, wave);
    }
    __syncthreads();
    f32x4 acc0, acc1;
    item_mma<T>(w, vt, kVRow, li, lq, ns, count - g0 > 16, acc0, acc1);
    // lane holds token li of each tile, rows 4*lq .. 4*lq+3 of the wave's 16
    const int row = row0 + 4 * lq;
    if (row < m) {  // m is a multiple of 4
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int j = g0 + 16 * t + li;
        if (j < count) {
          const f32x4 a = t ? acc1 : acc0;
          float* dst = to_part ? p.part + ((int64_t)ks * B + j) * m + row : p.Y + (int64_t)j * m + row;
          *reinterpret_cast<float4*>(dst) = float4{a[0], a[1], a[2], a[3]};
        }
      }
    }
  }
}

// Y[token j] (+)= sum over column slices of the partial products of the weight term.  Four threads share an
// output (each adds a quarter of the slices in order, the four sums are then added in order): fixed order, and
// one memory round trip up to 32 slices.
constexpr int kSumParts = 4, kSumOut = 256 / kSumParts;
__global__ __launch_bounds__(256) void tile_reduce(const LinBatch lb) {
  __shared__ float4 red[kSumParts][kSumOut];
  const LinTask& p = lb.t[blockIdx.y];
  const LinGroup& g = lb.g[p.group];
  const int B = lb.B, m = p.m;
  int count = B;
  if (!lb.dense) {
    const int nf = g.n_fired[0];
    count = nf < 0 ? 0 : (nf > B ? B : nf);
  }
  const int m4 = m >> 2;
  if ((int64_t)blockIdx.x * kSumOut >= (int64_t)count * m4) return;  // uniform
  const int el = threadIdx.x % kSumOut, part = threadIdx.x / kSumOut;
  const int64_t e = (int64_t)blockIdx.x * kSumOut + el;
  const bool live = e < (int64_t)count * m4;
  const int j = live ? (int)(e / m4) : 0, r4 = live ? (int)(e - (int64_t)j * m4) : 0;
  const float4* src = reinterpret_cast<const float4*>(p.part + (int64_t)j * m) + r4;
  const int64_t slice_stride = (int64_t)B * m4;
  const int per = (p.slices + kSumParts - 1) / kSumParts;
  const int s_begin = part * per, s_end = min(p.slices, s_begin + per);
  float4 s = float4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = s_begin; k0 < s_end; k0 += 8) {  // eight requests in flight; the sum keeps slice order
    float4 q[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) q[u] = src[min(k0 + u, p.slices - 1) * slice_stride];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (k0 + u < s_end) { s.x += q[u].x; s.y += q[u].y; s.z += q[u].z; s.w += q[u].w; }
  }
  red[part][el] = s;
  __syncthreads();
  if (part != 0 || !live) return;
#pragma unroll
  for (int w = 1; w < kSumParts; ++w) {
    const float4 q = red[w][el];
    s.x += q.x; s.y += q.y; s.z += q.z; s.w += q.w;
  }
  int tok = j;
  if (!lb.dense) tok = min(max(g.fired_idx[j], 0), B - 1);
  float4* y = reinterpret_cast<float4*>(p.Y + (int64_t)tok * m) + r4;
  if (lb.dense || g.wx) *y = s;
  else {
    const float4 o = *y;
    *y = float4{o.x + s.x, o.y + s.y, o.z + s.z, o.w + s.w};
  }
}


// ================================================================================================
// Projection of a decode batch (Algorithm 1, lines 1-3): c = U^T x, r = x - U c, |r|^2, |x|^2
// ================================================================================================
constexpr int kPBlock = 256;                 // partial-projection workgroup: 4 waves, one 16-column block each
constexpr int kPCols = 64;                   // columns of U per workgroup
constexpr int kPSteps = 4;                   // 32-row steps per slab of U (a slab is 128 rows)
constexpr int kPURow = kPCols + 4;           // bf16 per staged U row: the 136-byte stride keeps the four
                                             // row groups of the column-wise 16-bit reads on distinct banks
constexpr int kPXRow = kStepCols + 8;        // bf16 per staged token row (80 bytes): conflict-free 128-bit reads

// c partials: part_c[slab][t][j] = sum over the slab's rows i of U[i][j] x_t[i].
// The contraction runs over rows of U, which are not contiguous in memory, so a 32-row x 64-column tile of
// U is staged in LDS as it is stored and the A operand (16 columns x 32 rows) is gathered column-wise with
// 16-bit reads; it then serves every token tile (two MFMAs each: bf16 head and tail of the fp32 x).
// T: bf16 terms of x (bf16 activations: one, the others are zero and left out)
template <int XV, int T>  // XV = token groups of 32 the call may have (1, 2 or 4): sizes the register arrays
__global__ __launch_bounds__(kPBlock) void tile_proj_partial(const ProjBatch pb) {
  __shared__ __align__(16) uint16_t us[2][kStepCols][kPURow];
  __shared__ __align__(16) uint16_t xt[T][2][32 * XV][kPXRow];

  const int ti = find_task(pb.a_begin, pb.n, blockIdx.x);
  const ProjTask& p = pb.t[ti];
  const int local = blockIdx.x - pb.a_begin[ti];
  // the column groups of a row slab are a_slabs workgroups apart: on the same XCD when a_slabs is a multiple of 8
  // (workgroups go to the 8 XCDs in turn), and so is the residual workgroup of the same rows
  const int slab = local % p.a_slabs, cg = local / p.a_slabs;
  const int d = p.d, k = p.k, B = pb.B;
  if (local == 0 && threadIdx.x == 0) *p.sync = 0u;  // the residual launch counts its finished workgroups here
  const int row_begin = slab * p.a_rows;
  const int steps = (min(p.a_rows, d - row_begin)) / kStepCols;  // 1..4: d and a_rows are multiples of 32
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave, li = lane & 15, lq = lane >> 4;
  const int ntile = (B + 15) >> 4;
  const uint16_t* U = reinterpret_cast<const uint16_t*>(p.U);

  // staging roles: U tile 32 rows x 8 chunks of 16 bytes = 256 threads; x tile B tokens x 8 float4
  const int urow = threadIdx.x >> 3, uch = threadIdx.x & 7;
  // (columns past the rank repeat the last eight; their sums are not stored)
  const uint16_t* usrc = U + (int64_t)(row_begin + urow) * k + min(cg * kPCols + 8 * uch, k - 8);
  constexpr int kXV = XV;                     // float4 per thread and step: one per 32 tokens
  constexpr int kTiles = 2 * XV;              // MFMA token tiles
  const int xc4 = threadIdx.x & 7;
  int64_t xsrc[kXV];
#pragma unroll
  for (int u = 0; u < kXV; ++u) {
    const int t = min((int)(threadIdx.x >> 3) + 32 * u, B - 1);  // tokens past B repeat the last one
    xsrc[u] = (int64_t)t * d + row_begin + 4 * xc4;
  }
  // A slab is at most four steps (128 rows): everything it reads is requested at once, then staged and
  // consumed step by step (two LDS buffers), so the slab costs one memory round trip, not four.
  uint4 ur[kPSteps];
  float4 xr[kPSteps][kXV];
#pragma unroll
  for (int s = 0; s < kPSteps; ++s) {
    const int sc = min(s, steps - 1);  // steps past the slab repeat the last one and are not consumed
    ur[s] = *reinterpret_cast<const uint4*>(usrc + (int64_t)sc * kStepCols * k);
#pragma unroll
    for (int u = 0; u < kXV; ++u) xr[s][u] = load_act4<T == 2>(p.X, p.xdtype, xsrc[u] + sc * kStepCols);
  }
  __builtin_amdgcn_sched_barrier(0);  // every request of the slab is issued before the first wait
  auto commit = [&](int s, int buf) {
    uint2* ud = reinterpret_cast<uint2*>(&us[buf][urow][8 * uch]);
    ud[0] = uint2{ur[s].x, ur[s].y};
    ud[1] = uint2{ur[s].z, ur[s].w};
#pragma unroll
    for (int u = 0; u < kXV; ++u) {
      const int t = (threadIdx.x >> 3) + 32 * u;  // tokens past B hold a copy of the last one, never used
      uint2 term[T];
      split4<T>(xr[s][u], term);
#pragma unroll
      for (int q = 0; q < T; ++q) *reinterpret_cast<uint2*>(&xt[q][buf][t][4 * xc4]) = term[q];
    }
  };
  const int terms = p.xdtype == GSI_F32 ? T : 1;  // uniform

  constexpr int NA = T == 3 ? 2 : 1;  // three terms: the remainders have a sum of their own (add_tails)
  f32x4 acc[kTiles][NA];
#pragma unroll
  for (int t = 0; t < kTiles; ++t)
#pragma unroll
    for (int q = 0; q < NA; ++q) acc[t][q] = f32x4{0.f, 0.f, 0.f, 0.f};
  commit(0, 0);
#pragma unroll
  for (int s = 0; s < kPSteps; ++s) {
    if (s < steps) {  // uniform
      const int buf = s & 1;
      __syncthreads();  // step s is staged; step s-1 (the other buffer) has been read by every wave
      // A operand: lane (column li of the wave's block, row group lq) gathers rows 8 lq .. 8 lq + 7
      uint16_t a16[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) a16[e] = us[buf][8 * lq + e][16 * wave + li];
      uint4 ap;
      ap.x = (uint32_t)a16[0] | ((uint32_t)a16[1] << 16); ap.y = (uint32_t)a16[2] | ((uint32_t)a16[3] << 16);
      ap.z = (uint32_t)a16[4] | ((uint32_t)a16[5] << 16); ap.w = (uint32_t)a16[6] | ((uint32_t)a16[7] << 16);
      const bf16x8 a = __builtin_bit_cast(bf16x8, ap);
#pragma unroll
      for (int t = 0; t < kTiles; ++t) {
        if (t < ntile) {  // uniform
#pragma unroll
          for (int q = 0; q < T; ++q)
            if (q < terms) {
              f32x4& s16 = acc[t][NA == 2 && q > 0 ? 1 : 0];
              s16 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, *reinterpret_cast<const bf16x8*>(&xt[q][buf][16 * t + li][8 * lq]),
                                                            s16, 0, 0, 0);
            }
        }
      }
      if (s + 1 < kPSteps && s + 1 < steps) commit(s + 1, buf ^ 1);
    }
  }
  // lane holds token li of each tile, columns 4 lq .. 4 lq + 3 of the wave's block
#pragma unroll
  for (int t = 0; t < kTiles; ++t) {
    const int tok = 16 * t + li;
    if (t < ntile && tok < B && cg * kPCols + 16 * wave + 4 * lq < k) {
      float* dst = p.part_c + ((int64_t)slab * B + tok) * k + cg * kPCols + 16 * wave + 4 * lq;
      const f32x4 c = NA == 2 ? add_tails(acc[t][0], acc[t][NA - 1]) : acc[t][0];
      *reinterpret_cast<float4*>(dst) = float4{c[0], c[1], c[2], c[3]};
    }
  }
}

// C[t][j] = sum over slabs of the partial projections.  Sixteen threads share an output (each adds a sixteenth
// of the slabs in order, the sixteen sums are then added in order): fixed order, one or two memory round trips.
constexpr int kRedParts = 16, kRedOut = 256 / kRedParts;
__global__ __launch_bounds__(256) void tile_proj_reduce(const ProjBatch pb) {
  __shared__ float4 red[kRedParts][kRedOut];
  const ProjTask& p = pb.t[blockIdx.y];
  const int B = pb.B, k4 = p.k >> 2;
  const int el = threadIdx.x % kRedOut, part = threadIdx.x / kRedOut;
  const int e = blockIdx.x * kRedOut + el;
  const bool live = e < B * k4;
  const int per = (p.a_slabs + kRedParts - 1) / kRedParts;
  const int s_begin = part * per, s_end = min(p.a_slabs, s_begin + per);
  const float4* src = reinterpret_cast<const float4*>(p.part_c) + (live ? e : 0);
  const int64_t stride = (int64_t)B * k4;
  float4 s = float4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = s_begin; s0 < s_end; s0 += 8) {
    float4 q[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) q[u] = src[min(s0 + u, p.a_slabs - 1) * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (s0 + u < s_end) { s.x += q[u].x; s.y += q[u].y; s.z += q[u].z; s.w += q[u].w; }
  }
  red[part][el] = s;
  __syncthreads();
  if (part == 0 && live) {
    float4 t = red[0][el];
#pragma unroll
    for (int w = 1; w < kRedParts; ++w) {
      const float4 q = red[w][el];
      t.x += q.x; t.y += q.y; t.z += q.z; t.w += q.w;
    }
    reinterpret_cast<float4*>(p.C)[e] = t;
  }
}

// r = x - U c for 128 rows x 32 tokens per workgroup (the weights of this product are the rows of U, which are
// contiguous: same operand flow as tile_rows), R written, and the row block's share of |r|^2 and |x|^2.
// The workgroup of an input that finishes last (a counter in the workspace, zeroed by the partial-projection
// launch) turns the shares into the norms, the gate decisions and the list of fired tokens: no launch of its own.
//
// Image terms y = M c of a call's maps ride behind the residual workgroups (ib): both need c alone.  By itself the
// residual is short of work and bound by latency (160 workgroups of 128 rows for an MLP pair), and in front of the W
// items, where gated_linear alone still has them, the image items take the places of workgroups that stream weights.
// The pair of 4096 and 16384 columns, rank 256, 64 tokens: this launch 17.8 -> 20.6 us, the W items 62.6 -> 53 us; calls one
// after the other, us each: 97.5 -> 93.6 (20 tokens: 75.5 -> 73.7, 128: 125.3 -> 116.8; a block at rank 200, 24 tokens:
// 54.1 -> 47.2).  With other work between the calls they take 3 to 5 us more.
// LDS holds the operand of the launch's largest rank only (vrow), so that the short items of small ranks share a unit.
template <int TI, int N>
__device__ __forceinline__ void image_item(const TileImg& p, int item, int B, int per, uint16_t* vt, int vrow, int wave,
                                           int li, int lq) {
  const int nrb = (p.m + kItemRows - 1) / kItemRows;
  const int rb = item % nrb, end = min(B, (item / nrb + 1) * per);
  int g0 = (item / nrb) * per;
  const int m = p.m, k = p.k, ns = (k + kStepCols - 1) / kStepCols;
  const int row0 = rb * kItemRows + 16 * wave;
  float4 v[2][kHalfVec];
  stage_issue<TI>(v, end - g0 > 16, p.C, GSI_F32, k, nullptr, g0, end, B, 0, k, wave);
  __builtin_amdgcn_sched_barrier(0);
  uint4 w[N];
  weights_issue<TI>(w, reinterpret_cast<const char*>(p.M), (uint32_t)min(row0 + li, m - 1) * (uint32_t)k * 2u, lq, k, ns);
  __builtin_amdgcn_sched_barrier(0);
  stage_commit<TI>(v, end - g0 > 16, vt, vrow, k, wave);
  weights_clear_tail<TI>(w, lq, k, ns);
  for (;;) {
    const bool more = TI == 2 && N < kSteps && end - g0 > kRoundTok;  // uniform
    if (more) stage_issue<TI>(v, end - g0 > kRoundTok + 16, p.C, GSI_F32, k, nullptr, g0 + kRoundTok, end, B, 0, k, wave);
    __syncthreads();
    f32x4 acc0, acc1;
    item_mma<TI>(w, vt, vrow, li, lq, ns, end - g0 > 16, acc0, acc1);
    const int row = row0 + 4 * lq;
    if (row < m) {  // m is a multiple of 4
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int j = g0 + 16 * t + li;
        const f32x4 a = t ? acc1 : acc0;
        if (j < end) *reinterpret_cast<float4*>(p.Y + (int64_t)j * m + row) = float4{a[0], a[1], a[2], a[3]};
      }
    }
    if (!more) return;
    __syncthreads();  // the operands of this round have been read
    g0 += kRoundTok;
    stage_commit<TI>(v, end - g0 > 16, vt, vrow, k, wave);
  }
}

// N: steps of a rank, 16, or 8 or 4, where the registers of two terms have room for several rounds of 32 tokens (per tokens)
template <int T, int N>
__global__ __launch_bounds__(kTBlock, 4) void tile_residual(const ProjBatch pb, const TileImgBatch ib, int vrow, int per) {
  extern __shared__ __align__(16) uint16_t vt[];  // [T][kRoundTok][vrow]
  __shared__ int s_last;
  __shared__ float red[kTWaves][kRoundTok][2];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave, li = lane & 15, lq = lane >> 4;
  const int B = pb.B;
  if ((int)blockIdx.x >= pb.b_total) {
    const int item = blockIdx.x - pb.b_total;
    int ii = 0;
#pragma unroll
    for (int i = 1; i < kMaxLinTasks; ++i)
      if (i < ib.n && item >= ib.t[i].blk_begin) ii = i;
    const TileImg& p = ib.t[ii];
    if (T == 2 || p.terms == 2) image_item<2, N>(p, item - p.blk_begin, B, per, vt, vrow, wave, li, lq);
    else image_item<T, N>(p, item - p.blk_begin, B, per, vt, vrow, wave, li, lq);
    return;
  }
  const int ti = find_task(pb.b_begin, pb.n, blockIdx.x);
  const ProjTask& p = pb.t[ti];
  const int groups = (B + per - 1) / per;
  const int item = blockIdx.x - pb.b_begin[ti];
  const int nrb = p.d / kItemRows;  // row blocks; the token groups of a row block are nrb workgroups apart (same XCD)
  const int rb = item % nrb, end = min(B, (item / nrb + 1) * per);
  int g0 = (item / nrb) * per;
  const int d = p.d, k = p.k, ns = (k + kStepCols - 1) / kStepCols;
  const int row0 = rb * kItemRows + 16 * wave;  // d is a multiple of 128: every row exists
  const uint16_t* U = reinterpret_cast<const uint16_t*>(p.U);

  float4 v[2][kHalfVec];
  stage_issue<T>(v, end - g0 > 16, p.C, GSI_F32, k, nullptr, g0, end, B, 0, k, wave);
  __builtin_amdgcn_sched_barrier(0);
  uint4 w[N];
  weights_issue<T>(w, reinterpret_cast<const char*>(U), (uint32_t)(row0 + li) * (uint32_t)k * 2u, lq, k, ns);
  // x of the lane's outputs: token g0 + 16 t + li, rows row0 + 4 lq .. + 3
  float4 xv[2];
  auto request_x = [&](int g) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int j = min(g + 16 * t + li, B - 1);
      xv[t] = load_act4<T == 2>(p.X, p.xdtype, (int64_t)j * d + row0 + 4 * lq);
    }
  };
  request_x(g0);
  __builtin_amdgcn_sched_barrier(0);
  stage_commit<T>(v, end - g0 > 16, vt, vrow, k, wave);
  weights_clear_tail<T>(w, lq, k, ns);
  float4 r[2];
  auto store_r = [&]() {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int j = g0 + 16 * t + li;
      if (j < end) *reinterpret_cast<float4*>(p.R + (int64_t)j * d + row0 + 4 * lq) = r[t];
    }
  };
  for (;;) {
    const bool more = T == 2 && N < kSteps && end - g0 > kRoundTok;  // uniform
    if (more) stage_issue<T>(v, end - g0 > kRoundTok + 16, p.C, GSI_F32, k, nullptr, g0 + kRoundTok, end, B, 0, k, wave);
    __syncthreads();
    f32x4 acc0, acc1;
    item_mma<T>(w, vt, vrow, li, lq, ns, end - g0 > 16, acc0, acc1);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int j = g0 + 16 * t + li;
      const f32x4 a = t ? acc1 : acc0;
      const float4 x = xv[t];
      r[t] = float4{x.x - a[0], x.y - a[1], x.z - a[2], x.w - a[3]};
      float sr = 0.f, sx = 0.f;
      if (j < end) {
        sr = fmaf(r[t].x, r[t].x, fmaf(r[t].y, r[t].y, fmaf(r[t].z, r[t].z, r[t].w * r[t].w)));
        sx = fmaf(x.x, x.x, fmaf(x.y, x.y, fmaf(x.z, x.z, x.w * x.w)));
      }
      // the four row groups of the wave (lanes li, li+16, li+32, li+48), fixed order
      sr += __shfl_xor(sr, 16); sr += __shfl_xor(sr, 32);
      sx += __shfl_xor(sx, 16); sx += __shfl_xor(sx, 32);
      if (lq == 0) {
        red[wave][16 * t + li][0] = sr;
        red[wave][16 * t + li][1] = sx;
      }
    }
    __syncthreads();
    if (threadIdx.x < 2 * kRoundTok) {
      const int tl = threadIdx.x >> 1, c = threadIdx.x & 1;
      if (g0 + tl < end) {
        float sum = 0.f;
#pragma unroll
        for (int wv = 0; wv < kTWaves; ++wv) sum += red[wv][tl][c];
        // written through to memory (a store that is coherent across the chip), so that the workgroup that finishes
        // last can read it without anybody writing a whole L2 back: such a write-back costs about a microsecond per
        // workgroup, one after the other
        __hip_atomic_store(&p.part_n[((int64_t)rb * B + g0 + tl) * 2 + c], sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (!more) break;
    store_r();
    g0 += kRoundTok;
    request_x(g0);
    stage_commit<T>(v, end - g0 > 16, vt, vrow, k, wave);  // (every wave has read the operands of the round before)
  }
  if (!pb.norms) {  // uniform
    store_r();
    return;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the shares have reached memory ...
  __syncthreads();                                  // ... in every wave before the workgroup counts as done
  if (threadIdx.x == 0) {
    const unsigned done = __hip_atomic_fetch_add(p.sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = done + 1u == (unsigned)(nrb * groups);
  }
  store_r();  // (nothing of this launch reads R: behind the count, so that the wait above is not for it)
  __syncthreads();
  if (!s_last) return;  // uniform
  norms_and_gate<kTBlock>(p, B, pb.gate, pb.eps, reinterpret_cast<float2*>(vt),
                          reinterpret_cast<int*>(reinterpret_cast<float2*>(vt) + kTBlock));
}

}  // namespace

int tile_slices(int64_t d) { return (int)ceil_div(d, kSliceCols); }

// ---- projection ---------------------------------------------------------------------------------
bool tile_project_shape_ok(int64_t d, int64_t k, int64_t B, int udtype) {
  return udtype == GSI_BF16 && B >= 2 && B <= kMaxTok && d % kItemRows == 0 && k % 8 == 0 && k <= kSliceCols &&
         d < (1 << 24);
}

static int tile_slab_rows(int64_t) { return kPSteps * kStepCols; }

// A residual launch with images, of up to one and a half workgroups per compute unit, asks for more than half of a unit's LDS, so that
// the residual workgroups, which come first, have a unit each and the images the next free one: MLP pair of 4096 and 16384
// columns, rank 256 (320 workgroups), calls one after the other, 4 tokens 69.4 us each against 70.0, 16 tokens
// 70.6 against 71.5.  With more, two share
// a unit: a block at rank 200, 8 tokens (512 workgroups) 41.9 us against 46.4; the pair with 128 tokens 116.8 against 124.8.
constexpr int kFewItems = 384;
constexpr int kResident = 512;  // workgroups: two per compute unit
constexpr size_t kWholeUnit = 84 * 1024;

size_t tile_project_ws(int64_t d, int64_t k, int64_t B) {
  const int a_slabs = (int)ceil_div(d, tile_slab_rows(d));
  return align_up((size_t)a_slabs * B * k * 4, 256) + align_up((size_t)(d / kItemRows) * B * 2 * 4, 256) + 256;
}

void tile_project_fill(ProjTask& t, int64_t d, int64_t k, int64_t B, void* ws) {
  t.d = (int)d;
  t.k = (int)k;
  t.a_rows = tile_slab_rows(d);
  t.a_slabs = (int)ceil_div(d, t.a_rows);
  t.a_cblocks = (int)ceil_div(k, kPCols);
  t.b_rows = kItemRows;
  t.b_slabs = (int)(d / kItemRows);
  t.part_c = reinterpret_cast<float*>(ws);
  t.part_n = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + align_up((size_t)t.a_slabs * B * k * 4, 256));
  t.sync = reinterpret_cast<unsigned*>(reinterpret_cast<char*>(t.part_n) + align_up((size_t)t.b_slabs * B * 2 * 4, 256));
}

hipError_t tile_proj_reduce_launch(const ProjBatch& pb, hipStream_t s) {
  int max_k = 0;
  for (int i = 0; i < pb.n; ++i) max_k = max_k > pb.t[i].k ? max_k : pb.t[i].k;
  const dim3 grid((unsigned)ceil_div((int64_t)pb.B * (max_k / 4), kRedOut), (unsigned)pb.n);
  tile_proj_reduce<<<grid, 256, 0, s>>>(pb);
  return hipGetLastError();
}

hipError_t tile_project_launch(ProjBatch& pb, bool with_norms, bool with_gate, float eps, hipStream_t s, TileImgBatch& ib) {
  if (pb.n == 0 || pb.B == 0) return hipSuccess;
  int max_k = 0;
  for (int i = 0; i < pb.n; ++i) max_k = std::max(max_k, pb.t[i].k);  // (an image's rank is that of its input)
  const int steps = max_k <= kSliceCols / 4 ? kSteps / 4 : pb.t[0].tile == 2 && max_k <= kSliceCols / 2 ? kSteps / 2 : kSteps;
  // Tokens of a workgroup: as many rounds of 32, which share its rows, as let the whole launch be resident at once, while the registers of
  // the rank's steps leave room for the next round's tokens (two terms, ranks of up to 256).  us a call, 32 tokens a workgroup and
  // 16 steps / so: the pair 4096 / 16384 at rank 256, 64 tokens 96.9 / 92.6, 128 tokens 124.7 / 118.0, 4 tokens 74.2 / 71.6 (its eight
  // steps); a block at rank 128, 128 tokens 171 / 151; three terms, a block of 2560 / 10240 at rank 128, 23 tokens 64.4 / 62.8.
  int64_t blocks = 0;
  for (int i = 0; i < pb.n; ++i) blocks += pb.t[i].b_slabs;
  for (int i = 0; i < ib.n; ++i) blocks += ceil_div(ib.t[i].m, kItemRows);
  int per = kRoundTok;
  while (pb.t[0].tile == 2 && steps < kSteps && per < pb.B && blocks * ceil_div(pb.B, per) > kResident) per *= 2;
  const int rounds = (int)ceil_div(pb.B, per);
  int ta = 0, tb = 0;
  for (int i = 0; i < pb.n; ++i) {
    pb.a_begin[i] = ta;
    pb.b_begin[i] = tb;
    ta += pb.t[i].a_slabs * pb.t[i].a_cblocks;
    tb += pb.t[i].b_slabs * rounds;
  }
  pb.b_total = tb;
  pb.norms = with_norms ? 1 : 0;
  pb.gate = with_gate ? 1 : 0;
  pb.eps = eps;
  int imgs = 0;
  for (int i = 0; i < ib.n; ++i) {
    ib.t[i].blk_begin = imgs;
    imgs += (int)ceil_div(ib.t[i].m, kItemRows) * rounds;
  }
  const int vrow = (int)align_up((size_t)max_k, kStepCols) + 8;
  hipError_t err = hipSuccess;
  auto launch = [&](auto terms) {
    constexpr int T = decltype(terms)::value;
    constexpr size_t kScratch = kTBlock * sizeof(float2) + 16;  // norms_and_gate
    size_t smem = std::max((size_t)T * kRoundTok * vrow * sizeof(uint16_t), kScratch);
    if (imgs > 0 && per == kRoundTok && tb + imgs <= kFewItems) smem = std::max(smem, kWholeUnit);
    auto residual = [&](auto n) {  // (LDS: more than the default 64 KB at the largest ranks)
      constexpr int N = decltype(n)::value;
      static LdsLimit lds;
      const int most = std::max(T * kRoundTok * (N * kStepCols + 8) * (int)sizeof(uint16_t), (int)kWholeUnit);
      if (err == hipSuccess) err = lds.allow(reinterpret_cast<const void*>(&tile_residual<T, N>), most);
      if (err == hipSuccess) tile_residual<T, N><<<tb + imgs, kTBlock, smem, s>>>(pb, ib, vrow, per);
    };
    if (pb.B <= 32) tile_proj_partial<1, T><<<ta, kPBlock, 0, s>>>(pb);
    else if (pb.B <= 64) tile_proj_partial<2, T><<<ta, kPBlock, 0, s>>>(pb);
    else tile_proj_partial<4, T><<<ta, kPBlock, 0, s>>>(pb);
    err = tile_proj_reduce_launch(pb, s);
    if (err != hipSuccess) return;
    if (steps == kSteps / 4) residual(std::integral_constant<int, kSteps / 4>{});
    else if (steps == kSteps) residual(std::integral_constant<int, kSteps>{});
    else if constexpr (T == 2) residual(std::integral_constant<int, kSteps / 2>{});
  };
  if (pb.t[0].tile == 3) launch(std::integral_constant<int, 3>{});
  else launch(std::integral_constant<int, 2>{});
  if (err != hipSuccess) return err;
  return hipGetLastError();
}

// shapes the matrix-core linear kernel takes (alignments and the partial-product workspace apart: tile_rows_ok)
bool tile_rows_shape_ok(int64_t m, int64_t d, int64_t k, int64_t B, int wdtype) {
  return wdtype == GSI_BF16 && B >= 2 && B <= kMaxTok && d % kStepCols == 0 && m % 4 == 0 &&
         m * d * 2 < (1ll << 32) && (k == 0 || (k % 8 == 0 && k <= kSliceCols));
}

size_t tile_part_bytes(int64_t m, int64_t d, int64_t B) {
  if (B < 2 || B > kMaxTok || d % kStepCols || m % 4) return 0;
  return align_up((size_t)tile_slices(d) * B * m * sizeof(float), 256);
}

// three terms where the rows ran on fp32 FMAs before this kernel took them: ranks that are no multiple of 32, and bf16
// activations (themselves a single term)
int tile_rows_terms(const LinBatch& lb, int group) {
  const LinGroup& g = lb.g[group];
  return tile_image_terms(lb.dense ? 0 : g.k, lb.dense || g.wx, g.xdtype);
}
int tile_image_terms(int64_t k, bool reads_x, int xdtype) { return k % kStepCols || (reads_x && xdtype != GSI_F32) ? 3 : 2; }

// what the image items of tile_rows need of a map whose input's C they read
bool tile_image_ok(int64_t m, int64_t k, const void* M, const void* C, const void* Y) {
  return m % 4 == 0 && k % 8 == 0 && k <= kSliceCols && m * k * 2 < (1ll << 32) && reinterpret_cast<uintptr_t>(M) % 16 == 0 &&
         reinterpret_cast<uintptr_t>(C) % 16 == 0 && reinterpret_cast<uintptr_t>(Y) % 16 == 0;
}

// The dense product of two bf16 tokens with short rows (2048 columns, 2^24 elements): one launch of the FMA kernel is
// shorter than these rows and the launch that adds their slices.  us: 3072 x 768 7.5 against 10.6, 1000 x 1024 8.0 against
// 10.3; 8192 x 2048 12.6 against 14.1, 4096 x 4096 19.0 against 12.8; three tokens, 3072 x 768 9.9 against 10.7, 1000 x 1024
// 10.9 against 10.6.
bool tile_rows_longer(const LinBatch& lb, int task) {
  const LinTask& t = lb.t[task];
  const LinGroup& g = lb.g[t.group];
  return lb.dense && lb.B == 2 && g.xdtype != GSI_F32 && g.d <= 2048 && (int64_t)t.m * g.d <= (1 << 24);
}

bool tile_rows_ok(const LinBatch& lb, int wdtype) {
  if (wdtype != GSI_BF16 || lb.B < 2 || lb.B > kMaxTok) return false;
  for (int i = 0; i < lb.ng; ++i) {
    const LinGroup& g = lb.g[i];
    if (g.d % kStepCols) return false;
    if (lb.dense || g.wx) {
      if (reinterpret_cast<uintptr_t>(g.X) % 16) return false;
    }
    if (!lb.dense) {
      if (g.k % 8 || g.k > kSliceCols) return false;
      if (reinterpret_cast<uintptr_t>(g.C) % 16 || reinterpret_cast<uintptr_t>(g.R) % 16) return false;
    }
  }
  for (int i = 0; i < lb.n; ++i) {
    const LinTask& t = lb.t[i];
    if (tile_rows_longer(lb, i)) return false;
    if (t.m % 4 || reinterpret_cast<uintptr_t>(t.Y) % 16 || reinterpret_cast<uintptr_t>(t.W) % 16) return false;
    if ((int64_t)t.m * lb.g[t.group].d * 2 >= (1ll << 32)) return false;  // 32-bit byte offsets into a matrix
    if (!t.part || reinterpret_cast<uintptr_t>(t.part) % 16) return false;
    if (!lb.dense && reinterpret_cast<uintptr_t>(t.M) % 16) return false;
  }
  return true;
}

hipError_t tile_rows_launch(LinBatch& lb, hipStream_t s) {
  int total = 0, max_m = 0;
  for (int i = 0; i < lb.n; ++i) {
    lb.blk_begin2[i] = total;
    if (!lb.dense && !lb.t[i].img_done) total += (int)(ceil_div(lb.t[i].m, kItemRows) * ceil_div(lb.B, kRoundTok));
  }
  lb.tile_split = total;  // image items below, weight items from here on
  for (int i = 0; i < lb.n; ++i) {
    lb.t[i].slices = tile_slices(lb.g[lb.t[i].group].d);
    lb.blk_begin[i] = total;
    total += (int)ceil_div(lb.t[i].m, kItemRows) * lb.t[i].slices;
    if (lb.t[i].m > max_m) max_m = lb.t[i].m;
  }
  if (tile_rows_terms(lb, 0) == 3) tile_rows<3><<<total, kTBlock, 0, s>>>(lb);
  else tile_rows<2><<<total, kTBlock, 0, s>>>(lb);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  const dim3 grid((unsigned)ceil_div((int64_t)lb.B * (max_m / 4), kSumOut), (unsigned)lb.n);
  tile_reduce<<<grid, 256, 0, s>>>(lb);
  return hipGetLastError();
}

}  // namespace gsi
