// Prefill-sized products whose operands are bf16 in memory: from there to LDS without registers, 256 x 256 tiles.
//
// D = A B^T, both operands K-contiguous.  A workgroup of eight waves has a tile of 256 x 256; a k-tile is 64 columns, two of
// them in LDS (128 KB, one workgroup per compute unit).  The tile of each operand lies there as two halves of 128 rows.  A wave
// owns 64 rows and 32 columns of each pair of halves (waves 2 x 4), so a k-tile is four steps, one pair of halves each: A0 B0,
// A0 B1, A1 B1, A1 B0, sixteen v_mfma_f32_16x16x32_bf16 a step.  Four waves are half a step behind the other four: one wave of
// a SIMD reads its operands from LDS while the other one's products run (a barrier between the halves of a step keeps them
// so; all eight in step: 1188 TFLOP/s in place of 1372).  In every step a thread requests the two 16-byte pieces of a half two
// k-tiles ahead, into the half that was read last, and waits for those that the next step reads: six halves, 96 KB a unit, are
// always on their way.
// In LDS a row of a half is 128 bytes, its 16-byte piece c at c ^ (row / 2 % 8): sixteen rows of one piece, which a read of 128
// bits takes at a time, lie in distinct banks (c ^ row % 8: 1200 in place of 1354 TFLOP/s).  The loads write LDS in lane order,
// so it is the lane that loads another piece of its row.
// What bounds it is the power of the matrix cores: 8192^3 1467 TFLOP/s on random operands, 2022 on zeros; 32 x 32 x 16
// products 1251 and 1883.  2048 x 16384 x 4096: 1395 TFLOP/s (gemm_nt, whose operands go through registers: 1004).
#include <algorithm>

#include "gsi_mfma_device.h"

namespace gsi {
namespace {

constexpr int kWideThreads = 512;
constexpr int kWideTile = 256;
constexpr int kHalf = 128 * 128;       // bytes of a half: 128 rows of 64 columns
constexpr int kWideStage = 4 * kHalf;  // A0 A1 B0 B1

// Sums of a wave: [h][g][i][j][v]: row 128 h + 32 i + 16 wm + lane % 16 of the tile, column 128 g + 32 wn + 16 j + 4 (lane / 16) + v
// (the columns of B are the first operand of the products, so that a lane has four neighbouring columns of a row).
typedef f32x4 WideAcc[2][2][4][2];

// The sums of one tile over the k-tiles kt0 .. kt1 (at least one).  a, b: buffers over the rows of the tile; rows: how many A and
// B have (at least one; the last stands in for those past it, whose sums mean nothing); N0, N1: row fragments of 16 of each half
// that the wave multiplies (its own: the barriers are the same for all).  Every wave has passed the last barrier of the loop when it returns, and no load is on its way.
template <int N0, int N1>
__device__ __forceinline__ void wide_loop(char* lds, const u32x4& a, int64_t lda, int a_rows, const u32x4& b, int64_t ldb, int b_rows, int kt0,
                                          int kt1, WideAcc& acc) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w >> 2, wn = w & 3, lc = lane & 15, lq = lane >> 4;
  const int nk = kt1 - kt0;
  // requests: a wave has rows 8 w .. and 64 + 8 w .. of every half, eight lanes a row
  uint32_t va[2][2], vb[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int row = 64 * q + 8 * w + (lane >> 3);
      const uint32_t piece = 16u * ((lane & 7) ^ ((row >> 1) & 7));
      va[h][q] = (uint32_t)(min(128 * h + row, a_rows - 1) * lda * 2) + piece;
      vb[h][q] = (uint32_t)(min(128 * h + row, b_rows - 1) * ldb * 2) + piece;
    }
  const uint32_t to = (uint32_t)(uintptr_t)(lds_char*)lds + w * 1024;
  // which: 0 B0, 1 A0, 2 B1, 3 A1, the order in which they are read; past the range the last k-tile again, never read
  auto request = [&](int kt, int stage, int which) {
    const uint32_t soff = (uint32_t)(kt0 + min(kt, nk - 1)) * 128u;
    const uint32_t dst = to + stage * kWideStage + ((which & 1) ? 0 : 2 * kHalf) + (which >> 1) * kHalf;
    const int h = which >> 1;
    if (which & 1) {
      load_to_lds(dst, a, va[h][0], soff);
      load_to_lds(dst + kHalf / 2, a, va[h][1], soff);
    } else {
      load_to_lds(dst, b, vb[h][0], soff);
      load_to_lds(dst + kHalf / 2, b, vb[h][1], soff);
    }
  };
  uint32_t oa[2], ob[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int piece = 16 * ((4 * k + lq) ^ (lc >> 1));
    oa[k] = (16 * wm + lc) * 128 + piece;
    ob[k] = 2 * kHalf + (32 * wn + lc) * 128 + piece;
  }
#pragma unroll
  for (int f = 0; f < 32; ++f) acc[f >> 4][(f >> 3) & 1][(f >> 1) & 3][f & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 ra[4][2], rb0[2][2][2], rb1[2][2];
  auto read_a = [&](int stage, int h) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < (h ? N1 : N0); ++i) ra[i][k] = *reinterpret_cast<const bf16x8*>(lds + stage * kWideStage + oa[k] + h * kHalf + i * 4096);
  };
  auto read_b = [&](int stage, int g, bf16x8 (&x)[2][2]) {
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int j = 0; j < 2; ++j) x[j][k] = *reinterpret_cast<const bf16x8*>(lds + stage * kWideStage + ob[k] + g * kHalf + j * 2048);
  };
  auto products = [&](int h, int g, const bf16x8 (&x)[2][2]) {
    const int n = h ? N1 : N0;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < n; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[h][g][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[j][k], ra[i][k], acc[h][g][i][j], 0, 0, 0);
  };
  // A step: operands read and the next request out, then, behind the barrier that lets the other four waves read, the
  // products.  What has been read is in registers before that barrier: behind it its half may be overwritten.
  auto step = [&](int h, int g, const bf16x8 (&x)[2][2]) {
    wait_loads<12>();
    wait_lds();
    barrier();
    products(h, g, x);
    barrier();
  };
  for (int q = 0; q < 4; ++q) request(0, 0, q);
  for (int q = 0; q < 4; ++q) request(1, 1, q);
  wait_loads<12>();  // B0 and A0 of the first k-tile
  barrier();
  read_b(0, 0, rb0[0]);
  wait_lds();
  barrier();              // the first step requests into that half
  if (w >= 4) barrier();  // half a step behind
  auto tile = [&](int t, int stage, bf16x8 (&now)[2][2], bf16x8 (&next)[2][2]) {
    read_a(stage, 0);
    request(t + 2, stage, 0);
    step(0, 0, now);
    read_b(stage, 1, rb1);
    request(t + 2, stage, 1);
    step(0, 1, rb1);
    read_a(stage, 1);
    request(t + 2, stage, 2);
    step(1, 1, rb1);
    read_b(stage ^ 1, 0, next);
    request(t + 2, stage, 3);
    step(1, 0, now);
  };
  int t = 0;
  for (; t + 1 < nk; t += 2) {
    tile(t, 0, rb0[0], rb0[1]);
    tile(t + 1, 1, rb0[1], rb0[0]);
  }
  if (t < nk) tile(t, 0, rb0[0], rb0[1]);
  if (w < 4) barrier();
  wait_loads<0>();
}

// Scatter products over a device-side count of fired rows: A[i] is the i-th of them (round_rows), D's row is row_idx[i].  The
// workgroups of a launch are dealt to the pieces (row tile, column tile, part of the contraction) of the products in order, as
// many as the counts make; the others leave.  The row tiles of a product are of one height, a multiple of 16 rows, and the
// products of rows past it are left out (410 rows: two of 208).  Row tiles of a column tile are eight workgroups apart, on the
// same XCD: its L2 reads the weights once.
// The tiles are as high as 256 rows let them be only where the pieces of all products fill the chip: the parts, which the order of a sum
// follows, are the same for a map by itself as for one beside others, and a square map alone was 64 pieces.  With fewer pieces than half the
// chip has units there are up to eight times the row tiles, of as many rows less.  us a call of gsi_gated_linear at rank 128, one
// height / so: 4096 x 4096, 409 of 2048 tokens 83 / 72, 580 of 2900 117 / 96; 2176 x 7168, 409 of 2048 96 / 78; 2560 x 10240, 300 of 1500 104 / 91.
template <int ONCE>
__global__ __launch_bounds__(kWideThreads, 2) void wide_scatter_kernel(const GemmArgs args) {
  __shared__ __align__(1024) char lds[2 * kWideStage];
  const int lane = threadIdx.x & 63;
  // lane q: the pieces of product q
  int rows = 0, tiles = 0, each = 0;
  if (lane < args.n) {
    const GemmProb& g = args.p[lane];
    rows = min(g.n_rows_dev[0], g.M);
    if (rows > 0) {
      tiles = (rows + kWideTile - 1) / kWideTile;
      each = g.col_tiles * parts_for(g, rows);
    }
  }
  int all = 0;  // pieces of the launch
  for (int q = 0; q < args.n; ++q) all += __builtin_amdgcn_readlane(tiles * each, q);
  const int fold = max(1, min(8, kUnits / max(all, 1)));
  tiles = min(fold * tiles, (rows + 15) / 16);
  const int pieces = tiles * each;
  int local = blockIdx.x, pi = 0;
  for (; pi < args.n; ++pi) {
    const int n = __builtin_amdgcn_readlane(pieces, pi);
    if (local < n) break;
    local -= n;
  }
  if (pi == args.n) return;
  const GemmProb& g = args.p[pi];
  const int Mrows = __builtin_amdgcn_readlane(rows, pi);
  const int row_tiles = __builtin_amdgcn_readlane(tiles, pi), parts = parts_for(g, Mrows), ct = g.col_tiles;
  const int split = local / (ct * row_tiles), q = local - split * ct * row_tiles;
  int tile_m, tile_n;
  if (ct % 8 == 0) {
    tile_m = (q >> 3) % row_tiles;
    tile_n = (q >> 3) / row_tiles * 8 + (q & 7);
  } else {
    tile_m = q % row_tiles;
    tile_n = q / row_tiles;
  }
  const int height = 16 * ((Mrows + 16 * row_tiles - 1) / (16 * row_tiles));
  const int row0 = tile_m * height, a_rows = min(height, Mrows - row0), b_rows = min(kWideTile, g.N - tile_n * kWideTile);
  if (a_rows <= 0) return;  // (uniform; a few rows more than whole tiles of 16 can leave the last one without any)
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w >> 2, wn = w & 3;
  const int frags = (a_rows + 15) / 16;
  const int n0 = (min(frags, 8) + 1 - wm) / 2, n1 = (max(frags - 8, 0) + 1 - wm) / 2;
  const int nk = g.K / BK;
  const int64_t lda = g.lda, ldb = g.ldb, ldd = g.ldd;
  const u32x4 a = buffer_of(reinterpret_cast<const uint16_t*>(g.A) + row0 * lda, ((a_rows - 1) * lda + g.K) * 2);
  const u32x4 b = buffer_of(reinterpret_cast<const uint16_t*>(g.B) + (int64_t)tile_n * kWideTile * ldb, ((b_rows - 1) * ldb + g.K) * 2);
  WideAcc acc;
  const int kt0 = (int)((int64_t)nk * split / parts), kt1 = (int)((int64_t)nk * (split + 1) / parts);
  switch (n1) {  // (uniform in a wave)
    case 4: wide_loop<4, 4>(lds, a, lda, a_rows, b, ldb, b_rows, kt0, kt1, acc); break;
    case 3: wide_loop<4, 3>(lds, a, lda, a_rows, b, ldb, b_rows, kt0, kt1, acc); break;
    case 2: wide_loop<4, 2>(lds, a, lda, a_rows, b, ldb, b_rows, kt0, kt1, acc); break;
    case 1: wide_loop<4, 1>(lds, a, lda, a_rows, b, ldb, b_rows, kt0, kt1, acc); break;
    default:
      if (n0 > 2) wide_loop<4, 0>(lds, a, lda, a_rows, b, ldb, b_rows, kt0, kt1, acc);
      else wide_loop<2, 0>(lds, a, lda, a_rows, b, ldb, b_rows, kt0, kt1, acc);
  }

  // a lane has 16 bytes of a row, the four lanes of the row and the two fragments j a 128-byte line
  const int lc = lane & 15, lq = lane >> 4;
  const int col0 = tile_n * kWideTile + 32 * wn + 4 * lq;
  const bool partial = parts > 1;
  float* const base = partial ? g.part + (int64_t)split * Mrows * g.N : reinterpret_cast<float*>(g.D);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i >= (h ? n1 : n0)) continue;
      const int r = 128 * h + 32 * i + 16 * wm + lc;
      const bool live = r < a_rows;
      const int row = row0 + min(r, a_rows - 1);
      float* const dst = base + (partial ? (int64_t)row * g.N : (int64_t)g.row_idx[row] * ldd);
      float4 old[2][2];
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        const int col = col0 + 128 * (f >> 1) + 16 * (f & 1);
        old[f >> 1][f & 1] = float4{0.f, 0.f, 0.f, 0.f};
        if (!partial && live && col < g.N) old[f >> 1][f & 1] = load_row<ONCE != 0>(dst + col);
      }
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        const int col = col0 + 128 * (f >> 1) + 16 * (f & 1);
        if (!live || col >= g.N) continue;  // N is a multiple of 4
        const f32x4 s = acc[h][f >> 1][i][f & 1];
        const float4 o = old[f >> 1][f & 1];
        if (partial) *reinterpret_cast<float4*>(dst + col) = float4{s[0], s[1], s[2], s[3]};
        else store_row<ONCE != 0>(dst + col, float4{o.x + s[0], o.y + s[1], o.z + s[2], o.w + s[3]});
      }
    }
}

// The rows of C in two terms.
constexpr int kMaxSplitTasks = 64;
struct SplitArgs {
  SplitTask t[kMaxSplitTasks];
};
static_assert(sizeof(SplitArgs) <= 4096, "kernel arguments are limited to 4 KB");
// The fired rows of R, one after the other, rounded once to bf16.
constexpr int kMaxRoundTasks = 64;
struct RoundArgs {
  RoundTask t[kMaxRoundTasks];
};
static_assert(sizeof(RoundArgs) <= 4096, "kernel arguments are limited to 4 KB");
// pieces of eight: first, first + stride ..
template <int ONCE>
__device__ __forceinline__ void round_part(const RoundTask& t, int64_t first, int64_t stride) {
  const int n = min(t.n_fired[0], t.rows), d8 = t.d >> 3;
  const int64_t total = (int64_t)n * d8;
  for (int64_t e = first; e < total; e += stride) {
    const int row = (int)(e / d8), c = 8 * (int)(e - (int64_t)row * d8);
    const float* const src = t.R + (int64_t)t.fired_idx[row] * t.d + c;
    const float4 x = load_row<ONCE != 0>(src), y = load_row<ONCE != 0>(src + 4);
    const float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
    uint32_t o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const __bf16 lo = (__bf16)v[2 * q], hi = (__bf16)v[2 * q + 1];
      o[q] = (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
    }
    *reinterpret_cast<u32x4*>(t.out + (int64_t)row * t.d + c) = u32x4{o[0], o[1], o[2], o[3]};
  }
}
template <int ONCE>
__global__ __launch_bounds__(256) void round_rows(const RoundArgs args) {
  round_part<ONCE>(args.t[blockIdx.y], (int64_t)blockIdx.x * blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x);
}

// Products of an operand in two terms: A is fp32 laid out as bf16 head and tail (split_rows), D = head B^T + tail B^T.  The
// residual and image products of a prefill-sized call: short (the rank) with long epilogues (every row of R and Y), so a
// workgroup is four waves (2 x 2, 64 x 128 each) with a tile of 128 x 256 and half a compute unit: one's epilogue beside the
// other's products.  A k-tile is 32 columns: a row of A is 64 bytes of head and 64 of tail, laid out in LDS as in wide_loop, a
// row of B 64 bytes, whose piece c lies at c ^ {0, 3, 2, 1}[row / 4 % 4].  One read of B serves both terms.  Rows past the end are read as
// zero.  A wave has all the operands of a k-tile in registers before its products, so that the k-tile after the next is requested over it
// at once.
// As many workgroups as the chip holds take tile after tile; the first two k-tiles of a tile are requested beside the last
// two of the one before, and arrive before its epilogue begins.
// A block of 2048 tokens at rank 512 (275 GFLOP, 0.65 GB of x, R and Y): 310 to 350 us in gemm_nt, 290 here; without the
// stores 242, the epilogues alone 158.  No bank conflicts; the matrix cores are busy for 65 % of the time at 2.1 GHz (on zeros
// 270).  A workgroup per tile 304, with x requested strip by strip and a sum of 32 lanes per row 354; raised priority of the
// waves around their products 290.
constexpr int kTwoThreads = 256, kTwoRows = 128, kTwoCols = 256, kTwoGroups = 2 * kUnits;
constexpr int kTwoA = kTwoRows * 128, kTwoStage = kTwoA + kTwoCols * 64;
constexpr int kTwoStrip = 16 * 64 * 4;  // bytes of a wave's strip: 16 rows of 64 columns

// Eight sums over the 16 lanes of a row: lane l ends with sums 4 (l % 2) + 2 (l / 2 % 2) and the next.
__device__ __forceinline__ float2 sums_of_row(const float (&s)[8]) {
  const bool odd = threadIdx.x & 1, two = threadIdx.x & 2;
  float a[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) a[e] = (odd ? s[e + 4] : s[e]) + dpp_move<0xB1>(odd ? s[e] : s[e + 4]);  // lane ^ 1
  float t[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    t[e] = (two ? a[e + 2] : a[e]) + dpp_move<0x4E>(two ? a[e] : a[e + 2]);  // lane ^ 2
    t[e] += dpp_move<0x124>(t[e]);  // row_ror 4: the lanes of the row that hold the same sums
    t[e] += dpp_move<0x128>(t[e]);  // row_ror 8
  }
  return float2{t[0], t[1]};
}

template <int ONCE>
__global__ __launch_bounds__(kTwoThreads, 2) void wide_two_term_kernel(const GemmArgs args, const int tiles) {
  __shared__ __align__(1024) char lds[2 * kTwoStage + 4 * kTwoStrip];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w >> 1, wn = w & 1, lc = lane & 15, lq = lane >> 4;
  const uint32_t to = (uint32_t)(uintptr_t)(lds_char*)lds + w * 1024;

  // the tile whose operands are being requested
  struct Tile {
    int problem, m, n;
  };
  auto tile_of = [&](int b) {
    Tile t{0, 0, 0};
    for (int q = 1; q < args.n; ++q)
      if (b >= args.p[q].blk_begin) t.problem = q;
    const GemmProb& g = args.p[t.problem];
    const int local = b - g.blk_begin, row_tiles = (g.M + kTwoRows - 1) / kTwoRows;
    if (g.col_tiles % 8 == 0) {  // the row tiles of a column tile on one XCD, as in wide_scatter_kernel
      t.m = (local >> 3) % row_tiles;
      t.n = (local >> 3) / row_tiles * 8 + (local & 7);
    } else {
      t.m = local % row_tiles;
      t.n = local / row_tiles;
    }
    return t;
  };
  // a wave requests rows 32 q + 8 w .. + 7 of A and 64 q + 16 w .. + 15 of B; rows past the end read as zero
  u32x4 a, b;
  uint32_t va, vb, sa, sb;
  auto aim = [&](const Tile& t) {
    const GemmProb& g = args.p[t.problem];
    const int row0 = t.m * kTwoRows, col0 = t.n * kTwoCols;
    const int a_rows = min(kTwoRows, g.M - row0), b_rows = min(kTwoCols, g.N - col0);
    sa = 4u * g.K;
    sb = 2u * g.ldb;
    a = buffer_of(reinterpret_cast<const char*>(g.A) + (int64_t)row0 * sa, (int64_t)a_rows * sa);
    b = buffer_of(reinterpret_cast<const uint16_t*>(g.B) + (int64_t)col0 * g.ldb, ((int64_t)(b_rows - 1) * g.ldb + g.K) * 2);
    int l = lane;
    asm volatile("" : "+v"(l));  // (what follows from it is not kept in registers over the products)
    va = (8 * w + (l >> 3)) * sa + 16u * ((l & 7) ^ ((4 * w + (l >> 4)) & 7));
    vb = (16 * w + (l >> 2)) * sb + 16u * ((l & 3) ^ ((4 - ((l >> 4) & 3)) & 3));
  };
  auto request = [&](int kt, uint32_t stage) {
    const uint32_t sk = (uint32_t)kt;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      load_to_lds(to + stage + q * 4096, a, va + 32 * q * sa, sk * 128u);
      load_to_lds(to + stage + kTwoA + q * 4096, b, vb + 64 * q * sb, sk * 64u);
    }
  };
  const char* const pb = lds + kTwoA + (128 * wn + lc) * 64 + 16 * (lq ^ ((4 - (lc >> 2)) & 3));
  const char* const head = lds + (64 * wm + lc) * 128 + 16 * (lq ^ (lc >> 1));
  const char* const tail = lds + (64 * wm + lc) * 128 + 16 * ((4 + lq) ^ (lc >> 1));
  char* const strip = lds + 2 * kTwoStage + w * kTwoStrip;

  Tile now = tile_of(blockIdx.x);
  aim(now);
  request(0, 0);
  request(1, kTwoStage);
  wait_loads<0>();
  uint32_t stage = 0;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const GemmProb& g = args.p[now.problem];
    if (tile == g.blk_begin && tid == 0 && g.sync) *g.sync = 0u;
    const bool more = tile + (int)gridDim.x < tiles;
    const Tile next = tile_of(more ? tile + (int)gridDim.x : tile);
    const int nk = g.K / 32;  // two or more
    f32x4 acc[4][8];
#pragma unroll
    for (int f = 0; f < 32; ++f) acc[f >> 3][f & 7] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int t = 0; t < nk; ++t) {
      if (t >= 2) {  // all but the next k-tile's (the first two have arrived)
        if (t + 1 < nk || more) wait_loads<8>();
        else wait_loads<0>();
      }
      barrier();
      bf16x8 ah[4], al[4], bb[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        al[i] = *reinterpret_cast<const bf16x8*>(tail + stage + i * 2048);
        ah[i] = *reinterpret_cast<const bf16x8*>(head + stage + i * 2048);
      }
#pragma unroll
      for (int n = 0; n < 8; ++n) bb[n] = *reinterpret_cast<const bf16x8*>(pb + stage + n * 1024);
      if (t + 2 == nk && more) aim(next);
      wait_lds();
      barrier();
      if (t + 2 < nk || more) request(t + 2 < nk ? t + 2 : t + 2 - nk, stage);
      stage = kTwoStage - stage;
#pragma unroll
      for (int n = 0; n < 8; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bb[n], al[i], acc[i][n], 0, 0, 0);
#pragma unroll
      for (int n = 0; n < 8; ++n)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bb[n], ah[i], acc[i][n], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }

    // A lane has four neighbouring columns of row lc of a fragment; 16 rows of half the wave tile go through its strip (piece c
    // of a row at c ^ row), so that what touches memory is 256 bytes of a row: row 4 q + lane / 16, columns 4 (lane % 16) ..
    const int64_t ldd = g.ldd;
    int el = lane;
    asm volatile("" : "+v"(el));  // (as above)
    const int er = el >> 4, ec = 4 * (el & 15);
    const int row0 = now.m * kTwoRows + 64 * wm, col0 = now.n * kTwoCols + 128 * wn;
    auto put = [&](int s) {
#pragma unroll
      for (int n = 0; n < 4; ++n) *reinterpret_cast<f32x4*>(strip + (el & 15) * 256 + 16 * ((4 * n + er) ^ (el & 15))) = acc[s >> 1][4 * (s & 1) + n];
      __builtin_amdgcn_sched_barrier(0);
    };
    // (private to the wave, whose LDS operations execute in order: only the compiler has to be held)
    auto get = [&](f32x4 (&val)[4]) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int q = 0; q < 4; ++q) val[q] = *reinterpret_cast<const f32x4*>(strip + (4 * q + er) * 256 + 16 * ((el & 15) ^ (4 * q + er)));
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    if (g.epi != EPI_RESIDUAL) {
      wait_loads<0>();  // the next tile's first k-tiles have arrived: no wait counts the stores that follow for them
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        put(s);
        f32x4 val[4];
        get(val);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int row = row0 + 16 * (s >> 1) + 4 * q + er, col = col0 + 64 * (s & 1) + ec;
          if (row < g.M && col < g.N) store_row<ONCE != 0>(reinterpret_cast<float*>(g.D) + (int64_t)row * ldd + col, float4{val[q][0], val[q][1], val[q][2], val[q][3]});
        }
      }
    } else {
      auto residual = [&](auto element) {  // of x
        using T = decltype(element);
        decltype(load_row<false>(static_cast<const T*>(nullptr))) x[3][4];  // x of three half strips, as stored
        auto request_x = [&](int s) {  // (rows and columns past the end repeat the last)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            x[s % 3][q] = load_row<ONCE == 2>(reinterpret_cast<const T*>(g.X) + (int64_t)min(row0 + 16 * (s >> 1) + 4 * q + er, g.M - 1) * ldd +
                                              min(col0 + 64 * (s & 1) + ec, g.N - 4));
        };
        request_x(0);
        request_x(1);
        wait_loads<0>();  // (as above)
        float sums[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const int half = s & 1;
          put(s);
          if (s < 6) request_x(s + 2);
          f32x4 val[4];
          get(val);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int row = row0 + 16 * (s >> 1) + 4 * q + er, col = col0 + 64 * half + ec;
            const bool live = row < g.M && col < g.N;
            const float4 v = widen_row(x[s % 3][q]);
            const float4 r = float4{v.x - val[q][0], v.y - val[q][1], v.z - val[q][2], v.w - val[q][3]};
            if (live) store_row<ONCE != 0>(reinterpret_cast<float*>(g.D) + (int64_t)row * ldd + col, r);
            const float sr = live ? fmaf(r.x, r.x, fmaf(r.y, r.y, fmaf(r.z, r.z, r.w * r.w))) : 0.f;
            const float sx = live ? fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, v.w * v.w))) : 0.f;
            sums[2 * q] = half ? sums[2 * q] + sr : sr;
            sums[2 * q + 1] = half ? sums[2 * q + 1] + sx : sx;
          }
          if (half) {
            const float2 t = sums_of_row(sums);
            const int row = row0 + 16 * (s >> 1) + 4 * (2 * (el & 1) + ((el >> 1) & 1)) + er;
            if ((el & 15) < 4 && row < g.M && col0 < g.N) reinterpret_cast<float2*>(g.part_n)[(int64_t)(2 * now.n + wn) * g.M + row] = t;
          }
        }
      };
      if (g.xdtype == GSI_F32) residual(0.f);
      else residual(uint16_t{0});
    }
    now = next;
  }
}

// The image term of a map by itself: the products of wide_two_term_kernel in the same order, so the same bits, from c as the caller has it,
// in fp32.  A lane splits what it reads from LDS; laid out in two terms by a launch of its own (split_rows) first, it took 6 us of
// calls of 12 to 30.  Tiles of 64 x 256, a workgroup of four waves (2 x 2, 32 x 128 each), k-tiles of 32 columns, one barrier each: where every
// tile has a place at once two workgroups a unit with three k-tiles in LDS, else three with two.  A row of A is 128 bytes, piece c at
// c ^ (row / 2 % 8), one of B 64, as above.  Bound by the chain of a tile (few tiles), by LDS and the products (many).  The workgroups behind the
// tiles lay out fired rows for the W term, which is a launch less, too.
// us a call, none fired, on gemm_nt / with split_rows / so: 1024 x 1024 at rank 64, 140 tokens 13.4 / 19.0 / 12.6; 4096 x 512, rank 512, 1000
// 26.1 / 32.2 / 22.0; 11008 x 512, rank 512, 700 36.7 / 41.6 / 32.4; 16384 x 512, rank 64, 1200 31.2 / 29.2 / 25.9; 28672 x 512, rank 512, 330
// 38.0 / 45.3 / 40.4, 600 57.9 / 61.3 / 57.4.  Tiles of 128 rows, or waves of 64 x 64 (which split every row of A twice as often), 3 to 15 % more.
constexpr int kImageRows = 64;
template <int S>
__global__ __launch_bounds__(kTwoThreads, S == 2 ? 3 : 2) void wide_image_kernel(const GemmProb g, const int tiles, const RoundTask round) {
  constexpr int kA = kImageRows * 128, kStage = kA + kTwoCols * 64;
  __shared__ __align__(1024) char lds[S * kStage];
  const int tid = threadIdx.x, lane = tid & 63;
  if ((int)blockIdx.x >= tiles) {
    round_part<0>(round, (int64_t)(blockIdx.x - tiles) * kTwoThreads + tid, (int64_t)(gridDim.x - tiles) * kTwoThreads);
    return;
  }
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w >> 1, wn = w & 1, lc = lane & 15, lq = lane >> 4;
  const int row_tiles = (g.M + kImageRows - 1) / kImageRows;
  int tile_m = blockIdx.x % row_tiles, tile_n = blockIdx.x / row_tiles;
  if (g.col_tiles % 8 == 0) {  // the row tiles of a column tile on one XCD
    tile_m = (blockIdx.x >> 3) % row_tiles;
    tile_n = (blockIdx.x >> 3) / row_tiles * 8 + (blockIdx.x & 7);
  }
  const int row0 = tile_m * kImageRows, col0 = tile_n * kTwoCols, nk = g.K / 32;
  const int64_t lda = g.lda, ldb = g.ldb;
  // (rows past the end: zeros)
  const u32x4 a = buffer_of(reinterpret_cast<const float*>(g.A) + row0 * lda, ((min(kImageRows, g.M - row0) - 1) * lda + g.K) * 4);
  const u32x4 b = buffer_of(reinterpret_cast<const uint16_t*>(g.B) + col0 * ldb, ((min(kTwoCols, g.N - col0) - 1) * ldb + g.K) * 2);
  const uint32_t sa = 4u * g.lda, sb = 2u * g.ldb;
  const uint32_t va = (8 * w + (lane >> 3)) * sa + 16u * ((lane & 7) ^ ((4 * w + (lane >> 4)) & 7));
  const uint32_t vb = (16 * w + (lane >> 2)) * sb + 16u * ((lane & 3) ^ ((4 - ((lane >> 4) & 3)) & 3));
  const uint32_t to = (uint32_t)(uintptr_t)(lds_char*)lds + w * 1024;
  auto request = [&](int kt, uint32_t stage) {  // (past the last k-tile that again, never read)
    const uint32_t k = (uint32_t)min(kt, nk - 1);
#pragma unroll
    for (int q = 0; q < 2; ++q) load_to_lds(to + stage + q * 4096, a, va + 32 * q * sa, k * 128u);
#pragma unroll
    for (int q = 0; q < 4; ++q) load_to_lds(to + stage + kA + q * 4096, b, vb + 64 * q * sb, k * 64u);
  };
  const char* const pa = lds + (32 * wm + lc) * 128;
  const int p0 = 16 * ((2 * lq) ^ (lc >> 1)), p1 = 16 * ((2 * lq + 1) ^ (lc >> 1));
  const char* const pb = lds + kA + (128 * wn + lc) * 64 + 16 * (lq ^ ((4 - (lc >> 2)) & 3));
  f32x4 acc[2][8];
#pragma unroll
  for (int f = 0; f < 16; ++f) acc[f >> 3][f & 7] = f32x4{0.f, 0.f, 0.f, 0.f};
  request(0, 0);
  if constexpr (S == 3) request(1, kStage);
  uint32_t stage = 0, free = (S - 1) * kStage;
  for (int t = 0; t < nk; ++t) {
    wait_loads<(S - 2) * 6>();  // this k-tile has arrived
    wait_lds();                 // and the one before is in registers
    barrier();                  // ... in every wave
    f32x4 av[2][2];
    bf16x8 bb[8];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      av[i][0] = *reinterpret_cast<const f32x4*>(pa + stage + i * 2048 + p0);
      av[i][1] = *reinterpret_cast<const f32x4*>(pa + stage + i * 2048 + p1);
    }
#pragma unroll
    for (int n = 0; n < 8; ++n) bb[n] = *reinterpret_cast<const bf16x8*>(pb + stage + n * 1024);
    request(t + S - 1, free);
    free = stage;
    stage = stage == (S - 1) * kStage ? 0 : stage + kStage;
    bf16x8 ah[2], al[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x = av[i][e >> 2][e & 3];
        const __bf16 h = (__bf16)x;
        ah[i][e] = h;
        al[i][e] = (__bf16)(x - __uint_as_float((uint32_t)__builtin_bit_cast(uint16_t, h) << 16));
      }
#pragma unroll
    for (int n = 0; n < 8; ++n)
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bb[n], al[i], acc[i][n], 0, 0, 0);
#pragma unroll
    for (int n = 0; n < 8; ++n)
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bb[n], ah[i], acc[i][n], 0, 0, 0);
  }
  wait_loads<0>();
  wait_lds();
  barrier();  // every k-tile has been read: the strips of the epilogue (as in wide_two_term_kernel) lie over them
  char* const strip = lds + w * kTwoStrip;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
#pragma unroll
    for (int n = 0; n < 4; ++n) *reinterpret_cast<f32x4*>(strip + lc * 256 + 16 * ((4 * n + lq) ^ lc)) = acc[s >> 1][4 * (s & 1) + n];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 4 * q + lq, row = row0 + 32 * wm + 16 * (s >> 1) + r, col = col0 + 128 * wn + 64 * (s & 1) + 4 * lc;
      const f32x4 v = *reinterpret_cast<const f32x4*>(strip + r * 256 + 16 * (lc ^ r));
      if (row < g.M && col < g.N) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.D) + (int64_t)row * g.ldd + col) = v;  // N is a multiple of 4
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Ht[row] = the heads of 32 columns of a row of C, their tails, the next 32 columns ...
__global__ __launch_bounds__(256) void split_rows(const SplitArgs args) {
  const SplitTask& t = args.t[blockIdx.y];
  const int k4 = t.k >> 2;
  const int64_t total = (int64_t)t.rows * k4;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = e / k4;
    store_two_terms(t.Ht, row, t.k, 4 * (int)(e - row * k4), *reinterpret_cast<const float4*>(t.C + 4 * e));
  }
}

}  // namespace

hipError_t wide_split_rows(const SplitTask* tasks, int n, hipStream_t s) {
  for (int i = 0; i < n;) {
    SplitArgs a;
    int c = 0;
    int64_t most = 0;
    for (; i < n && c < kMaxSplitTasks; ++i, ++c) {
      a.t[c] = tasks[i];
      most = std::max(most, ceil_div((int64_t)tasks[i].rows * (tasks[i].k / 4), 256));
    }
    split_rows<<<dim3((unsigned)std::min<int64_t>(most, 2048), (unsigned)c), 256, 0, s>>>(a);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t wide_two_term(const GemmProb* probs, int n, int once, hipStream_t s) {
  for (int i = 0; i < n;) {
    GemmArgs g;
    g.n = 0;
    int64_t blocks = 0;
    for (; i < n && g.n < kMaxProbs; ++i) {
      GemmProb& p = g.p[g.n++];
      p = probs[i];
      p.col_tiles = (int)ceil_div(p.N, kTwoCols);
      p.blk_begin = (int)blocks;
      blocks += p.col_tiles * ceil_div(p.M, kTwoRows);
    }
    if (blocks >= (1ll << 31) - kTwoGroups) return hipErrorInvalidValue;
    const unsigned groups = (unsigned)std::min<int64_t>(blocks, kTwoGroups);
    if (once == 0) wide_two_term_kernel<0><<<groups, kTwoThreads, 0, s>>>(g, (int)blocks);
    else if (once == 1) wide_two_term_kernel<1><<<groups, kTwoThreads, 0, s>>>(g, (int)blocks);
    else wide_two_term_kernel<2><<<groups, kTwoThreads, 0, s>>>(g, (int)blocks);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

// workgroups that round the fired rows of a task: what a quarter of the tokens keeps busy
static int64_t round_groups(const RoundTask& t) { return ceil_div(wide_rows_expected(t.rows) * (t.d / 8), 256); }

hipError_t wide_image(const GemmProb& prob, const RoundTask* round, hipStream_t s) {
  GemmProb g = prob;
  g.col_tiles = (int)ceil_div(g.N, kTwoCols);
  const int64_t tiles = g.col_tiles * ceil_div(g.M, kImageRows), rest = round ? std::min<int64_t>(round_groups(*round), 1024) : 0;
  if (tiles >= (1ll << 31) - rest) return hipErrorInvalidValue;
  const RoundTask r = round ? *round : RoundTask{};
  if (tiles <= 2 * kUnits) wide_image_kernel<3><<<(unsigned)(tiles + rest), kTwoThreads, 0, s>>>(g, (int)tiles, r);
  else wide_image_kernel<2><<<(unsigned)(tiles + rest), kTwoThreads, 0, s>>>(g, (int)tiles, r);
  return hipGetLastError();
}

hipError_t wide_round_rows(const RoundTask* tasks, int n, bool once, hipStream_t s) {
  for (int i = 0; i < n;) {
    RoundArgs a;
    int c = 0;
    int64_t most = 0;
    for (; i < n && c < kMaxRoundTasks; ++i, ++c) {
      a.t[c] = tasks[i];
      most = std::max(most, round_groups(tasks[i]));
    }
    const dim3 grid((unsigned)std::min<int64_t>(most, 2048), (unsigned)c);
    if (once) round_rows<1><<<grid, 256, 0, s>>>(a);
    else round_rows<0><<<grid, 256, 0, s>>>(a);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t wide_scatter(const GemmProb* probs, int n, bool once, hipStream_t s) {
  for (int i = 0; i < n;) {
    GemmArgs g;
    g.n = 0;
    for (; i < n && g.n < kMaxProbs; ++i) g.p[g.n++] = probs[i];
    int64_t blocks = 0;
    for (int q = 0; q < g.n; ++q) {
      GemmProb& p = g.p[q];
      p.tile_rows = kWideTile;
      p.splits = p.max_splits;
      p.min_parts = std::min(p.splits, (int)ceil_div(p.K, BK * kMaxDepth));
      p.col_tiles = (int)ceil_div(p.N, kWideTile);
      // the most pieces that any count makes (parts_for)
      const int64_t want = p.row_tiles ? (int64_t)p.splits * p.row_tiles : 0, tiles = ceil_div(p.M, kWideTile);
      blocks += p.col_tiles * (p.row_tiles ? std::max({want, (int64_t)kUnits / p.col_tiles, tiles * p.min_parts}) : tiles * p.splits);
    }
    blocks = std::max<int64_t>(blocks, kUnits);  // (lower tiles, where the pieces are fewer)
    if (blocks >= (1ll << 31)) return hipErrorInvalidValue;
    std::stable_sort(g.p, g.p + g.n, [](const GemmProb& x, const GemmProb& y) {  // the longest parts first, as in mfma_gemm_nt
      return (int64_t)x.K * y.splits > (int64_t)y.K * x.splits;
    });
    if (once) wide_scatter_kernel<1><<<(unsigned)blocks, kWideThreads, 0, s>>>(g);
    else wide_scatter_kernel<0><<<(unsigned)blocks, kWideThreads, 0, s>>>(g);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    if (hipError_t e = mfma_finish_scatter(g, once, s); e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace gsi
