// Products with a stored basis as the right factor: D = A U, A[M, K] bf16 row-major, U[K, N] bf16 row-major, the image M = W U of a
// block's preparation and the coefficients C = X U of prefill-sized bf16 activations.
//
// Both operands go from memory to LDS without registers (load_to_lds) as they are stored; a lane's eight values of a column of U, which
// lie in eight rows, are read with the transposing reads of LDS (two of four rows by sixteen columns).  A workgroup of eight waves has
// TM x 256 of D; a k-tile is TM rows of 64 columns of A (128 bytes a row, piece c at c ^ row / 2 % 8) and 64 rows of 256 columns of U
// (512 bytes a row, the pair of pieces of a fragment at pair ^ (row % 4 + 4 (row / 8 % 2)): the rows that a read takes lie in distinct
// banks).  Three or four k-tiles in LDS; four of the waves are half a k-tile behind the other four, so that one wave of a SIMD reads LDS
// while the other multiplies (as in wide_loop, gsi_wide.hip).
#include <algorithm>

#include "gsi_mfma_device.h"

namespace gsi {
namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kBasisThreads = 512, kBasisCols = 256;

template <int TM, int EPI>
__global__ __launch_bounds__(kBasisThreads, 2) void basis_product(const GemmArgs args) {
  constexpr int WM = TM / 64, WN = 8 / WM, NF = kBasisCols / WN / 16;  // waves, and fragments of 16 columns of a wave (of 64 rows)
  constexpr int kA = TM * 128, kStage = kA + 64 * kBasisCols * 2, S = TM == 64 ? 4 : 3, kLoads = TM / 64 + 4;
  __shared__ __align__(1024) char lds[S * kStage];
  int pi = 0;
  for (int q = 1; q < args.n; ++q)
    if ((int)blockIdx.x >= args.p[q].blk_begin) pi = q;
  const GemmProb& g = args.p[pi];
  // the parts of a tile side by side: with eight and more, an XCD's L2 holds the rows of U that its parts take
  const int local = blockIdx.x - g.blk_begin, split = local % g.splits, tile = local / g.splits;
  const int row0 = tile / g.col_tiles * TM, col0 = tile % g.col_tiles * kBasisCols;
  const int lane = threadIdx.x & 63, lc = lane & 15, lq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = w / WN, wn = w % WN;
  const int nk = g.K / BK, kt0 = (int)((int64_t)nk * split / g.splits), kt1 = (int)((int64_t)nk * (split + 1) / g.splits);
  // (rows past the end of A: zeros, sums that are not stored)
  const u32x4 a = buffer_of(reinterpret_cast<const uint16_t*>(g.A) + (int64_t)row0 * g.lda, ((int64_t)(min(TM, g.M - row0) - 1) * g.lda + g.K) * 2);
  const u32x4 b = buffer_of(reinterpret_cast<const uint16_t*>(g.B) + col0, ((int64_t)g.K * g.ldb - col0) * 2);
  const int ar = 8 * w + (lane >> 3), br = 2 * w + (lane >> 5);
  const uint32_t sa = 2u * g.lda, sb = 2u * g.ldb;
  const uint32_t va = ar * sa + 16u * ((lane & 7) ^ ((ar >> 1) & 7));
  const uint32_t vb = br * sb + 16u * ((lane & 31) ^ (2 * ((br & 3) + 4 * ((br >> 3) & 1))));
  // columns past the end of U: zeros, not the next row's (us, images, asked for / not: 16384 x 4096 x 64 43.5 / 39.0, 8192 x 8192 x 320 83.2 / 70.9)
  const bool has = (int)((vb - br * sb) / 2) < g.N - col0;
  const uint32_t to = (uint32_t)(uintptr_t)(lds_char*)lds + w * 1024;
  auto request = [&](int kt, uint32_t stage) {  // past the range: nothing is read, and zeros written that are never read
    const bool in = kt < kt1;
    const uint32_t k = in ? kt : kt0;
#pragma unroll
    for (int q = 0; q < TM / 64; ++q) load_to_lds(to + stage + q * 8192, a, in ? va + 64 * q * sa : 0xfffffff0u, k * 128u);
#pragma unroll
    for (int q = 0; q < 4; ++q) load_to_lds(to + stage + kA + q * 8192, b, in && has ? vb + 16 * q * sb : 0xfffffff0u, k * 64u * sb);
  };
  const char* const pa = lds + (64 * wm + lc) * 128;
  const int p0 = 16 * (lq ^ (lc >> 1)), p1 = 16 * ((4 + lq) ^ (lc >> 1));
  uint32_t pb[NF];  // rows 8 lq + lc / 4, columns 4 (lc % 4) .. of fragment n
#pragma unroll
  for (int n = 0; n < NF; ++n)
    pb[n] = kA + (8 * lq + (lc >> 2)) * 512 + 32 * ((NF * wn + n) ^ ((lc >> 2) + 4 * (lq & 1))) + 8 * (lc & 3);
  f32x4 acc[4][NF];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int n = 0; n < NF; ++n) acc[i][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int q = 0; q < S - 1; ++q) request(kt0 + q, q * kStage);
  wait_loads<(S - 2) * kLoads>();
  barrier();
  if (w >= 4) barrier();  // half a k-tile behind
  uint32_t stage = 0, last = (S - 1) * kStage;  // of this k-tile, and of the one before
  for (int t = kt0; t < kt1; ++t) {
    bf16x8 ra[4][2], rb[NF][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ra[i][0] = *reinterpret_cast<const bf16x8*>(pa + stage + i * 2048 + p0);
      ra[i][1] = *reinterpret_cast<const bf16x8*>(pa + stage + i * 2048 + p1);
    }
#pragma unroll
    for (int n = 0; n < NF; ++n)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lds + stage + pb[n] + k * 16384));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lds + stage + pb[n] + k * 16384 + 2048));
        rb[n][k] = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    request(t + S - 1, last);
    wait_loads<(S - 2) * kLoads>();  // the next k-tile has arrived
    wait_lds();
    barrier();
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int n = 0; n < NF; ++n) acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rb[n][k], ra[i][k], acc[i][n], 0, 0, 0);
    barrier();
    last = stage;
    stage = stage == (S - 1) * kStage ? 0 : stage + kStage;
  }
  if (w < 4) barrier();
  wait_loads<0>();

  // a lane has four neighbouring columns of row lc of a fragment
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = row0 + 64 * wm + 16 * i + lc;
    if (row >= g.M) continue;
#pragma unroll
    for (int n = 0; n < NF; ++n) {
      const int col = col0 + 16 * (NF * wn + n) + 4 * lq;
      if (col >= g.N) continue;  // N is a multiple of 4
      const float4 v = float4{acc[i][n][0], acc[i][n][1], acc[i][n][2], acc[i][n][3]};
      if (g.splits > 1) {
        store_row<false>(g.part + ((int64_t)split * g.M + row) * g.N + col, v);
      } else if constexpr (EPI == EPI_STORE_BF16) {
        *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(g.D) + (int64_t)row * g.ldd + col) = u32x2{
            (uint32_t)f32_to_bf16_bits(v.x) | ((uint32_t)f32_to_bf16_bits(v.y) << 16), (uint32_t)f32_to_bf16_bits(v.z) | ((uint32_t)f32_to_bf16_bits(v.w) << 16)};
      } else {
        store_row<false>(reinterpret_cast<float*>(g.D) + (int64_t)row * g.ldd + col, v);
        if (g.Ht) store_two_terms(g.Ht, row, g.N, col, v);
      }
    }
  }
}

template <int EPI>
hipError_t launch(GemmArgs& g, int tm, int once, hipStream_t s) {
  int64_t blocks = 0;
  bool split = false;
  for (int i = 0; i < g.n; ++i) {
    GemmProb& p = g.p[i];
    p.col_tiles = (int)ceil_div(p.N, kBasisCols);
    p.splits = p.part ? p.max_splits : 1;
    p.row_tiles = 0;
    p.blk_begin = (int)blocks;
    blocks += ceil_div(p.M, tm) * p.col_tiles * p.splits;
    split |= p.splits > 1;
  }
  if (blocks >= (1ll << 31)) return hipErrorInvalidValue;
  if (tm == 64) basis_product<64, EPI><<<(unsigned)blocks, kBasisThreads, 0, s>>>(g);
  else basis_product<128, EPI><<<(unsigned)blocks, kBasisThreads, 0, s>>>(g);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  return split ? mfma_finish_basis(g, EPI, once != 0, s) : hipSuccess;
}

}  // namespace

// Images are alone in their launch: as many parts as the chip takes, of eight k-tiles at least.  us, doubled while they fit / so: 2560 x 10240
// x 256 36.9 / 30.7, 6144 x 6144 x 256 38.8 / 36.3, 3072 x 3072 x 256 22.3 / 19.4.
int basis_splits(int64_t M, int64_t N, int64_t K, int tm) {
  const int64_t tiles = ceil_div(M, tm) * ceil_div(N, kBasisCols), nk = ceil_div(K, BK);
  return (int)std::max<int64_t>(1, std::min<int64_t>({32, kUnits / tiles, nk / 8}));
}

// Coefficients share their launch with those of other inputs: parts of 4096 rows of the basis where a product has fewer tiles than the
// chip units; those of few tiles as many parts as half the chip takes, of 512 rows at least, or 256 where there are at most four
// tiles.  us a call, none fired, cut by doubling to half the chip or just beyond, 256 rows at least / so: a block of 2048 / 8192 at
// rank 256, 777 tokens 100 / 90, at rank 512, 500 tokens 100 / 90; 2560 / 10240 at rank 256, 1024 tokens 122 / 114; 4096 / 16384, 777
// tokens 150 / 138; the pair 2048 / 8192 at rank 256, 777 tokens 74 / 68; 4096 / 16384, 1024 tokens 105 / 100.  From an eighth of the units on they
// are left: beside others they fill the chip.  us a call, none fired, left from a sixteenth on / from an eighth: a block of 4096 / 16384 at
// rank 512, 1664 tokens 361 / 365, 1920 395 / 407; the pair, 1024 tokens 202 / 178, 1664 262 / 259, 1920 286 / 283; one input of 4096, 1664 tokens 101 / 65.
// From an eighth / from a quarter: the block, 2048 tokens 414 / 435, 2304 453 / 480; the pair, 2048 307 / 308.
int basis_coeff_splits(int64_t M, int64_t N, int64_t K) {
  const int64_t tiles = ceil_div(M, 128) * ceil_div(N, kBasisCols), nk = ceil_div(K, BK);
  int s = tiles < kUnits ? (int)std::min<int64_t>(ceil_div(nk, kMaxDepth), 32) : 1;
  if (tiles >= kUnits / 8) return s;
  return (int)std::min<int64_t>(std::max<int64_t>(s, std::min<int64_t>(kUnits / 2 / tiles, nk / (tiles <= kUnits / 64 ? 4 : 8))), 32);
}

hipError_t basis_products(const GemmProb* probs, int n, int epi, int tm, int once, hipStream_t s) {
  for (int i = 0; i < n;) {
    GemmArgs g;
    g.n = 0;
    for (; i < n && g.n < kMaxProbs; ++i) g.p[g.n++] = probs[i];
    std::stable_sort(g.p, g.p + g.n, [](const GemmProb& x, const GemmProb& y) {  // the longest parts first, as in mfma_gemm_nt
      return (int64_t)x.K * y.max_splits > (int64_t)y.K * x.max_splits;
    });
    // Coefficients: tiles of 64 rows where those of 128 leave half the chip idle.  (The parts are those of the product, whatever its launch,
    // and a tile has the same sums in the same order.)  A projection by itself, us, tiles of 128 / so: 4096 at rank 384, 2048 tokens 98 / 88, rank
    // 512, 2304 111 / 99; 2048 at rank 384, 2048 tokens 69 / 61; 1024 at rank 512, 2048 58 / 51; 768 at rank 320, 600 48 / 41, rank 64 33 / 29.
    int64_t blocks = 0;
    for (int q = 0; q < g.n; ++q) blocks += ceil_div(g.p[q].M, 128) * ceil_div(g.p[q].N, kBasisCols) * (g.p[q].part ? g.p[q].max_splits : 1);
    const int rows = tm ? tm : 2 * blocks <= kUnits ? 64 : 128;
    if (hipError_t e = epi == EPI_STORE_BF16 ? launch<EPI_STORE_BF16>(g, rows, once, s) : launch<EPI_STORE_F32>(g, rows, once, s); e != hipSuccess)
      return e;
  }
  return hipSuccess;
}

}  // namespace gsi
