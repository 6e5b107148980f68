// Dense contractions of libgsi on the matrix cores (gfx950 MFMA, bf16 inputs, fp32 accumulation):
// the one-time image build M = W U (Eq. (exact), Section 4 "Storage") and the prefill-sized batched
// path (hundreds of tokens per call), where the work really is a GEMM:
//     C = X U            R = X - C U^T  (+ per-token partial norms)          Algorithm 1, lines 1-3
//     Y = C M^T          Y[fired] += R[fired] W^T                            Eq. (exact)
//
// Where the call's workspace is what the query names (kWsFull), images and the coefficients of bf16 activations run on the products of
// gsi_basis.hip, residual rows, image terms and W r of many tokens on those of gsi_wide.hip; here is what these do not take.
//
// One kernel, D = A B^T with both operands K-contiguous ("NT"): A[M,K], B[N,K] row-major.  A is bf16,
// or fp32 split on the fly into a bf16 head and a bf16 tail (two MFMA passes) so that an fp32 operand
// on the main term is not rounded to 8 bits (the bf16 image already uses most of the 2e-3 budget).
//
// Workgroup tile 256 x 256 x 64 (or 128 x 256 x 64), eight waves 4 x 2 (2 x 4; two per SIMD, so that one wave's MFMAs
// cover the other's LDS reads and staging), each wave 64 x 128 (64 x 64) as v_mfma_f32_32x32x16_bf16 fragments.
// Both operand tiles are staged in LDS as bf16 (row stride padded to 144 bytes: conflict-free 128-bit
// reads); an fp32 A operand is converted on the way in.  Global loads are whole 128-byte row segments per
// eight lanes.  LDS holds two k-tiles: tile t is multiplied while tile t + 1 is written, a unit per MFMA step,
// from registers that are asked for tile t + 2 at once; one barrier per tile.  A k-tile is 64 columns deep, or
// 32 for the head + tail form (two tiles of A per stage, two MFMA passes per step: as many MFMAs between
// barriers).  Within a k-tile the lane half l/32 takes one half of the columns, eight per MFMA step: any order
// of the contraction index is as good as another as long as both operands agree.
// What bounds the loop is LDS, not the matrix cores: a k-tile is 2048 MFMA cycles per SIMD, and its LDS
// traffic (192 KB of operand reads at 128 bytes a cycle, 64 KB of staging writes at about 75) is 2400.
// (Built and measured beside it: 256 x 256 tiles by four waves of 128 x 128, accumulators in AGPRs, memory to LDS without
// registers: 1012 TFLOP/s against 1004 on 2048 x 16384 x 4096, 899 against 998 at 16384 columns, and no second workgroup
// to cover an epilogue; with eight waves in two groups half a step apart it pays, gsi_wide.hip; 128 x 256 x 32 tiles by four waves, two
// workgroups per unit: 795.)
// A launch takes the products of all inputs, or of all maps, of a call (GemmProb): one product of a block is 64 to 512
// tiles, one or two rounds of the 256 compute units with a ramp and a tail of its own.  The row tile is chosen
// for the whole launch (plan_rows).  A block's prefill, 2048 tokens at rank 512: 36 launches 1007 us, 7 launches
// 730 us; the pair 4096 / 16384, 333 tokens at rank 256: 14 launches 438 us, 7 launches 162 us.
// Problems with few output tiles split the contraction; the partial sums go to the workspace
// and a second kernel adds them in split order and applies the epilogue.
// The residual and image products are short (the rank) with long epilogues (every output row of a block: 0.5 GB), so they
// run on tiles of 128 rows, two workgroups per unit: one's epilogue beside the other's products.  (One per unit where an fp32
// operand meets a basis as stored, the coefficients of fp32 tokens.)
// A right operand that is N-contiguous in memory (U as the factor of W U and X U) is transposed on its way to LDS: a thread
// has four columns of BKT / 8 rows, packs two rows into a word and writes four columns.  Where that costs more than it saves
// (many row tiles of bf16 activations: mfma_project; large images: gsi_build_image), or its rows are no whole 8-byte pieces,
// it is transposed once into the workspace.  The six images of a block (4096 / 16384, rank 256): a launch of 5 us each less.
#include <algorithm>

#include "gsi_device.h"
#include "gsi_mfma_device.h"

namespace gsi {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int BN = 256;
constexpr int WTM = 64;                         // rows of a wave tile
constexpr int kThreads = 512;
constexpr int kAF = WTM / 32;                   // A fragments per wave

// AM: how the A operand is stored and fed: 0 bf16; 1 fp32, split into bf16 head + tail (two LDS tiles, two
// MFMA passes); 2 fp32, rounded once to bf16.
// Geometry of a staged k-tile by mode.  The head + tail form keeps two tiles of A per stage, so its k-tile is 32
// columns deep (two MFMA steps of two passes each: as many MFMAs between barriers as the 64-deep tile of the
// other modes) and two stages still fit in LDS.
// TM: rows of the workgroup tile, 256, 128 or 64 (eight waves 4 x 2, 2 x 4 or 1 x 8, each 64 x 128, 64 x 64 or 64 x 32).
// BT: the right operand is stored with the contraction along its rows (the basis, U[l][j]): it is transposed on its way to LDS.
template <int AM, int TM, bool BT>
struct Geo {
  static constexpr int BKT = AM == 1 ? 32 : 64;          // columns of a k-tile
  static constexpr int LD = BKT + 8;                     // padded LDS row stride, bf16 elements (80 or 144 bytes:
                                                         // conflict-free 128-bit reads either way)
  static constexpr int KS = BKT / 16;                    // MFMA steps per k-tile
  static constexpr int CPR = BKT / 8;                    // staging units (8 elements) per tile row
  static constexpr int RPP = kThreads / CPR;             // tile rows covered by one unit index of all threads
  static constexpr int NU = BN / RPP;                    // units of B per thread and k-tile
  static constexpr int NA = TM / RPP;                    // ... and of A
  static constexpr int NP = AM == 1 ? 2 : 1;             // LDS tiles of A per stage
  static constexpr int kATile = TM * LD;                 // elements of one LDS tile of A
  static constexpr int kBPad = BT ? 3 * 32 : 0;          // see b_row
  static constexpr int kStage = (NP * TM + BN) * LD + kBPad;  // elements of one stage
  static constexpr int WN = TM == 256 ? 2 : TM == 128 ? 4 : 8;  // waves side by side
  static constexpr int WTN = BN / WN;                    // columns of a wave tile
  static constexpr int kBF = WTN / 32;                   // B fragments per wave
  static_assert(NU == KS, "one staging unit of B per MFMA step");
};

template <int AM, int TM, bool BT>
struct Stage {
  u32x4 a[Geo<AM, TM, BT>::NA][AM ? 2 : 1];
  u32x4 b[Geo<AM, TM, BT>::NU];  // BT: rows 2 u and 2 u + 1 of the thread's, four columns each
};

// LDS row of column n of the right operand's tile.  Transposed, a thread has four neighbouring columns: those of one
// remainder modulo four are kept together, so that neighbouring threads write neighbouring rows, and the four groups lie 64
// bytes further apart than their rows, so that sixteen neighbouring columns are read from distinct banks.
template <int AM, int TM, bool BT>
__device__ __forceinline__ int b_row(int n) {
  using G = Geo<AM, TM, BT>;
  return BT ? (n & 3) * (BN / 4 * G::LD + 32) + (n >> 2) * G::LD : n * G::LD;
}

// 8 fp32 -> 8 bf16 (RNE), and the bf16 of what is left
__device__ __forceinline__ u32x4 round8(const u32x4& x0, const u32x4& x1, u32x4* tail) {
  const float x[8] = {__uint_as_float(x0[0]), __uint_as_float(x0[1]), __uint_as_float(x0[2]), __uint_as_float(x0[3]),
                      __uint_as_float(x1[0]), __uint_as_float(x1[1]), __uint_as_float(x1[2]), __uint_as_float(x1[3])};
  uint16_t h[8], l[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const __bf16 hb = (__bf16)x[e];
    h[e] = __builtin_bit_cast(uint16_t, hb);
    const __bf16 lb = (__bf16)(x[e] - __uint_as_float((uint32_t)h[e] << 16));
    l[e] = __builtin_bit_cast(uint16_t, lb);
  }
  if (tail)
    *tail = u32x4{(uint32_t)l[0] | ((uint32_t)l[1] << 16), (uint32_t)l[2] | ((uint32_t)l[3] << 16),
                  (uint32_t)l[4] | ((uint32_t)l[5] << 16), (uint32_t)l[6] | ((uint32_t)l[7] << 16)};
  return u32x4{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16),
               (uint32_t)h[4] | ((uint32_t)h[5] << 16), (uint32_t)h[6] | ((uint32_t)h[7] << 16)};
}

// A transposed right operand: bytes per row of it, and the lane's offset in a row (its rows' addresses are uniform)
struct BSrc {
  int64_t row;
  uint32_t lane;
};
// requests unit u of k-tile kt of both operands (unit u of a thread: tile row tid / CPR + RPP u, columns
// 8 (tid % CPR) .. + 8; the pointers already point at that row and column of k-tile 0).  A transposed right operand's units
// are needed together and requested with the last: wave w has rows BKT / 8 * w .. of a k-tile, a lane four columns.
template <int AM, int TM, bool BT>
__device__ __forceinline__ void issue_unit(Stage<AM, TM, BT>& st, int u, const char* const (&ap)[Geo<AM, TM, BT>::NA],
                                           const char* const (&bp)[Geo<AM, TM, BT>::NU], int kt, const BSrc& bs) {
  using G = Geo<AM, TM, BT>;
  constexpr int ES = AM ? 4 : 2;
  if (u < G::NA) {
    const char* p = ap[u] + (int64_t)kt * G::BKT * ES;
    st.a[u][0] = *reinterpret_cast<const u32x4*>(p);
    if constexpr (AM != 0) st.a[u][1] = *reinterpret_cast<const u32x4*>(p + 16);
  }
  if constexpr (!BT) {
    st.b[u] = *reinterpret_cast<const u32x4*>(bp[u] + (int64_t)kt * G::BKT * 2);
  } else if (u == G::NU - 1) {
    const char* p = bp[0] + (int64_t)kt * G::BKT * bs.row;
#pragma unroll
    for (int r = 0; r < 2 * G::NU; ++r) {
      const u32x2 x = *reinterpret_cast<const u32x2*>(p + r * bs.row + bs.lane);
      st.b[r >> 1][2 * (r & 1)] = x[0];
      st.b[r >> 1][2 * (r & 1) + 1] = x[1];
    }
  }
}
template <int AM, int TM, bool BT>
__device__ __forceinline__ void issue(Stage<AM, TM, BT>& st, const char* const (&ap)[Geo<AM, TM, BT>::NA],
                                      const char* const (&bp)[Geo<AM, TM, BT>::NU], int kt, const BSrc& bs) {
#pragma unroll
  for (int u = 0; u < Geo<AM, TM, BT>::NU; ++u) issue_unit<AM, TM, BT>(st, u, ap, bp, kt, bs);
}

// writes unit u of the staged k-tile to the LDS stage at `stage` as bf16 (fp32 A: rounded, or head and tail tiles)
template <int AM, int TM, bool BT>
__device__ __forceinline__ void commit_unit(const Stage<AM, TM, BT>& st, int u, uint16_t* stage, int tid) {
  using G = Geo<AM, TM, BT>;
  const int off = ((tid / G::CPR) + G::RPP * u) * G::LD + 8 * (tid % G::CPR);
  if (u < G::NA) {
    u32x4* d0 = reinterpret_cast<u32x4*>(stage + off);
    if constexpr (AM == 0) {
      *d0 = st.a[u][0];
    } else if constexpr (AM == 2) {
      *d0 = round8(st.a[u][0], st.a[u][1], nullptr);
    } else {
      u32x4 tail;
      *d0 = round8(st.a[u][0], st.a[u][1], &tail);
      *reinterpret_cast<u32x4*>(stage + G::kATile + off) = tail;
    }
  }
  uint16_t* bs = stage + G::NP * G::kATile;
  if constexpr (!BT) {
    *reinterpret_cast<u32x4*>(bs + off) = st.b[u];
  } else {  // columns 4 (tid % 64) + j: all of the thread's rows, two in a word; unit u writes its share of the four
    constexpr int R = 2 * G::NU, per = 4 / G::NU;
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int j = per * u; j < per * (u + 1); ++j) {
      uint32_t w[R / 2];
#pragma unroll
      for (int q = 0; q < R / 2; ++q) {
        const uint32_t lo = st.b[q][j >> 1], hi = st.b[q][2 + (j >> 1)];  // rows 2 q and 2 q + 1
        w[q] = (j & 1) ? (lo >> 16) | (hi & 0xffff0000u) : (lo & 0xffffu) | (hi << 16);
      }
      uint16_t* d = bs + b_row<AM, TM, BT>(4 * lane + j) + R * wave;
      if constexpr (R == 8) *reinterpret_cast<u32x4*>(d) = u32x4{w[0], w[1], w[2], w[3]};
      else *reinterpret_cast<u32x2*>(d) = u32x2{w[0], w[1]};
    }
  }
}
template <int AM, int TM, bool BT>
__device__ __forceinline__ void commit(const Stage<AM, TM, BT>& st, uint16_t* stage, int tid) {
#pragma unroll
  for (int u = 0; u < Geo<AM, TM, BT>::NU; ++u) commit_unit<AM, TM, BT>(st, u, stage, tid);
}

// The MFMA operands of one step (16 columns of the k-tile) of a wave: lane half lh takes one half of the tile's
// columns, eight per step (both operands in the same order, so the order of the contraction index does not
// matter)
template <int AM, int TM, bool BT>
struct Ops {
  bf16x8 a[kAF];
  bf16x8 al[AM == 1 ? kAF : 1];
  bf16x8 b[Geo<AM, TM, BT>::kBF];
};
template <int AM, int TM, bool BT>
__device__ __forceinline__ void read_ops(Ops<AM, TM, BT>& o, const uint16_t* stage, int wm, int wn, int lc, int lh, int j) {
  using G = Geo<AM, TM, BT>;
  const int col = (G::BKT / 2) * lh + 8 * j;
  const uint16_t* Bq = stage + G::NP * G::kATile;
#pragma unroll
  for (int n = 0; n < G::kBF; ++n) o.b[n] = *reinterpret_cast<const bf16x8*>(Bq + b_row<AM, TM, BT>(G::WTN * wn + 32 * n + lc) + col);
#pragma unroll
  for (int i = 0; i < kAF; ++i) {
    const int off = (WTM * wm + 32 * i + lc) * G::LD + col;
    o.a[i] = *reinterpret_cast<const bf16x8*>(stage + off);
    if constexpr (AM == 1) o.al[i] = *reinterpret_cast<const bf16x8*>(stage + G::kATile + off);
  }
}
template <int AM, int TM, bool BT>
__device__ __forceinline__ void mma(const Ops<AM, TM, BT>& o, f32x16 (&acc)[kAF][Geo<AM, TM, BT>::kBF]) {
  constexpr int kBF = Geo<AM, TM, BT>::kBF;
#pragma unroll
  for (int i = 0; i < kAF; ++i) {
#pragma unroll
    for (int n = 0; n < kBF; ++n) acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.a[i], o.b[n], acc[i][n], 0, 0, 0);
    if constexpr (AM == 1) {
#pragma unroll
      for (int n = 0; n < kBF; ++n) acc[i][n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.al[i], o.b[n], acc[i][n], 0, 0, 0);
    }
  }
}

template <int AM, int EPI, int TM, bool BT, int ONCE>
__global__ __launch_bounds__(kThreads, (AM == 1 && TM == 128 ? 4 : 2)) void gemm_nt(const GemmArgs args) {
  using G = Geo<AM, TM, BT>;
  constexpr int WTN = G::WTN, kBF = G::kBF;
  // two stages, each the tile(s) of A followed by the tile of B
  __shared__ __align__(16) uint16_t lds[2 * G::kStage];

  // the problem of this workgroup, and its tile: column tiles of a row tile side by side, row tiles of a split, splits
  int pi = 0;
  for (int q = 1; q < args.n; ++q)
    if ((int)blockIdx.x >= args.p[q].blk_begin) pi = q;
  const GemmProb& g = args.p[pi];
  const int local = blockIdx.x - g.blk_begin;
  if constexpr (EPI == EPI_PROJECTED) {
    if (local == 0 && threadIdx.x == 0 && g.sync) *g.sync = 0u;
  }
  int Mrows = g.M;
  if (g.n_rows_dev) {
    const int nd = g.n_rows_dev[0];
    Mrows = nd < Mrows ? nd : Mrows;
  }
  if (Mrows <= 0) return;  // uniform, as the next one
  const int splits = EPI == EPI_SCATTER ? parts_for(g, Mrows) : g.splits;
  const int row_tiles = ((EPI == EPI_SCATTER && g.row_tiles ? Mrows : g.M) + TM - 1) / TM;
  const int tile_n = local % g.col_tiles, tile_m = (local / g.col_tiles) % row_tiles, split = local / (g.col_tiles * row_tiles);
  if (tile_m * TM >= Mrows || split >= splits) return;
  const int N = g.N;
  void* const Dmat = g.D;
  const int64_t lda = g.lda, ldb = g.ldb, ldd = g.ldd;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lc = lane & 31, lh = lane >> 5;
  const int wm = wave / G::WN, wn = wave % G::WN;
  constexpr int ES = AM ? 4 : 2;  // bytes per element of A

  // k-tiles of this split
  const int nk = g.K / G::BKT;  // K is a multiple of 64
  const int kt0 = (int)(((int64_t)nk * split) / splits), kt1 = (int)(((int64_t)nk * (split + 1)) / splits);

  // staging pointers: a thread's unit u is tile row tid / CPR + RPP u, 8 columns at 8 (tid % CPR); rows past the
  // end repeat the last one (their results are not stored)
  const char* ap[G::NA];
  const char* bp[G::NU];
#pragma unroll
  for (int u = 0; u < G::NA; ++u) {
    int grow = tile_m * TM + (tid / G::CPR) + G::RPP * u;
    grow = grow < Mrows ? grow : Mrows - 1;
    if (g.row_idx) grow = g.row_idx[grow];
    ap[u] = reinterpret_cast<const char*>(g.A) + ((int64_t)grow * lda + 8 * (tid % G::CPR)) * ES;
  }
  BSrc bsrc{0, 0u};
  if constexpr (BT) {  // columns past the end repeat the last four
    bsrc = BSrc{ldb * 2, 2u * (uint32_t)min(tile_n * BN + 4 * lane, N - 4)};
    bp[0] = reinterpret_cast<const char*>(g.B) + (int64_t)(G::BKT / 8) * wave * bsrc.row;
  }
#pragma unroll
  for (int u = 0; !BT && u < G::NU; ++u) {
    int grow = tile_n * BN + (tid / G::CPR) + G::RPP * u;
    grow = grow < N ? grow : N - 1;
    bp[u] = reinterpret_cast<const char*>(g.B) + ((int64_t)grow * ldb + 8 * (tid % G::CPR)) * 2;
  }

  f32x16 acc[kAF][kBF];
#pragma unroll
  for (int i = 0; i < kAF; ++i)
#pragma unroll
    for (int j = 0; j < kBF; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  if (kt0 < kt1) {
    // Tile t is multiplied out of stage t & 1 while tile t + 1 (in registers since the tile before) is written
    // to the other stage, a unit per MFMA step, and each unit's registers are asked for tile t + 2 at once.
    // One barrier per tile, before the last step: by then every wave has written its share of the next stage
    // and has the last step's operands in registers, so the first operands of the next tile are read behind
    // the last step's MFMAs.  Past the range the last tile is requested (and staged) again and never used.
    Stage<AM, TM, BT> st;
    issue<AM, TM, BT>(st, ap, bp, kt0, bsrc);
    commit<AM, TM, BT>(st, lds, tid);
    issue<AM, TM, BT>(st, ap, bp, kt0 + 1 < kt1 ? kt0 + 1 : kt0, bsrc);
    __syncthreads();
    if constexpr (AM == 1 && TM == 128) {
      // Residual and image rows, W r of few rows: two workgroups per compute unit (one's epilogue beside the other's products),
      // operands are read step by step, the other waves of the SIMD cover the reads.  The form that transposes its right
      // operand has the same loop but one workgroup per unit (82304 bytes of LDS, 134 registers).  With the column groups'
      // rows swapped in place of the padding two fit (81920 bytes, 128 registers, four waves per SIMD), which was no faster: us,
      // coefficients of fp32 tokens, a block of 4096 / 16384, one / two: rank 256, 1024 tokens 148 / 157, 2048 234 / 252, rank 512, 768
      // tokens (384 workgroups) 164 / 179, 1500 255 / 252, 2048 348 / 345.
      const char* pa = ap[0] + (int64_t)(kt0 + 1 < kt1 ? kt0 + 1 : kt0) * G::BKT * ES;  // the k-tile requested last
      const char* pb[G::NU];
#pragma unroll
      for (int u = 0; u < (BT ? 1 : G::NU); ++u) pb[u] = bp[u] + (int64_t)(kt0 + 1 < kt1 ? kt0 + 1 : kt0) * G::BKT * 2 * (BT ? ldb : 1);
      static_assert(G::NA == 1, "one staging unit of A per thread");
      int cur = 0;
      for (int kt = kt0; kt < kt1; ++kt) {
        const int step = kt + 2 < kt1 ? G::BKT : 0;
#pragma unroll
        for (int j = 0; j < G::KS; ++j) {
          Ops<AM, TM, BT> o;
          read_ops<AM, TM, BT>(o, lds + cur, wm, wn, lc, lh, j);
          mma<AM, TM, BT>(o, acc);
          commit_unit<AM, TM, BT>(st, j, lds + (G::kStage - cur), tid);
          if (j == 0) {
            pa += step * ES;
            st.a[0][0] = *reinterpret_cast<const u32x4*>(pa);
            st.a[0][1] = *reinterpret_cast<const u32x4*>(pa + 16);
          }
          if constexpr (BT) {
            if (j == G::KS - 1) {
              pb[0] += step * bsrc.row;
#pragma unroll
              for (int r = 0; r < 2 * G::NU; ++r) {
                const u32x2 x = *reinterpret_cast<const u32x2*>(pb[0] + r * bsrc.row + bsrc.lane);
                st.b[r >> 1][2 * (r & 1)] = x[0];
                st.b[r >> 1][2 * (r & 1) + 1] = x[1];
              }
            }
          } else {
            pb[j] += step * 2;
            st.b[j] = *reinterpret_cast<const u32x4*>(pb[j]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        cur = G::kStage - cur;
        __syncthreads();
      }
    } else {
      Ops<AM, TM, BT> o[2];
      read_ops<AM, TM, BT>(o[0], lds, wm, wn, lc, lh, 0);
      for (int kt = kt0; kt < kt1; ++kt) {
        uint16_t* cur = lds + ((kt - kt0) & 1) * G::kStage;
        uint16_t* nxt = lds + (((kt - kt0) & 1) ^ 1) * G::kStage;
        const int kt2 = kt + 2 < kt1 ? kt + 2 : kt1 - 1;
#pragma unroll
        for (int j = 0; j < G::KS; ++j) {
          if (j + 1 < G::KS) {
            read_ops<AM, TM, BT>(o[(j + 1) & 1], cur, wm, wn, lc, lh, j + 1);
          } else {
            __syncthreads();
            read_ops<AM, TM, BT>(o[(j + 1) & 1], nxt, wm, wn, lc, lh, 0);
          }
          mma<AM, TM, BT>(o[j & 1], acc);
          if (j + 1 < G::KS) {
            // a unit behind every step but the last two, which share the step before the barrier
            commit_unit<AM, TM, BT>(st, j, nxt, tid);
            issue_unit<AM, TM, BT>(st, j, ap, bp, kt2, bsrc);
            if (j + 2 == G::KS) {
              commit_unit<AM, TM, BT>(st, j + 1, nxt, tid);
              issue_unit<AM, TM, BT>(st, j + 1, ap, bp, kt2, bsrc);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }

  // ---- epilogue --------------------------------------------------------------------------------------
  // Element v of lane l of fragment (i, n) is row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 of the
  // fragment.  The accumulators go through LDS eight rows at a time (a private strip per wave), so that
  // what touches memory is row-contiguous: a lane then owns four consecutive columns of a row.
  __syncthreads();  // the operand tiles are no longer read
  constexpr int kSR = 8, kSLD = WTN + 4;  // strip rows, padded strip stride (floats)
  float* strip = reinterpret_cast<float*>(lds) + wave * (kSR * kSLD);
  const bool partial = splits > 1;
  float* const pdst = partial ? g.part + (int64_t)split * Mrows * N : nullptr;
  // a lane reads four columns of one row, the wave kRL rows at a time
  constexpr int kLR = WTN / 4, kRL = kWave / kLR, kReads = kSR / kRL;  // lanes per strip row, rows per read, reads per strip
  const int er = lane / kLR, ec = 4 * (lane % kLR);
#pragma unroll
  for (int c = 0; c < WTM / kSR; ++c) {
    // strip c: rows 8 c .. 8 c + 7 of the wave tile = fragment c / 4, accumulator elements 4 (c % 4) .. + 3
    const int i = c >> 2, vbase = 4 * (c & 3);
#pragma unroll
    for (int vv = 0; vv < 4; ++vv) {
      const int rl = 4 * lh + vv;
#pragma unroll
      for (int n = 0; n < kBF; ++n) strip[rl * kSLD + 32 * n + lc] = acc[i][n][vbase + vv];
    }
    // The strip is private to the wave and a wave's LDS operations execute in order, so no workgroup barrier is
    // needed (one would also wait for the stores of the round before to complete); the fence only keeps the
    // compiler from moving a lane's reads above the other lanes' writes.
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int col = tile_n * BN + WTN * wn + ec;
    float4 val[kReads];
    int row[kReads];
#pragma unroll
    for (int q = 0; q < kReads; ++q) {
      row[q] = tile_m * TM + WTM * wm + kSR * c + kRL * q + er;
      val[q] = *reinterpret_cast<const float4*>(&strip[(kRL * q + er) * kSLD + ec]);
    }
    if (partial) {
#pragma unroll
      for (int q = 0; q < kReads; ++q)
        if (row[q] < Mrows && col < N)  // N is a multiple of 4 here (checked on the host)
          *reinterpret_cast<float4*>(pdst + (int64_t)row[q] * N + col) = val[q];
    } else if (EPI == EPI_PROJECTED && g.epi == EPI_RESIDUAL) {
      // r = x - acc; R written; per row the sums of r^2 and x^2 over this wave's columns (128; 64 with tiles of 128 rows)
      float4 x[kReads];
#pragma unroll
      for (int q = 0; q < kReads; ++q) {
        x[q] = float4{0.f, 0.f, 0.f, 0.f};
        if (row[q] < Mrows && col < N) {
          if (g.xdtype == GSI_F32) {
            x[q] = load_row<ONCE == 2>(reinterpret_cast<const float*>(g.X) + (int64_t)row[q] * ldd + col);
          } else {
            const uint2 xb = load_row<ONCE == 2>(reinterpret_cast<const uint16_t*>(g.X) + (int64_t)row[q] * ldd + col);
            x[q] = float4{bf16_lo(xb.x), bf16_hi(xb.x), bf16_lo(xb.y), bf16_hi(xb.y)};
          }
        }
      }
#pragma unroll
      for (int q = 0; q < kReads; ++q) {
        const bool live = row[q] < Mrows && col < N;
        const float4 r = float4{x[q].x - val[q].x, x[q].y - val[q].y, x[q].z - val[q].z, x[q].w - val[q].w};
        float sr = 0.f, sx = 0.f;
        if (live) {
          store_row<ONCE != 0>(reinterpret_cast<float*>(Dmat) + (int64_t)row[q] * ldd + col, r);
          sr = fmaf(r.x, r.x, fmaf(r.y, r.y, fmaf(r.z, r.z, r.w * r.w)));
          sx = fmaf(x[q].x, x[q].x, fmaf(x[q].y, x[q].y, fmaf(x[q].z, x[q].z, x[q].w * x[q].w)));
        }
        sr = group_sum_rt(sr, kLR);
        sx = group_sum_rt(sx, kLR);
        if (lane % kLR == 0 && row[q] < Mrows && tile_n * BN + WTN * wn < N) {
          float* pn = g.part_n + ((int64_t)(tile_n * G::WN + wn) * g.M + row[q]) * 2;
          pn[0] = sr;
          pn[1] = sx;
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < kReads; ++q) {
        if (row[q] < Mrows && col < N) {
          if constexpr (EPI == EPI_STORE_BF16) {
            uint2 o;
            o.x = (uint32_t)f32_to_bf16_bits(val[q].x) | ((uint32_t)f32_to_bf16_bits(val[q].y) << 16);
            o.y = (uint32_t)f32_to_bf16_bits(val[q].z) | ((uint32_t)f32_to_bf16_bits(val[q].w) << 16);
            *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(Dmat) + (int64_t)row[q] * ldd + col) = o;
          } else if constexpr (EPI == EPI_STORE_F32 || EPI == EPI_PROJECTED) {
            float* const dp = reinterpret_cast<float*>(Dmat) + (int64_t)row[q] * ldd + col;
            store_row<ONCE != 0>(dp, val[q]);
            if constexpr (EPI == EPI_STORE_F32)
              if (g.Ht) store_two_terms(g.Ht, row[q], N, col, val[q]);
          } else {  // scatter: one workgroup owns an output element, so the update is ordered
            const int drow = g.row_idx ? g.row_idx[row[q]] : row[q];
            float* const dp = reinterpret_cast<float*>(Dmat) + (int64_t)drow * ldd + col;
            if (g.epi == EPI_SCATTER_STORE) {
              store_row<ONCE != 0>(dp, val[q]);
            } else {
              const float4 o = load_row<ONCE != 0>(dp);
              store_row<ONCE != 0>(dp, float4{o.x + val[q].x, o.y + val[q].y, o.z + val[q].z, o.w + val[q].w});
            }
          }
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the strip is rewritten by the next round
    __builtin_amdgcn_wave_barrier();
  }
}

// Adds the partial sums of a split contraction in split order and applies the epilogue (store / scatter-add).
// A thread owns four consecutive columns; the blocks stride over the live rows (a device-side count for the
// scatter-add product), so the launch does not grow with rows that did not fire.
template <int EPI, int ONCE>
__global__ __launch_bounds__(256) void splitk_finish(const GemmArgs args) {
  const GemmProb& g = args.p[blockIdx.y];
  if (g.splits <= 1 && !g.row_tiles) return;
  int Mrows = g.M;
  if (g.n_rows_dev) {
    const int nd = g.n_rows_dev[0];
    Mrows = nd < Mrows ? nd : Mrows;
  }
  if (Mrows <= 0) return;
  const int splits = EPI == EPI_SCATTER ? parts_for(g, Mrows) : g.splits;
  if (splits <= 1) return;
  const int n4 = g.N >> 2;
  const int64_t total = (int64_t)Mrows * n4, stride = (int64_t)Mrows * g.N;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int row = (int)(e / n4), col = 4 * (int)(e - (int64_t)row * n4);
    const float* src = g.part + (int64_t)row * g.N + col;
    float4 s = float4{0.f, 0.f, 0.f, 0.f};
    for (int z0 = 0; z0 < splits; z0 += 8) {
      float4 q[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) q[u] = load_row<ONCE != 0>(src + (int64_t)min(z0 + u, splits - 1) * stride);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (z0 + u < splits) { s.x += q[u].x; s.y += q[u].y; s.z += q[u].z; s.w += q[u].w; }
    }
    if constexpr (EPI == EPI_STORE_BF16) {
      uint2 o;
      o.x = (uint32_t)f32_to_bf16_bits(s.x) | ((uint32_t)f32_to_bf16_bits(s.y) << 16);
      o.y = (uint32_t)f32_to_bf16_bits(s.z) | ((uint32_t)f32_to_bf16_bits(s.w) << 16);
      *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(g.D) + (int64_t)row * g.ldd + col) = o;
    } else if constexpr (EPI == EPI_STORE_F32) {
      *reinterpret_cast<float4*>(reinterpret_cast<float*>(g.D) + (int64_t)row * g.ldd + col) = s;
      if (g.Ht) store_two_terms(g.Ht, row, g.N, col, s);
    } else {
      const int drow = g.row_idx ? g.row_idx[row] : row;
      float* const dp = reinterpret_cast<float*>(g.D) + (int64_t)drow * g.ldd + col;
      if (g.epi == EPI_SCATTER_STORE) {
        store_row<ONCE != 0>(dp, s);
      } else {
        const float4 o = load_row<ONCE != 0>(dp);
        store_row<ONCE != 0>(dp, float4{o.x + s.x, o.y + s.y, o.z + s.z, o.w + s.w});
      }
    }
  }
}

// Ut[j][i] = U[i][j] for bf16 matrices U[rows, cols]: 64 x 64 tiles through LDS, whole 128-byte rows on both sides
// (32 x 32 tiles: 64-byte rows, 8.4 us for 4096 x 512; the block's four bases at rank 512, 15 us in one launch)
constexpr int kMaxTransposes = 64;
struct TransposeArgs {
  TransposeTask t[kMaxTransposes];
  int n;
};
static_assert(sizeof(TransposeArgs) <= 4096, "kernel arguments are limited to 4 KB");
__global__ __launch_bounds__(256) void transpose_bf16(const TransposeArgs a) {
  constexpr int T = 64;
  __shared__ uint16_t tile[T][T + 2];
  int ti = 0;
  for (int q = 1; q < a.n; ++q)
    if ((int)blockIdx.x >= a.t[q].blk_begin) ti = q;
  const TransposeTask& t = a.t[ti];
  const uint16_t* __restrict__ U = reinterpret_cast<const uint16_t*>(t.U);
  uint16_t* __restrict__ Ut = reinterpret_cast<uint16_t*>(t.Ut);
  const int rows = t.rows, cols = t.cols, ct = (cols + T - 1) / T;
  const int local = blockIdx.x - t.blk_begin;
  const int r0 = (local / ct) * T, c0 = (local % ct) * T;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  uint16_t v[T / 4];
#pragma unroll
  for (int q = 0; q < T / 4; ++q) {
    const int r = r0 + ty + 4 * q, c = c0 + tx;
    v[q] = (r < rows && c < cols) ? U[(int64_t)r * cols + c] : (uint16_t)0;
  }
#pragma unroll
  for (int q = 0; q < T / 4; ++q) tile[ty + 4 * q][tx] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < T / 4; ++q) {
    const int c = c0 + ty + 4 * q, r = r0 + tx;
    if (r < rows && c < cols) Ut[(int64_t)c * rows + r] = tile[tx][ty + 4 * q];
  }
}

// of the sums of a launch's parts: a thread per four elements of the largest result, up to a limit
dim3 finish_grid(const GemmArgs& g) {
  int64_t most = 1;
  for (int i = 0; i < g.n; ++i) {
    const GemmProb& p = g.p[i];
    if (p.splits > 1 || p.row_tiles)
      most = std::max(most, (int64_t)(p.row_tiles && p.splits == 1 ? std::min(p.M, p.tile_rows * p.row_tiles) : p.M) * (p.N / 4));
  }
  return dim3((unsigned)std::min<int64_t>(ceil_div(most, 256), 4096), (unsigned)g.n);
}

template <int AM, int EPI, bool BT, int ONCE = 0>
hipError_t launch_group(GemmArgs& g, int tm, hipStream_t s) {
  constexpr int R = EPI == EPI_STORE_F32 || EPI == EPI_STORE_BF16 ? 0 : ONCE;  // (the next launch reads coefficients; images stay)
  int64_t blocks = 0;
  bool split = false;
  for (int i = 0; i < g.n; ++i) {
    GemmProb& p = g.p[i];
    p.col_tiles = (int)ceil_div(p.N, BN);
    p.blk_begin = (int)blocks;
    blocks += (int64_t)p.col_tiles * ceil_div(p.M, tm) * p.splits;
    split |= p.splits > 1 || p.row_tiles;
  }
  if (blocks >= (1ll << 31)) return hipErrorInvalidValue;
  if (tm == 256) {
    gemm_nt<AM, EPI, 256, BT, R><<<(unsigned)blocks, kThreads, 0, s>>>(g);
  } else if (tm == 128) {
    gemm_nt<AM, EPI, 128, BT, R><<<(unsigned)blocks, kThreads, 0, s>>>(g);
  } else {
    if constexpr (EPI == EPI_STORE_BF16) gemm_nt<AM, EPI, 64, BT, R><<<(unsigned)blocks, kThreads, 0, s>>>(g);
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  if constexpr (EPI != EPI_PROJECTED)
    if (split) splitk_finish<EPI, ONCE><<<finish_grid(g), 256, 0, s>>>(g);
  return hipGetLastError();
}

// the forms of the operands that a caller has with each epilogue, and no others
hipError_t launch_epi(GemmArgs& g, int a_f32, int epi, bool bt, int once, int tm, hipStream_t s) {
  switch (epi) {
    case EPI_STORE_BF16:
      if (a_f32 != 0) break;
      if (once) return bt ? launch_group<0, EPI_STORE_BF16, true, 1>(g, tm, s) : launch_group<0, EPI_STORE_BF16, false, 1>(g, tm, s);
      return bt ? launch_group<0, EPI_STORE_BF16, true>(g, tm, s) : launch_group<0, EPI_STORE_BF16, false>(g, tm, s);
      break;
    case EPI_STORE_F32:
      if (once) {
        if (a_f32 == 0) return bt ? launch_group<0, EPI_STORE_F32, true, 1>(g, tm, s) : launch_group<0, EPI_STORE_F32, false, 1>(g, tm, s);
        if (a_f32 == 1) return bt ? launch_group<1, EPI_STORE_F32, true, 1>(g, tm, s) : launch_group<1, EPI_STORE_F32, false, 1>(g, tm, s);
        break;
      }
      if (a_f32 == 0) return bt ? launch_group<0, EPI_STORE_F32, true>(g, tm, s) : launch_group<0, EPI_STORE_F32, false>(g, tm, s);
      if (a_f32 == 1) return bt ? launch_group<1, EPI_STORE_F32, true>(g, tm, s) : launch_group<1, EPI_STORE_F32, false>(g, tm, s);
      break;
    case EPI_PROJECTED:
      if (a_f32 != 1 || bt) break;
      if (once == 0) return launch_group<1, EPI_PROJECTED, false>(g, tm, s);
      return once == 1 ? launch_group<1, EPI_PROJECTED, false, 1>(g, tm, s) : launch_group<1, EPI_PROJECTED, false, 2>(g, tm, s);
    case EPI_SCATTER:
      if (bt) break;
      if (a_f32 == 0) return once ? launch_group<0, EPI_SCATTER, false, 1>(g, tm, s) : launch_group<0, EPI_SCATTER, false>(g, tm, s);
      if (a_f32 == 1) return once ? launch_group<1, EPI_SCATTER, false, 1>(g, tm, s) : launch_group<1, EPI_SCATTER, false>(g, tm, s);
      if (a_f32 == 2) return once ? launch_group<2, EPI_SCATTER, false, 1>(g, tm, s) : launch_group<2, EPI_SCATTER, false>(g, tm, s);
      break;
  }
  return hipErrorInvalidValue;
}

// rows that a product is sized for: the scatter products run over the fired rows only (a device-side count): a quarter
int64_t rows_expected(int64_t M, int epi) {
  return (epi == EPI_SCATTER_ADD || epi == EPI_SCATTER_STORE) ? std::max<int64_t>(std::min<int64_t>(M, 128), M / 4) : M;
}
constexpr int kMaxSplits = 32;

// Small images run on tiles of 64 rows: they are cut until the chip is full, and what the parts write and the sums read back is
// a good part of the time: half the rows, half the parts.  us, tiles of 128 / 64 rows, at rank 64 and 256: 1024 x 1024
// 15 / 13, 16 / 14; 2176 x 2176 17 / 15, 21 / 18; 4096 x 4096 20 / 22, 28 / 26; 4096 x 14720 39 / 50, 50 / 56; at rank 512, 1024 x 1024
// 17 / 15, 2176 x 2176 22 / 28.
bool image_rows64(int64_t M, int64_t N, int64_t K) { return mfma_image_work(M, N, K) <= 640; }

}  // namespace

// The split is a property of the product alone, so that a product gives the same bits in whatever launch it runs (the
// row tile, which plan_rows chooses for a launch, does not change the order of a sum), and over a device-side count of rows
// of that count (parts_for).  Products of fewer tiles (of 128
// rows) than there are units are cut into parts of 4096 columns, which makes the products of a block alike; those of so few
// tiles (less than an eighth of the units) that even their parts are less than a quarter of the chip, and image builds,
// which are alone in their launch, are cut further, down to 512 columns.  Measured, GEMM + sums of the partials: projections of a block, 2048 tokens:
// parts of 4096 columns 85 + 7 us, 2048: 91 + 15, 1024: 108 + 25; the projections of the pair at 333 tokens 105 + 5, 59 + 5,
// 34 + 5; an image of 4096 x 4096 x 256: 57, 33 + 6, 22 + 7 (on tiles of 128 rows).
// Products of up to half the units are cut again while their parts fit the chip at once, down to 1024 columns (512 for an
// eighth of the units): a workgroup takes 0.75 us per 64 columns, 1.5 us with a two-term operand, however few there are.  In
// eight at most; a two-term contraction of 8192 columns and more even beyond the chip.  Scatter products of more than one row
// tile are cut so in two, or until half the chip has a part: others of their block share the launch.  The
// coefficients of a projection are cut so only with a two-term operand.  Measured, us per call without / with this second cut
// (calls replayed from a graph): 129 x 4096 x 4096 48 / 23, two-term 97 / 36; 512 rows 50 / 33, 101 / 47; 1024 rows 53 / 50,
// 104 / 77; W r of 4096 x 4096 with 205 of 1024 rows fired 78 / 42; the projection of 2048 fp32 tokens, 4096 x 512
// 141 / 77; the block of 2048 tokens 742 / 730 (its W r launch 295 + 15 / 268 + 31).
// Where the workspace has room, two-term coefficients are cut into as many parts as half the chip takes: the second cut ends at eight,
// which leaves a long contraction of few tiles on a quarter of it (4096 / 16384, 400 tokens at rank 512: 192 workgroups, the longest of 32
// k-tiles), and it doubles, which leaves 40 or 160 k-tiles in parts of 10 and 13.  Down to 512 columns, or 256 where there are at most
// four tiles; with more, the other inputs of a block fill the chip already, and half as deep again was slower: a block of 2048 / 8192 and
// 4096 / 16384 at rank 256, 777 tokens 98 / 104, 158 / 165; 4096 / 16384, 640 tokens 128 / 133; cut to the whole chip, 4096 / 16384 at rank
// 512, 1000 tokens 272 / 295.  us a call, none fired, without / with it: the pair 1024 / 4096 at rank 64, 200 tokens 44 / 40;
// 2560 / 10240 54 / 46, 640 tokens 66 / 60; at rank 256, 500 tokens 71 / 65; 4096 / 16384 at rank 256, 400 tokens 87 / 79, 900 134 / 117; at rank
// 512, 400 tokens 126 / 106; a block of 2560 / 10240 at rank 64, 200 tokens 63 / 55, 640 86 / 80; 4096 / 16384 at rank 256, 900 tokens
// 184 / 171; of 85 calls none slower by more than runs differ.
int mfma_splits(int64_t M, int64_t N, int64_t K, int epi, bool two_term, WsLevel level) {
  if (epi == EPI_RESIDUAL) return 1;
  const int64_t m = rows_expected(M, epi), nk = ceil_div(K, BK);
  int s = 1;
  if (level == kWsFirst) {
    const int64_t tiles = ceil_div(std::max<int64_t>(m, 256), 256) * ceil_div(N, BN);
    while (s < 8 && tiles * s < kUnits && nk / (s * 2) >= 4) s *= 2;
    return s;
  }
  const int64_t tiles = ceil_div(m, 128) * ceil_div(N, BN);
  if (tiles < kUnits) s = (int)std::min<int64_t>(ceil_div(nk, kMaxDepth), kMaxSplits);
  const int64_t want = epi == EPI_STORE_BF16 ? kUnits : tiles < kUnits / 8 ? kUnits / 4 : 0;
  while (s * 2 <= kMaxSplits && tiles * s < want && nk / (s * 2) >= kMinDepth) s *= 2;
  if (epi == EPI_STORE_BF16 && image_rows64(M, N, K)) {  // (never more parts than tiles of 128 rows had)
    const int64_t tiles64 = ceil_div(M, 64) * ceil_div(N, BN);
    int t = 1;
    while (t < s && tiles64 * t < kUnits) t *= 2;
    return std::min(s, t);
  }
  if (level == kWsCoarse || epi == EPI_STORE_BF16 || (epi == EPI_COEFF && !two_term)) return s;
  const bool shares = (epi == EPI_SCATTER_ADD || epi == EPI_SCATTER_STORE) && m > 128;
  const int64_t room = two_term && nk >= 2 * kMaxDepth ? 2 * kUnits : kUnits;
  while (s < 8 && tiles * s * 2 <= (shares && s > 1 ? kUnits / 2 : room) &&
         nk / (s * 2) >= (tiles * s > kUnits / 8 ? 2 * kMinDepth : kMinDepth))
    s *= 2;
  if (level == kWsFull && epi == EPI_COEFF)
    s = (int)std::min<int64_t>(std::max<int64_t>(s, std::min<int64_t>(kUnits / 2 / tiles, nk / (tiles <= kUnits / 64 ? kMinDepth / 2 : kMinDepth))), kMaxSplits);
  return s;
}

size_t mfma_part_bytes(int64_t M, int64_t N, int64_t K, int epi, WsLevel level) {
  const int s = std::max(mfma_splits(M, N, K, epi, false, level), mfma_splits(M, N, K, epi, true, level));
  const int64_t rows = s > 1 ? s * M : 128 * mfma_follow(M, K, epi, 1, level);
  return align_up((size_t)rows * N * sizeof(float), 256);
}

// Nothing to follow: one tile in one part, or a contraction too short to cut.
int mfma_follow(int64_t M, int64_t K, int epi, int splits, WsLevel level) {
  if (level < kWsFine || (epi != EPI_SCATTER_ADD && epi != EPI_SCATTER_STORE) || K < 2 * kMinDepth * BK) return 0;
  const int t = (int)ceil_div(rows_expected(M, epi), 128);
  return t * splits > 1 ? t : 0;
}

// The same for products on tiles of 256 rows over the fired rows (gsi_wide.hip): parts of 4096 columns where a product has fewer
// tiles than the chip units, and cut further, down to 1024 columns (512 for an eighth of the units), while the parts of one row
// tile fit the chip and those of several a quarter of it: others of their block share the launch.
int wide_splits(int64_t M, int64_t N, int64_t K) {
  const int64_t m = wide_rows_expected(M), nk = ceil_div(K, BK), tiles = ceil_div(m, 256) * ceil_div(N, BN);
  int64_t s = tiles < kUnits ? std::min<int64_t>(ceil_div(nk, kMaxDepth), kMaxSplits) : 1;
  while (s * 2 <= kMaxSplits && tiles * s < (tiles < kUnits / 8 ? kUnits / 4 : 0) && nk / (s * 2) >= kMinDepth) s *= 2;
  const int64_t room = m > 256 ? kUnits / 4 : kUnits;
  while (s < 8 && tiles * s * 2 <= room && nk / (s * 2) >= (tiles * s > kUnits / 8 ? 2 * kMinDepth : kMinDepth)) s *= 2;
  return (int)s;
}
int wide_follow(int64_t M, int64_t K, int splits) {
  if (K < 2 * kMinDepth * BK) return 0;
  const int t = (int)ceil_div(wide_rows_expected(M), 256);
  return t * splits > 1 ? t : 0;
}
size_t wide_part_bytes(int64_t M, int64_t N, int64_t K) {
  const int s = wide_splits(M, N, K);
  const int64_t rows = std::max<int64_t>(s > 1 ? s * M : 0, 256 * s * (int64_t)wide_follow(M, K, s));
  return align_up((size_t)rows * N * sizeof(float), 256);
}

hipError_t mfma_finish_basis(const GemmArgs& g, int epi, bool once, hipStream_t s) {
  const dim3 grid = finish_grid(g);
  if (epi == EPI_STORE_BF16 && once) splitk_finish<EPI_STORE_BF16, 1><<<grid, 256, 0, s>>>(g);
  else if (epi == EPI_STORE_BF16) splitk_finish<EPI_STORE_BF16, 0><<<grid, 256, 0, s>>>(g);
  else if (once) splitk_finish<EPI_STORE_F32, 1><<<grid, 256, 0, s>>>(g);
  else splitk_finish<EPI_STORE_F32, 0><<<grid, 256, 0, s>>>(g);
  return hipGetLastError();
}

hipError_t mfma_finish_scatter(const GemmArgs& g, bool once, hipStream_t s) {
  bool split = false;
  for (int i = 0; i < g.n; ++i) split |= g.p[i].splits > 1 || g.p[i].row_tiles;
  if (!split) return hipSuccess;
  if (once) splitk_finish<EPI_SCATTER, 1><<<finish_grid(g), 256, 0, s>>>(g);
  else splitk_finish<EPI_SCATTER, 0><<<finish_grid(g), 256, 0, s>>>(g);
  return hipGetLastError();
}

namespace {

// Row tile of a launch: the one with the least estimated time.  A workgroup takes its k-tiles and the time of about six
// more for its first loads and its epilogue; a tile of 128 rows takes 0.6 of the time of one of 256 (the same right-hand
// tile, half the products); the launch lasts as long as the work spread over the units, or its longest workgroup, and about
// half of that workgroup again for the tail.  (Work is spread evenly here; tiles of 256 rows hold a unit each and run in
// whole rounds, so between one round and a few the estimate is low for them.)
int plan_rows(const GemmArgs& g, int epi) {
  // (the norm shares of a residual are per 64 columns with tiles of 128 rows, per 128 with 256)
  if (epi == EPI_PROJECTED) return g.p[0].res_cols == 64 ? 128 : 256;
  if (epi == EPI_STORE_BF16 && image_rows64(g.p[0].M, g.p[0].N, g.p[0].K)) return 64;  // (a launch holds one image)
  double cost[2];
  for (int t = 0; t < 2; ++t) {
    const int tm = t ? 128 : 256;
    const double per = t ? 0.6 : 1.0;
    double total = 0.0, longest = 0.0;
    for (int i = 0; i < g.n; ++i) {
      const GemmProb& p = g.p[i];
      const double one = per * (double)(ceil_div(ceil_div(p.K, BK), p.splits) + 6);
      total += one * (double)(p.splits * ceil_div(rows_expected(p.M, p.epi), tm) * ceil_div(p.N, BN));
      longest = std::max(longest, one);
    }
    cost[t] = std::max(total / kUnits, longest) + 0.5 * longest;
  }
  return cost[1] < 0.999 * cost[0] ? 128 : 256;  // (a tie up to rounding: 256; dense fp32, 2048 x 4096 x 16384: 514 / 496 us)
}

}  // namespace

hipError_t mfma_gemm_nt(const GemmProb* probs, int n, int a_f32, int epi, hipStream_t s, bool b_rows, int once) {
  GemmArgs g;
  int i = 0;
  while (i < n) {
    g.n = 0;
    for (; i < n && g.n < kMaxProbs; ++i)
      if (probs[i].M > 0 && probs[i].N > 0) g.p[g.n++] = probs[i];
    if (g.n == 0) break;
    for (int q = 0; q < g.n; ++q) {
      g.p[q].splits = g.p[q].part ? g.p[q].max_splits : 1;
      if (!g.p[q].part) g.p[q].row_tiles = 0;
      g.p[q].tile_rows = 128;
      g.p[q].min_parts = std::min(g.p[q].splits, (int)ceil_div(g.p[q].K, BK * kMaxDepth));
    }
    // The products with the longest parts first: workgroups hold a unit each and go out in order, and what is long and
    // comes last runs on a part of the chip.  (W r of the pair 4096 / 16384, 50 of 333 rows fired: 256 parts of 16 k-tiles,
    // and 128 of 32 that came last: 79.5 -> 72.4 us.)
    std::stable_sort(g.p, g.p + g.n, [](const GemmProb& x, const GemmProb& y) {
      return (int64_t)x.K * y.splits > (int64_t)y.K * x.splits;
    });
    const int tm = plan_rows(g, epi);
    if (hipError_t e = launch_epi(g, a_f32, epi, b_rows, once, tm, s); e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t mfma_transpose_bf16(TransposeTask* tasks, int n, hipStream_t s) {
  for (int i = 0; i < n;) {
    TransposeArgs a;
    int blocks = 0;
    for (a.n = 0; i < n && a.n < kMaxTransposes; ++i, ++a.n) {
      a.t[a.n] = tasks[i];
      a.t[a.n].blk_begin = blocks;
      blocks += (int)(ceil_div(tasks[i].rows, 64) * ceil_div(tasks[i].cols, 64));
    }
    transpose_bf16<<<(unsigned)blocks, 256, 0, s>>>(a);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace gsi
