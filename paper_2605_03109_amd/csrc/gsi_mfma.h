// Host interface of the matrix-core GEMM used by the image build and the prefill-sized batched path.
#pragma once
#include "gsi_internal.h"

namespace gsi {

// What becomes of A B^T.  EPI_RESIDUAL and EPI_STORE_F32 problems share launches (EPI_PROJECTED: a residual and the image
// rows beside it), and so do EPI_SCATTER_ADD and EPI_SCATTER_STORE (EPI_SCATTER).
enum { EPI_STORE_BF16 = 0, EPI_STORE_F32 = 1, EPI_RESIDUAL = 2, EPI_SCATTER_ADD = 3, EPI_SCATTER_STORE = 4,
       EPI_PROJECTED = 5, EPI_SCATTER = 6, EPI_COEFF = 7 };

// One product D = A B^T of a launch: A[M,K] (bf16, or fp32 fed as bf16), B[N,K] bf16, both row-major.
struct GemmProb {
  const void* A;
  const void* B;
  void* D;                    // bf16 or fp32 [.., ldd]
  const void* X;              // residual: D = X - A B^T, X[M, ldd]
  float* part_n;              // ... and per-row partial sums of squares [column tiles][M][2]
  unsigned* sync;             // ... and a counter that the launch clears for the norm kernel behind it (may be null)
  const int32_t* row_idx;     // optional: row i of A is A[row_idx[i]], and (scatter) row i of D is D[row_idx[i]]
  const int32_t* n_rows_dev;  // optional: device count of valid rows (<= M)
  uint16_t* Ht;               // EPI_STORE_F32: D in two bf16 terms as well (wide_two_term), or null
  float* part;                // split contraction: workspace [splits][rows][N] of partial sums, or null (then no split)
  int lda, ldb, ldd;
  int M, N, K;                // K a multiple of 64; M * N below 2^31
  int epi;
  int xdtype;
  int max_splits;             // in: splits of the contraction that `part` has room for (mfma_splits), 1 without it
  int row_tiles;              // in: tiles of tile_rows rows that max_splits is meant for, where it follows the count (mfma_follow), or 0
  int tile_rows;              // in: 128 (256: wide_scatter)
  int res_cols;               // EPI_PROJECTED: columns per partial norm, 64 or 128 (the same in every problem)
  int splits, col_tiles, blk_begin, min_parts;  // filled at launch
};
constexpr int kMaxProbs = 24;
struct GemmArgs {
  GemmProb p[kMaxProbs];
  int n;
};
static_assert(sizeof(GemmArgs) <= 4096, "kernel arguments are limited to 4 KB");

// How many ways the contraction of an M x N x K product is split, and the workspace that takes (whatever the form of its
// operand).  epi: of the problem, or EPI_COEFF for the product of a projection.  two_term: A is fed as head + tail.
int mfma_splits(int64_t M, int64_t N, int64_t K, int epi, bool two_term, WsLevel level);
// ... and whether the split of a product over a device-side count of rows follows that count: the tiles of 128 rows that
// mfma_splits (splits) expects, or 0.
int mfma_follow(int64_t M, int64_t K, int epi, int splits, WsLevel level);
// work of an image build: its tiles of 128 rows times its k-tiles
inline int64_t mfma_image_work(int64_t m, int64_t k, int64_t d) { return ceil_div(m, 128) * ceil_div(k, 256) * ceil_div(d, 64); }
size_t mfma_part_bytes(int64_t M, int64_t N, int64_t K, int epi, WsLevel level);

// Products of one launch (n of any number; more than kMaxProbs take several launches).  a_f32: A is 0: bf16; 1: fp32, fed as
// bf16 head + tail (two passes); 2: fp32, rounded once to bf16.  epi: EPI_STORE_BF16 (A bf16), EPI_STORE_F32 (bf16 or head +
// tail), EPI_PROJECTED (head + tail) or EPI_SCATTER; every problem's own epi belongs to it.
// b_rows: B is stored [K, N] (ldb elements a row, whole 8-byte pieces) and transposed on its way (EPI_STORE_BF16, EPI_STORE_F32).
// once: EPI_PROJECTED and EPI_SCATTER: the rows of D go past the caches (1), x of a residual too (2).
hipError_t mfma_gemm_nt(const GemmProb* probs, int n, int a_f32, int epi, hipStream_t s, bool b_rows = false, int once = 0);

// Products of the fired rows (EPI_SCATTER_ADD) whose A is bf16, the fired rows one after the other (gsi_wide.hip).
struct RoundTask {
  const float* R;
  uint16_t* out;              // [rows, d]: the fired rows of R, rounded
  const int32_t* fired_idx;
  const int32_t* n_fired;
  int rows, d;                // d a multiple of 8
};
hipError_t wide_round_rows(const RoundTask* tasks, int n, bool once, hipStream_t s);
hipError_t wide_scatter(const GemmProb* probs, int n, bool once, hipStream_t s);
// Products of an operand in two terms: A is Ht, the rows of an fp32 operand as bf16 (of 32 columns the heads, their tails, the
// next 32 columns: wide_split_rows, or GemmProb::Ht of the product that makes the operand); epi EPI_RESIDUAL or EPI_STORE_F32,
// K a multiple of 64.
struct SplitTask {
  const float* C;
  uint16_t* Ht;               // [rows, wide_two_term_ld(k)]
  int rows, k;                // k a multiple of 64
};
inline int64_t wide_two_term_ld(int64_t k) { return 2 * k; }  // elements of a row of Ht
hipError_t wide_split_rows(const SplitTask* tasks, int n, hipStream_t s);
hipError_t wide_two_term(const GemmProb* probs, int n, int once, hipStream_t s);
// One such product (EPI_STORE_F32) by itself, whose A is fp32, K a multiple of 64; round: fired rows that the launch rounds beside it, or
// null.  wide_image_ok: where that is no slower than wide_split_rows and wide_two_term, whose larger tiles pay for a launch more at large
// ranks once tiles of 64 rows are more than three a unit (us, laid out first / split on the way: 11008 rows, rank 512, 1000 tokens 46.6 / 39.4,
// 1200 46.8 / 54.0, 2048 64.8 / 68.7; rank 192, 1200 32.4 / 31.8, 2048 41.1 / 41.8; 28672 rows, rank 64, 2048 tokens 59.5 / 58.0).
inline bool wide_image_ok(int64_t M, int64_t N, int64_t K) { return K <= 192 || ceil_div(M, 64) * ceil_div(N, 256) <= 3 * 256; }
hipError_t wide_image(const GemmProb& prob, const RoundTask* round, hipStream_t s);
// the split of such a product, the row tiles it is meant for, and the workspace of its partial sums
int wide_splits(int64_t M, int64_t N, int64_t K);
int wide_follow(int64_t M, int64_t K, int splits);
size_t wide_part_bytes(int64_t M, int64_t N, int64_t K);
inline bool wide_ok(int64_t K) { return K <= (1 << 22); }  // (offsets in a tile of 256 rows are 32 bits)
inline int64_t wide_rows_expected(int64_t M) { return M < 512 ? (M < 128 ? M : 128) : M / 4; }
// Products with a stored basis as the right factor (gsi_basis.hip): D = A B, A[M, K] bf16, B[K, N] bf16 as stored (ldb), K a multiple of
// 64, N of 8, B 16-byte aligned and below 2 GiB; epi EPI_STORE_BF16 or EPI_STORE_F32 (with Ht).  tm: rows of a tile, 64 or 128, or
// 0: as the launch has it.
hipError_t basis_products(const GemmProb* probs, int n, int epi, int tm, int once, hipStream_t s);
int basis_splits(int64_t M, int64_t N, int64_t K, int tm);  // of an image
int basis_coeff_splits(int64_t M, int64_t N, int64_t K);     // of coefficients (tm 128)
inline bool basis_ok(int64_t K, int64_t N) { return K % 64 == 0 && N % 8 == 0 && K <= (1 << 22) && K * N < (1ll << 30); }
// adds the partial sums of the products of a launch
hipError_t mfma_finish_basis(const GemmArgs& g, int epi, bool once, hipStream_t s);
hipError_t mfma_finish_scatter(const GemmArgs& g, bool once, hipStream_t s);

// Ut[j][i] = U[i][j] for n bf16 matrices U[rows, cols]
struct TransposeTask {
  const void* U;
  void* Ut;
  int rows, cols;
  int blk_begin;  // filled at launch
};
hipError_t mfma_transpose_bf16(TransposeTask* tasks, int n, hipStream_t s);
// columns per partial norm of the residual GEMM, and its partial norms per token
inline int mfma_res_cols(WsLevel level) { return level == kWsCoarse || level == kWsFine ? 64 : 128; }
inline int mfma_res_tiles(int64_t d, WsLevel level) { return (int)ceil_div(d, mfma_res_cols(level)); }

}  // namespace gsi
