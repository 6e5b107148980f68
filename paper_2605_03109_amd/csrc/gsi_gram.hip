// E = U^T U - I, the departure of a stored basis from orthonormality (one-time companion of the single-pass gate),
// accumulated in fp64 on the matrix cores.
//
// A workgroup owns one 16 x 16 tile of E on or above the diagonal (E is symmetric: the tile is written twice), its
// sixteen waves every sixteenth chunk of U's rows, four rows per v_mfma_f64_16x16x4_f64; the waves' sums meet in LDS
// in wave order.  The entry point has no workspace, so the rows cannot be split over workgroups; small tiles keep
// most of the chip busy instead (rank 256: 136 workgroups; 32 x 32 tiles would be 36).
// What bounds it: a unit's share of the fp64 matrix rate (27 us for 16384 rows if nothing else took its time) and the
// conversions that feed it.  d = 16384, rank 256: 51 us (633 us as fp64 FMAs out of LDS, 77 us with two-byte operand
// loads in place of the strips, which the address units bound); d = 4096: 15.5 us (160 us).
#include "gsi_device.h"
#include "gsi_internal.h"

namespace gsi {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kGWaves = 16;
constexpr int kGBlock = kGWaves * kWave;

// VEC: rows are whole 16-byte pieces (rank a multiple of 8 in bf16, 4 in fp32, aligned basis)
template <class T, bool VEC>
__global__ __launch_bounds__(kGBlock) void gram_tiles(const typename T::storage* __restrict__ U, int64_t d, int64_t k,
                                                      float* __restrict__ E) {
  using S = typename T::storage;
  constexpr int V = T::kVec;
  constexpr int R = kWave / (16 / V);  // rows of a chunk: one 16-byte load per lane covers R rows of 16 columns
  __shared__ __align__(16) double sums[kGWaves][256];  // the waves' sums; before that, their staged operands
  static_assert(2 * R * 16 * sizeof(S) <= sizeof(sums[0]), "two staged operands of a wave");
  const int tc = blockIdx.x, tr = blockIdx.y;
  if (tc < tr) return;  // below the diagonal: written by the tile above it

  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int li = lane & 15, lq = lane >> 4;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  if constexpr (VEC) {
    // A wave's chunk of R rows goes through a strip of LDS of its own, which turns whole 16-byte pieces of rows into
    // operands (row lq, column li of a step); the next chunk is requested first.  Rows past the end are zero, pieces
    // past the rank repeat its last one (their sums are not stored).
    S* const strip = reinterpret_cast<S*>(&sums[wave][0]);
    const int prow = lane / (16 / V), pcol = V * (lane % (16 / V));
    const int64_t ca = min((int64_t)tr * 16 + pcol, k - V), cb = min((int64_t)tc * 16 + pcol, k - V);
    const int64_t chunks = (d + R - 1) / R;
    uint4 pa, pb;
    auto request = [&](int64_t c) {
      const int64_t r = c * R + prow;
      const S* src = U + min(r, d - 1) * k;
      pa = *reinterpret_cast<const uint4*>(src + ca);
      pb = *reinterpret_cast<const uint4*>(src + cb);
      if (r >= d) pa = pb = uint4{0u, 0u, 0u, 0u};
    };
    if (wave < chunks) request(wave);
    for (int64_t c = wave; c < chunks; c += kGWaves) {
      *reinterpret_cast<uint4*>(strip + prow * 16 + pcol) = pa;
      *reinterpret_cast<uint4*>(strip + (R + prow) * 16 + pcol) = pb;
      if (c + kGWaves < chunks) request(c + kGWaves);
      // the strip is private to the wave, whose LDS operations execute in order: only the compiler has to be held
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int s = 0; s < R / 4; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)T::load(strip, (4 * s + lq) * 16 + li),
                                                   (double)T::load(strip, (R + 4 * s + lq) * 16 + li), acc, 0, 0, 0);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
  } else {
    // element by element, eight four-row steps requested together
    constexpr int kSteps = 8;
    const int64_t ci = min((int64_t)tr * 16 + li, k - 1), cj = min((int64_t)tc * 16 + li, k - 1);
    const int64_t steps = (d + 3) / 4;
    for (int64_t s0 = (int64_t)wave * kSteps; s0 < steps; s0 += kGWaves * kSteps) {
      float a[kSteps], c[kSteps];
#pragma unroll
      for (int q = 0; q < kSteps; ++q) {
        const int64_t rc = min((s0 + q) * 4 + lq, d - 1);
        a[q] = T::load(U, rc * k + ci);
        c[q] = T::load(U, rc * k + cj);
      }
#pragma unroll
      for (int q = 0; q < kSteps; ++q) {
        const bool live = (s0 + q) * 4 + lq < d;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(live ? (double)a[q] : 0.0, live ? (double)c[q] : 0.0, acc, 0, 0, 0);
      }
    }
  }
  // element v of a lane: row 4 v + lane / 16, column lane % 16
#pragma unroll
  for (int v = 0; v < 4; ++v) sums[wave][(4 * v + lq) * 16 + li] = acc[v];
  __syncthreads();
  if (threadIdx.x >= 256) return;
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < kGWaves; ++w) t += sums[w][threadIdx.x];
  const int64_t row = (int64_t)tr * 16 + threadIdx.x / 16, col = (int64_t)tc * 16 + threadIdx.x % 16;
  if (row >= k || col >= k) return;
  const float e = (float)(t - (row == col ? 1.0 : 0.0));
  E[row * k + col] = e;
  if (tr != tc) E[col * k + row] = e;
}

}  // namespace

hipError_t build_gram(const void* U, int64_t d, int64_t k, int udtype, float* E, hipStream_t s) {
  const dim3 grid((unsigned)ceil_div(k, 16), (unsigned)ceil_div(k, 16));  // (the entry point keeps both below 2^16)
  const bool vec = k % (udtype == GSI_BF16 ? 8 : 4) == 0 && reinterpret_cast<uintptr_t>(U) % 16 == 0;
  if (udtype == GSI_BF16) {
    if (vec) gram_tiles<BF16, true><<<grid, kGBlock, 0, s>>>((const uint16_t*)U, d, k, E);
    else gram_tiles<BF16, false><<<grid, kGBlock, 0, s>>>((const uint16_t*)U, d, k, E);
  } else {
    if (vec) gram_tiles<F32, true><<<grid, kGBlock, 0, s>>>((const float*)U, d, k, E);
    else gram_tiles<F32, false><<<grid, kGBlock, 0, s>>>((const float*)U, d, k, E);
  }
  return hipGetLastError();
}

}  // namespace gsi
