// Device code shared by the decode-batch kernels of bf16 and of fp32 storage (gsi_tile.hip, gsi_tile_f32.hip).
#pragma once
#include "gsi_decode.h"
#include "gsi_device.h"

namespace gsi {

constexpr int kMaxTok = kMaxTileTok;  // tokens per call

// four consecutive activations at element offset i (a multiple of four) as fp32; F32: known to be
template <bool F32_ONLY>
__device__ __forceinline__ float4 load_act4(const void* p, int dtype, int64_t i) {
  if (F32_ONLY || dtype == GSI_F32) return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(p) + i);
  const uint2 b = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(p) + i);
  return float4{bf16_lo(b.x), bf16_hi(b.x), bf16_lo(b.y), bf16_hi(b.y)};
}

// |r|, |x| per token from the row blocks' shares, then the gate and the ordered list of fired tokens
// (Eq. (gate); Algorithm 1, line 4), by the NB threads of one workgroup.  NB / 32 threads share a token
// (NB / 64 beyond 32 tokens, NB / 128 beyond 64): each adds its part of the shares in order, the part sums are then added in order.
// red: NB float2, wave_count: two ints of LDS.
template <int NB>
__device__ __forceinline__ void norms_and_gate(const ProjTask& p, int B, int do_gate, float eps, float2* red,
                                               int* wave_count) {
  const int slots = B <= 32 ? 32 : B <= 64 ? 64 : kMaxTok, parts = NB / slots;
  const int t = threadIdx.x % slots, part = threadIdx.x / slots;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int per = (p.b_slabs + parts - 1) / parts;
  const int s_begin = part * per, s_end = min(p.b_slabs, s_begin + per);
  constexpr int kFlight = 16;  // requests in flight: one round trip for 128 row blocks of up to 64 tokens
  float sr = 0.f, sx = 0.f;
  const float2* src = reinterpret_cast<const float2*>(p.part_n) + min(t, B - 1);
  for (int s0 = s_begin; s0 < s_end; s0 += kFlight) {
    unsigned long long q[kFlight];  // (|r|^2, |x|^2) shares, read past the caches: other workgroups of this launch wrote them
#pragma unroll
    for (int u = 0; u < kFlight; ++u)
      q[u] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(src + (int64_t)min(s0 + u, p.b_slabs - 1) * B),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int u = 0; u < kFlight; ++u)
      if (s0 + u < s_end) { sr += __uint_as_float((unsigned)q[u]); sx += __uint_as_float((unsigned)(q[u] >> 32)); }
  }
  red[part * slots + t] = float2{sr, sx};
  __syncthreads();
  // the threads of part 0 (thread index = token) finish the job; the others only keep the barriers
  const bool head = part == 0;
  sr = red[t].x;
  sx = red[t].y;
  for (int w = 1; w < parts; ++w) {
    sr += red[w * slots + t].x;
    sx += red[w * slots + t].y;
  }
  const float rn = sqrtf(sr), xn = sqrtf(sx);
  if (head && t < B) {
    p.rnorm[t] = rn;
    p.xnorm[t] = xn;
  }
  if (!do_gate) return;  // uniform
  const bool fired = head && t < B && gate_fires(rn, xn, eps);
  if (head && t < B) p.mask[t] = fired ? 1 : 0;
  const unsigned long long ballot = __ballot(fired);
  const int rank_in_wave = __popcll(ballot & ((1ull << lane) - 1ull));
  if (wave < kMaxTok / kWave && lane == 0) wave_count[wave] = __popcll(ballot);
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int wv = 0; wv < kMaxTok / kWave; ++wv) {
    const int c = wave_count[wv];
    if (wv < wave) before += c;
    total += c;
  }
  if (fired) p.fired_idx[before + rank_in_wave] = t;
  if (threadIdx.x == 0) p.n_fired[0] = total;
}

}  // namespace gsi
