// comp.hip -- front-to-back volume rendering of each ray's samples with early ray
// termination (Section 3.1 defers the accumulation to the NeRF quadrature; Section 4.1
// uses early termination).
//
// Per ray: tau_j = sigma_j delta_j, S_j = sum_{i<j} tau_i accumulated in float32 with
// compensation (log-space transmittance), T_j = exp(-S_j), w_j = T_j * (1 - exp(-tau_j))
// via expm1, stop after the first j with T_{j+1} < eps.
#include <algorithm>

#include "internal.hpp"
#include "devcommon.hpp"

namespace amn {
namespace {

constexpr int kThreads = 256;

// Output heads and exponentials from the hardware base-2 exponential, logarithm and
// reciprocal (about 1 ulp each; the float32 result stays far inside the 1e-5 parity
// tolerance).
constexpr float kLog2e = 1.44269504f, kLn2 = 0.693147181f;
__device__ __forceinline__ float exp_neg(float x) { return __builtin_amdgcn_exp2f(-kLog2e * x); }
// softplus z = max(z, 0) + log(1 + e^-|z|), with log1p(e) = e (1 - e/2) below 2^-12
__device__ __forceinline__ float softplusf(float z) {
  const float e = exp_neg(fabsf(z));
  const float l = e < 2.44140625e-4f ? e * fmaf(-0.5f, e, 1.f) : __builtin_amdgcn_logf(1.f + e) * kLn2;
  return fmaxf(z, 0.f) + l;
}
__device__ __forceinline__ float logisticf(float z) { return __builtin_amdgcn_rcpf(1.f + exp_neg(z)); }
// 1 - e^-t for t >= 0: a quartic Taylor polynomial below 1/16, else from the exponential
__device__ __forceinline__ float one_minus_exp_neg(float t) {
  if (t < 0.0625f) return t * fmaf(t, fmaf(t, fmaf(t, -1.f / 24.f, 1.f / 6.f), -0.5f), 1.f);
  return 1.f - exp_neg(t);
}

// Unevaluated float pair hi + lo (compensated sums).
struct DF {
  float hi, lo;
};

__device__ __forceinline__ DF df_add(DF a, DF b) {
  float s = a.hi + b.hi;
  float bb = s - a.hi;
  float e = (a.hi - (s - bb)) + (b.hi - bb);   // TwoSum error of the high parts
  e += a.lo + b.lo;
  float h = s + e;
  return {h, e - (h - s)};
}

// exp(-(hi + lo)) for |lo| << 1: exp(-hi) * (1 - lo).
__device__ __forceinline__ float df_exp_neg(DF a) { return exp_neg(a.hi) * (1.f - a.lo); }

// Compensated sums of a window of 64 samples, 16 lanes at a time.  High parts are added with an
// exact TwoSum; low parts, and each TwoSum's rounding error, go into a plain running sum of low
// parts (the pair is normalised once, at the end).
__device__ __forceinline__ void df_accumulate(DF& v, float hi, float lo) {
  const float s = v.hi + hi;
  const float bb = s - v.hi;
  const float e = (v.hi - (s - bb)) + (hi - bb);
  v.lo = v.lo + lo + e;
  v.hi = s;
}

// Inclusive prefix sum over the 16 lanes of a row, not normalised (shifts by 1, 2, 4, 8; lanes
// whose source is outside the row add 0).
template <int CTRL>
__device__ __forceinline__ void df_scan_step(DF& v) {
  df_accumulate(v, dpp_or_zero<CTRL, 0xF>(v.hi), dpp_or_zero<CTRL, 0xF>(v.lo));
}
__device__ __forceinline__ DF row_scan_incl(float x) {
  DF v = {x, 0.f};
  df_scan_step<0x111>(v);
  df_scan_step<0x112>(v);
  df_scan_step<0x114>(v);
  df_scan_step<0x118>(v);
  return v;
}

// Sum over the row, in its last lane (the other lanes hold partial sums).
__device__ __forceinline__ float row_sum_last(float v) {
  v += dpp_or_zero<0x111, 0xF>(v);
  v += dpp_or_zero<0x112, 0xF>(v);
  v += dpp_or_zero<0x114, 0xF>(v);
  v += dpp_or_zero<0x118, 0xF>(v);
  return v;
}
// Sums of w * x over the row for four values x, value i's in lane 12 + i (the other lanes hold
// partial sums): pairs, fours, eights and the row are added as row_sum_last adds them, and at
// the first two levels every lane keeps half of the values.  A pair's sum is the odd lane's
// product, exact, added to the even lane's, rounded (one fused multiply-add).
__device__ __forceinline__ float row_pair2(float w_odd, float w, float x0, float x1, bool odd) {
  const float x0_odd = dpp_or_zero<0xF5, 0xF>(x0);          // quad_perm 1 1 3 3
  const float p1_even = dpp_or_zero<0xA0, 0xF>(w * x1);     // quad_perm 0 0 2 2
  return fmaf(w_odd, odd ? x1 : x0_odd, odd ? p1_even : w * x0);
}
__device__ __forceinline__ float row_sums4(float w, float a, float b, float c, float d, bool bit0, bool bit1) {
  const float w_odd = dpp_or_zero<0xF5, 0xF>(w);
  const float ab = row_pair2(w_odd, w, a, b, bit0), cd = row_pair2(w_odd, w, c, d, bit0);
  float v = (bit1 ? cd : ab) + dpp_or_zero<0x4E, 0xF>(bit1 ? ab : cd);   // quad_perm 2 3 0 1
  v += dpp_or_zero<0x124, 0xF>(v);   // row_ror:4
  v += dpp_or_zero<0x128, 0xF>(v);   // row_ror:8
  return v;
}
__device__ __forceinline__ float row_last(float v) { return dpp_or_zero<0x15F, 0xF>(v); }   // row_newbcast:15

// Four rays per wave, a row of 16 lanes each, 16 samples of every ray per step.  Lane c of a
// row handles sample base + c: tau_j, then S_j = sum_{i<j} tau_i by a compensated (float pair)
// prefix scan across the row plus the running total of earlier steps; T_j = exp(-S_j), w_j =
// T_j (1 - e^-tau_j).  Early termination: the first lane whose T_{j+1} < eps keeps its sample
// and later lanes (and steps) of its ray contribute nothing, whatever they hold: a ray's result
// depends neither on the rays beside it, which may march on, nor on what lies behind its stop.
// T_j is the neighbouring lane's T_{j+1}, so one exponential per sample serves both.
//
// Sums run over windows of 64 samples (the four steps q = 0..3 of a window) in one fixed order,
// that of a 64-lane prefix sum over rows of 16: with R_q the row's sum of step q, a window's sum
// is (R3 + R2) + (R1 + R0), and step q's prefix sums get R0 (q = 1), R1 + R0 (q = 2), or R2 and
// then R1 + R0 (q = 3) added.  Training depends on it: colours that differ in their last bit
// give gradients that do, and the optimiser, which divides by the gradients' own size, carries
// that into the bfloat16 weights.
//
// What bounds it is the latency of a ray's chain (offsets -> interval records and samples ->
// scan) and the vector work per ray.  One wave per ray (64 samples per step, a 6-step scan and
// five 6-step reductions for rays that composite 26 to 52 samples on average, most of them
// stopping in their first step) issued about three times the instructions per ray and held a
// quarter of the rays in flight: 800x800 frame 334 -> 211 us (61 M samples, 2.9 -> 4.6
// TB/s), planned 267 -> 145 us (each lane keeping sums of its own over a window took 201 and
// 140, in another order).  A step's samples are loaded two steps ahead.
//
// The ray's interval records are staged in LDS (kStage of them; the rest are read from
// memory).  UNIFORM: every interval of a ray has the same number of samples (all but planned
// intervals), so a sample's interval is a quotient; otherwise a binary search over the
// intervals' first samples.
//
// ROUND: one 64-sample window (`round`) of every ray that is still marching, the state of the
// earlier windows read from and written back to `carry`; a ray's outputs are written when it
// terminates or its last window is done.  The arithmetic of a window is the same as in the
// single pass, so a render in rounds is bit-identical to one in a single pass.
constexpr uint32_t kStage = 64;
constexpr uint32_t kRays = 4;      // per wave
constexpr uint32_t kDone = 0x80000000u;

template <bool ROUND, bool UNIFORM>
__global__ __launch_bounds__(kThreads, 8) void k_composite(
    uint32_t nr, IvSet iv, const float* __restrict__ smp_out, int64_t r0, int jitter,
    uint64_t seed, float eps, float* __restrict__ rgb, float* __restrict__ depth,
    float* __restrict__ opac, float* __restrict__ weights, uint32_t* __restrict__ ray_used,
    ChunkCounts* __restrict__ counts, CompCarry* __restrict__ carry_st, uint32_t round) {
  constexpr uint32_t kRows = kThreads / 64 * kRays;
  __shared__ float s_t0[kRows][kStage], s_delta[kRows][kStage];
  __shared__ uint32_t s_base[UNIFORM ? 1 : kRows][kStage];   // first sample, relative to the ray's
  const int lane = threadIdx.x & 63, row = threadIdx.x >> 4;
  const uint32_t c = (uint32_t)lane & 15u;
  const uint32_t r = blockIdx.x * kRows + (uint32_t)row;
  const bool live = r < nr;
  const uint32_t i0 = live ? iv.iv_off[r] : 0u, m = live ? iv.iv_off[r + 1] - i0 : 0u;
  const uint32_t s0 = live ? iv.smp_off[r] : 0u, ns = live ? iv.smp_off[r + 1] - s0 : 0u;
  uint32_t sb = 0, se = ns;                    // this launch's samples of the ray
  bool marching = live;
  DF S = {0.f, 0.f};                           // sum of tau before the current window
  // sums of the windows so far: lanes 12..15 of the row hold red, green, blue and depth in tot;
  // lane 15 holds the opacity
  float tot = 0.f, tot_a = 0.f;
  if (ROUND) {
    sb = 64u * round;
    if (sb >= ns && !(ns == 0 && round == 0)) marching = false;   // finished in an earlier window
    if (marching && round > 0) {
      const CompCarry cy = carry_st[r];
      if (cy.state & kDone) marching = false;
      S = {cy.s_hi, cy.s_lo};
      tot = (c & 2u) ? ((c & 1u) ? cy.dep : cy.cb) : ((c & 1u) ? cy.cg : cy.cr);
      tot_a = cy.acc;
    }
    se = sb + 64u < ns ? sb + 64u : ns;
  }
  if (__ballot(marching) == 0) return;
  bool done = !marching;
  auto load = [&](uint32_t j) {
    float4 z = {0.f, 0.f, 0.f, 0.f};
    if (!done && j < se) z = *reinterpret_cast<const float4*>(smp_out + 4 * (uint64_t)(s0 + j));
    return z;
  };
  float4 z0 = load(sb + c), z1 = load(sb + 16u + c);
  // samples per interval (UNIFORM) and floor(x / n) = umulhi(x, ceil(2^32 / n)), x < 2^16
  const uint32_t n = UNIFORM && m > 0 ? ns / m : 1u;
  const uint32_t m32 = n > 1u ? 0xFFFFFFFFu / n + 1u : 0u;
  if (marching)
    for (uint32_t k = c; k < m && k < kStage; k += 16u) {
      s_t0[row][k] = iv.t0[i0 + k];
      s_delta[row][k] = iv.dt[i0 + k] / (float)(UNIFORM ? n : key_n(iv.key[i0 + k]));
      if (!UNIFORM) s_base[row][k] = iv.base[i0 + k] - s0;
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const uint64_t wbase = counts->smp_global + s0;
  uint32_t used = ns;   // samples composited: up to and including the stop sample
  uint32_t next = sb;   // first sample after the last step processed
  bool stopped = false;
  const bool bit0 = (c & 1u) != 0, bit1 = (c & 2u) != 0;
  float sum = 0.f, sum_a = 0.f, sum01 = 0.f, sum01_a = 0.f;   // of this pair of steps; of the window's first pair
  DF scan_row = {0.f, 0.f}, scan01 = {0.f, 0.f};   // R_q of the optical depth; R1 + R0 (not normalised)
  float Tlast = 0.f;                               // T after the step before
  uint32_t q = 0;                                  // step in the window
  for (uint32_t base = sb; __ballot(!done && base < se) != 0; base += 16u, q = (q + 1u) & 3u) {
    const uint32_t j = base + c;
    const float4 z = z0;
    z0 = z1;
    z1 = load(j + 32u);
    const bool valid = !done && j < se;
    uint32_t k = 0, jj = 0;
    float t0 = 0.f, delta = 0.f;
    if (valid) {
      if (UNIFORM) {
        k = n > 1u ? __umulhi(j, m32) : j;
        jj = j - k * n;
        if (k < kStage) {
          t0 = s_t0[row][k];
          delta = s_delta[row][k];
        } else {
          t0 = iv.t0[i0 + k];
          delta = iv.dt[i0 + k] / (float)n;
        }
      } else if (m <= kStage) {
        uint32_t lo = 0, hi = m;
        while (hi - lo > 1) {
          const uint32_t mid = (lo + hi) >> 1;
          if (s_base[row][mid] <= j) lo = mid; else hi = mid;
        }
        k = lo;
        jj = j - s_base[row][k];
        t0 = s_t0[row][k];
        delta = s_delta[row][k];
      } else {
        const uint32_t i = find_interval(iv.base, i0, i0 + m, s0 + j);
        k = i - i0;
        jj = s0 + j - iv.base[i];
        t0 = iv.t0[i];
        delta = iv.dt[i] / (float)key_n(iv.key[i]);
      }
    }
    const float u = jitter ? stratum_u(1, seed, (uint64_t)(r0 + r), k) : 0.5f;
    const float t = sample_t(t0, delta, jj, u);
    const float tau = valid ? softplusf(z.x) * delta : 0.f;   // sigma = softplus, rgb = logistic
    // inclusive compensated scan of tau over the window so far; exclusive = shifted by one lane
    DF v = row_scan_incl(tau);
    const DF row_v = {row_last(v.hi), row_last(v.lo)};
    if (q & 1u) df_accumulate(v, scan_row.hi, scan_row.lo);
    if (q & 2u) df_accumulate(v, scan01.hi, scan01.lo);
    if (q == 1u) scan01 = {row_last(v.hi), row_last(v.lo)};
    scan_row = row_v;
    const float h = v.hi + v.lo;
    const DF Sn = df_add(S, {h, v.lo - (h - v.hi)});
    const float Tn = df_exp_neg(Sn);                     // T_{j+1}
    if (q == 0u) Tlast = df_exp_neg(S);
    const float Tsh = dpp_or_zero<0x111, 0xF>(Tn);       // row_shr:1: lane c - 1's T_{j+1}
    const float T = c == 0 ? Tlast : Tsh;
    Tlast = row_last(Tn);
    float w = valid ? T * one_minus_exp_neg(tau) : 0.f;
    const bool stop = valid && eps > 0.f && Tn < eps;
    const uint32_t stops = (uint32_t)(__ballot(stop) >> (lane & 48)) & 0xFFFFu;
    const bool now = stops != 0;
    const uint32_t first = (uint32_t)__ffs((int)stops) - 1u;
    const bool counts_in = valid && !(now && c > first);
    if (!counts_in) w = 0.f;
    // (selected, not multiplied by that 0: a NaN or an infinity behind the stop must not count)
    const float x = row_sums4(w, counts_in ? logisticf(z.y) : 0.f, counts_in ? logisticf(z.z) : 0.f,
                              counts_in ? logisticf(z.w) : 0.f, counts_in ? t : 0.f, bit0, bit1);
    const float xa = row_sum_last(w);
    if (q & 1u) {
      sum = x + sum;
      sum_a = xa + sum_a;
    } else {
      sum = x;
      sum_a = xa;
    }
    if (weights && valid) weights[wbase + j] = w;
    if (!done) next = base + 16u;
    if (now) {
      used = base + first + 1u;
      stopped = true;
      done = true;
    }
    if (q == 1u) {
      sum01 = sum;
      sum01_a = sum_a;
      sum = sum_a = 0.f;
    }
    if (q == 3u) {   // the window is complete
      S = {row_last(Sn.hi), row_last(Sn.lo)};
      tot += sum + sum01;
      tot_a += sum_a + sum01_a;
      sum = sum_a = sum01 = sum01_a = 0.f;
    }
  }
  tot += sum + sum01;   // what is left of the last window
  tot_a += sum_a + sum01_a;
  const bool odd_value = !isfinite(tot) || (c == 15u && !isfinite(tot_a));
  const uint32_t bad = (uint32_t)(__ballot(odd_value) >> (lane & 48)) & 0xF000u;   // of this ray
  if (!marching) return;
  // a ray that stopped has weight 0 on every later sample
  if (weights && stopped)
    for (uint32_t j = next + c; j < ns; j += 16) weights[wbase + j] = 0.f;
  if (c < 12u) return;
  const uint32_t i = c - 12u;
  if (ROUND && !stopped && se < ns) {
    CompCarry* cy = carry_st + r;
    (&cy->cr)[i] = tot;
    if (i == 3u) {
      cy->s_hi = S.hi;
      cy->s_lo = S.lo;
      cy->acc = tot_a;
      cy->state = 0u;
    }
    return;
  }
  if (i < 3u) {
    rgb[3 * (uint64_t)(r0 + r) + i] = tot;
    return;
  }
  if (ROUND) carry_st[r].state = kDone;
  ray_used[r] = used;
  if (depth) depth[r0 + r] = tot;
  if (opac) opac[r0 + r] = tot_a;
  if (bad) atomicAdd(reinterpret_cast<unsigned long long*>(&counts->nonfinite), 1ull);
}

// End of a chunk: counts->composited += sum of ray_used[0, nr) (block sums in a fixed order, one
// integer atomic per block), and the chunk's totals are recorded for the host, the samples of the
// sorted intervals checked against the rays' offsets, and the global sample base advanced.  (As
// two launches 1.4 us more a pass: a 64x64 render of a small scene 49.3 -> 47.8 us.)
__global__ __launch_bounds__(kThreads) void k_chunk_finish(uint32_t nr, const uint32_t* __restrict__ ray_used,
                                                           ChunkCounts* __restrict__ counts, const uint32_t* smp_total,
                                                           const uint32_t* iv_total, const uint32_t* plain_total,
                                                           int rounds) {
  __shared__ uint32_t sh[kThreads / 64];
  uint32_t s = 0;
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < nr; i += gridDim.x * kThreads) s += ray_used[i];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x != 0) return;
  uint64_t t = 0;
  for (int w = 0; w < kThreads / 64; ++w) t += sh[w];
  if (t) atomicAdd(reinterpret_cast<unsigned long long*>(&counts->composited), (unsigned long long)t);
  if (blockIdx.x != 0) return;
  const uint32_t n = *smp_total;
  if (!rounds) counts->evaluated += n;   // (in rounds: added by each round's selection)
  counts->unreached += n > counts->n_smp ? n - counts->n_smp : counts->n_smp - n;
  counts->smp_global += n;
  counts->iv_global += *iv_total;
  counts->plain_smp += *plain_total;
}

// Adds another lane's running totals into the first lane's counters.
__global__ void k_counts_merge(ChunkCounts* a, const ChunkCounts* b) {
  if (threadIdx.x != 0) return;
  a->smp_global += b->smp_global;
  a->iv_global += b->iv_global;
  a->nonfinite += b->nonfinite;
  a->fallback += b->fallback;
  a->plain_smp += b->plain_smp;
  a->unreached += b->unreached;
  a->composited += b->composited;
  a->evaluated += b->evaluated;
}

__global__ __launch_bounds__(kThreads) void k_pass_begin(ChunkCounts* counts, int reset, uint64_t* __restrict__ state,
                                                         uint64_t words) {
  if (reset && blockIdx.x == 0 && threadIdx.x == 0) {
    ChunkCounts z = {};
    *counts = z;
  }
  for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < words; i += (uint64_t)gridDim.x * kThreads)
    state[i] = 0ull;
}

}  // namespace

hipError_t launch_composite(uint32_t nr, const IvSet& iv, bool uniform, const float* smp_out, int64_t r0,
                            int jitter, uint64_t seed, float ert_eps, float* rgb, float* depth,
                            float* opac, float* weights, uint32_t* ray_used, ChunkCounts* counts,
                            hipStream_t st) {
  if (nr == 0) return hipSuccess;
  const uint32_t rays = kThreads / 64 * kRays;
  hipLaunchKernelGGL((uniform ? k_composite<false, true> : k_composite<false, false>), dim3((nr + rays - 1) / rays),
                     dim3(kThreads), 0, st, nr, iv, smp_out, r0, jitter, seed, ert_eps, rgb, depth, opac, weights,
                     ray_used, counts, nullptr, 0u);
  return hipGetLastError();
}

hipError_t launch_composite_round(uint32_t nr, const IvSet& iv, bool uniform, const float* smp_out, int64_t r0,
                                  int jitter, uint64_t seed, float ert_eps, float* rgb, float* depth, float* opac,
                                  float* weights, uint32_t* ray_used, ChunkCounts* counts, CompCarry* carry,
                                  uint32_t round, hipStream_t st) {
  if (nr == 0) return hipSuccess;
  const uint32_t rays = kThreads / 64 * kRays;
  hipLaunchKernelGGL((uniform ? k_composite<true, true> : k_composite<true, false>), dim3((nr + rays - 1) / rays),
                     dim3(kThreads), 0, st, nr, iv, smp_out, r0, jitter, seed, ert_eps, rgb, depth, opac, weights,
                     ray_used, counts, carry, round);
  return hipGetLastError();
}

hipError_t launch_chunk_finish(uint32_t nr, const uint32_t* ray_used, ChunkCounts* counts,
                               const uint32_t* smp_off_total, const uint32_t* iv_off_total,
                               const uint32_t* plain_smp_total, int rounds, hipStream_t st) {
  const uint32_t grid = std::max(1u, std::min<uint32_t>(256u, (nr + 4 * kThreads - 1) / (4 * kThreads)));
  hipLaunchKernelGGL(k_chunk_finish, dim3(grid), dim3(kThreads), 0, st, nr, ray_used, counts, smp_off_total,
                     iv_off_total, plain_smp_total, rounds);
  return hipGetLastError();
}

hipError_t launch_counts_merge(ChunkCounts* a, const ChunkCounts* b, hipStream_t st) {
  hipLaunchKernelGGL(k_counts_merge, dim3(1), dim3(64), 0, st, a, b);
  return hipGetLastError();
}

hipError_t launch_pass_begin(ChunkCounts* counts, bool reset, uint64_t* state, uint64_t words, hipStream_t st) {
  const uint64_t blocks = std::min<uint64_t>(256u, words / (4 * kThreads) + 1);
  hipLaunchKernelGGL(k_pass_begin, dim3((uint32_t)blocks), dim3(kThreads), 0, st, counts, reset ? 1 : 0, state, words);
  return hipGetLastError();
}

}  // namespace amn
