// rows.hpp -- how the leaf-MLP kernels come by the samples of a tile: the wave's rows of the
// next tile are found and loaded while the current tile's layers run.
//
// Two sources.  From the sorted intervals (FUSED): a wave's window of 64 rows starts in a
// known interval (win); the next 64 intervals' first samples are one coalesced read, the ones
// that start inside the window mark their row, and a prefix maximum gives every row its
// interval, whose 16-byte record holds ray, position and step (centred strata; jittered ones
// would need a fifth word).  From sample records: one record per row, as the expansion or the
// rounds' selection wrote them.
//
// Writing and reading a 12-byte record per sample was 24 B of traffic for a sample of about 19
// per interval, and a launch: 315 us of an 800x800 frame, 0.6 ms of a 1920x1080 pass.  Finding
// the rows here costs about 40 vector instructions per 64 rows next to the layers' 1 100.
#pragma once

#include "internal.hpp"
#include "devcommon.hpp"

namespace amn {

// ROWS rows per wave (64, or 32 with both halves of the wave on the same rows).
template <bool FUSED, int ROWS>
struct RowFetch {
  // the next tile's rows [row0, end) of this wave; this lane's sample
  uint32_t qb, row0, end;
  uint32_t perm;
  float t, o[3], d[3];
  // in flight between the stages
  uint32_t ray, p0, st, j;
  float t0, delta;
  // ROWS = 32: 32 for the waves on the upper half of a window
  uint32_t window_shift;

  __device__ __forceinline__ void init(uint32_t leaf, int wave) {
    qb = leaf;
    window_shift = ROWS == 32 ? 32u * (uint32_t)(wave & 1) : 0u;
    row0 = end = 0;
    perm = ray = p0 = st = j = 0u;
    t = t0 = delta = 0.f;
#pragma unroll
    for (int a = 0; a < 3; ++a) o[a] = d[a] = 0.f;
  }

  // 1: which rows, and the first read.  n_iv: intervals of the pass.
  __device__ __forceinline__ void locate(const RowSource& s, const uint32_t* __restrict__ bucket_off,
                                         const uint32_t* __restrict__ tile_off, uint32_t tile, int wave, int lane,
                                         uint32_t n_iv) {
    while (tile_off[qb + 1] <= tile) ++qb;
    row0 = bucket_off[qb] + (tile - tile_off[qb]) * kMlpTileRows + (uint32_t)wave * ROWS;
    end = bucket_off[qb + 1];
    ray = 0u; perm = 0u; t = 0.f;
    if constexpr (FUSED) {
      if (row0 >= end) return;   // (a window without rows has no entry)
      p0 = s.win[4u * tile + (uint32_t)wave * ROWS / 64u];
      const uint32_t p = p0 + (uint32_t)lane;
      st = p < n_iv ? s.ssb[p] : 0xFFFFFFFFu;
    } else {
      const uint32_t row = row0 + (uint32_t)(lane & (ROWS - 1));
      if (row < end) {
        ray = s.ray[row];
        t = s.t[row];
        perm = s.perm[row];
      }
    }
  }

  // 2: FUSED: each row's interval and its record; records: the rays.  mark: 64 bytes of LDS of
  // this wave.
  __device__ __forceinline__ void fetch(const RowSource& s, uint8_t* mark, const float* __restrict__ ro,
                                        const float* __restrict__ rd, int64_t stride, int64_t r0, int lane) {
    if constexpr (FUSED) {
      if (row0 >= end) return;
      const uint32_t q0 = row0 - window_shift;   // the window's first row
      mark[lane] = 0;   // interval p0 covers the window's start
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const uint32_t at = st - q0;   // (intervals that start at or before it wrap around)
      if (at - 1u < 63u) mark[at] = (uint8_t)lane;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      int k = wave_max_incl((int)mark[lane]);
      uint32_t w = (uint32_t)lane;
      if (ROWS != 64) {
        w = window_shift + (uint32_t)(lane & (ROWS - 1));   // this lane's row in the window
        k = __shfl(k, (int)w, 64);
      }
      j = q0 + w - (uint32_t)__shfl((int)st, k, 64);
      const float4 r = *reinterpret_cast<const float4*>(s.rec + p0 + (uint32_t)k);
      t0 = r.x;
      delta = r.y;
      ray = __float_as_uint(r.z);
      perm = __float_as_uint(r.w);
    } else {
      rays(ro, rd, stride, r0);
    }
  }

  // 3: FUSED: the rays.
  __device__ __forceinline__ void gather(const float* __restrict__ ro, const float* __restrict__ rd, int64_t stride,
                                         int64_t r0) {
    if constexpr (FUSED) {
      if (row0 >= end) return;
      t = sample_t(t0, delta, j, 0.5f);
      perm += j;
      rays(ro, rd, stride, r0);
    }
  }

 private:
  __device__ __forceinline__ void rays(const float* __restrict__ ro, const float* __restrict__ rd, int64_t stride,
                                       int64_t r0) {
    const int64_t ri = r0 + ray;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      o[a] = ro[a * stride + ri];
      d[a] = rd[a * stride + ri];
    }
  }
};

}  // namespace amn
