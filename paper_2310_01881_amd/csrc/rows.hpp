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
// the rows here costs about 40 vector instructions per 64 rows next to the layers' 1 100 (the
// bf16 kernel 1.83 -> 1.87 ms for 61 M samples) as long as no read is waited for where it is
// issued; with such waits it took 2.05 ms.
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
  uint32_t ray, p0, p_ahead, st, j;
  float t0, delta;
  bool past;
  // ROWS = 32: 32 for the waves on the upper half of a window
  uint32_t window_shift;

  // leaf: of the first tile located.
  __device__ __forceinline__ void init(const RowSource& s, uint32_t leaf, uint32_t tile, int wave) {
    qb = leaf;
    p_ahead = FUSED ? s.win[4u * tile + (uint32_t)wave * ROWS / 64u] : 0u;
    window_shift = ROWS == 32 ? 32u * (uint32_t)(wave & 1) : 0u;
    row0 = end = 0;
    past = false;
    perm = ray = p0 = st = j = 0u;
    t = t0 = delta = 0.f;
#pragma unroll
    for (int a = 0; a < 3; ++a) o[a] = d[a] = 0.f;
  }

  // The stages run for every tile, the last one and windows without rows included (they load
  // something valid that nobody uses): a condition around a load would have its result copied
  // where the paths meet, which waits for it.

  // 1: which rows, and the first read.  n_iv: intervals of the pass (at least 1); tiles are
  // located in turn, up to `last` (the window's entry is read a tile ahead: the read that
  // depends on it starts without a wait).
  __device__ __forceinline__ void locate(const RowSource& s, const uint32_t* __restrict__ bucket_off,
                                         const uint32_t* __restrict__ tile_off, uint32_t tile, uint32_t last, int wave,
                                         int lane, uint32_t n_iv) {
    while (tile_off[qb + 1] <= tile) ++qb;
    row0 = bucket_off[qb] + (tile - tile_off[qb]) * kMlpTileRows + (uint32_t)wave * ROWS;
    end = bucket_off[qb + 1];
    if constexpr (FUSED) {
      p0 = min(p_ahead, n_iv - 1u);   // (a window without rows has no entry)
      p_ahead = s.win[4u * min(tile + 1, last) + (uint32_t)wave * ROWS / 64u];
      const uint32_t p = p0 + (uint32_t)lane;
      const uint32_t v = s.ssb[min(p, n_iv)];
      st = v;
      past = p >= n_iv;
    } else {
      const uint32_t row = min(row0 + (uint32_t)(lane & (ROWS - 1)), end - 1u);
      ray = s.ray[row];
      t = s.t[row];
      perm = s.perm[row];
    }
  }

  // 2: FUSED: each row's interval and its record; records: the rays.  mark: 64 bytes of LDS of
  // this wave.
  __device__ __forceinline__ void fetch(const RowSource& s, uint8_t* mark, const float* __restrict__ ro,
                                        const float* __restrict__ rd, int64_t stride, int64_t r0, int lane) {
    if constexpr (FUSED) {
      // (the compiler would share what follows with the path that skips a tile without rows, and
      // move it up to the read that st comes from)
      asm volatile("" : "+v"(st));
      const uint32_t q0 = row0 - window_shift;   // the window's first row
      mark[lane] = 0;   // interval p0 covers the window's start
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const uint32_t at = st - q0;   // (intervals that start at or before it wrap around)
      if (at - 1u < 63u && !past) mark[at] = (uint8_t)lane;
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
      t = sample_t(t0, delta, j, 0.5f);
      perm += j;
      rays(ro, rd, stride, r0);
    }
  }

  // Waits for the loads (for the path that skips a tile: where the paths meet, the layers'
  // registers would otherwise be taken for the targets of loads in flight).
  __device__ __forceinline__ void settle() const { __builtin_amdgcn_s_waitcnt(0x0F70); }   // vmcnt(0)

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
