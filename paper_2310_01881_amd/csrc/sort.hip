// sort.hip -- stable sort of samples by leaf slot and bucket compaction (Section 3.5:
// samples are sorted with their ray id and node id, then inferred per node).
//
// All samples of one leaf interval share its slot and are contiguous in ray-major order,
// so the stable sort of samples equals the stable sort of intervals, each expanded into
// its samples in place.  The sort therefore runs on intervals (about S_max / n fewer keys
// than samples):
//   hist    one wave per segment of `seg` consecutive intervals: LDS histogram of slots
//           (intervals and samples in one word), written column-wise into a [slot][segment]
//           matrix (row length = the chunk's actual segment count, so the matrix and its scan
//           scale with the intervals present, and there is a segment per wave across the
//           machine);
//   scan    exclusive scan of that matrix in slot-major order = the first sorted position
//           and the first sorted sample of (slot, segment), hence the leaves' buckets and tiles;
//   scatter one wave per segment again, 64 intervals at a time: lanes holding the same
//           slot find each other with one ballot per key bit; rank = earlier lanes of the
//           same slot, on top of a per-slot running count in LDS -> stable positions; the
//           samples before an interval likewise (one ballot per bit of the sample count), so
//           its place among the sorted samples needs no scan of its own.  Each interval's
//           16-byte record goes to its sorted position, and the 64-row windows of the MLP
//           tiles that start inside it get its position;
//   expand  (where one record per sample is needed: rounds, the backward pass, calibration,
//           inspection) each sorted interval writes its samples' records.
#include <algorithm>

#include "internal.hpp"
#include "devcommon.hpp"

namespace amn {
namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr uint32_t kMaxGrid = 16384;

// Block numbers dealt so that each of the eight dies (blocks go to them in turn) has a run of
// consecutive ones: k in [0, 8 ceil(n / 8)) -> number, n or more for none.  Each die has an L2
// of its own, and what neighbouring segments write (matrix entries, a leaf's places) is
// neighbouring too: random rays of a training batch (1.7 M intervals) scatter in 39 us instead
// of 84, and the count matrix of a 1.4 M-ray pass takes 134 instead of 173.
constexpr uint32_t kDies = 8;
__device__ __forceinline__ uint32_t die_runs(uint32_t n) { return (n + kDies - 1) / kDies; }
__device__ __forceinline__ uint32_t die_block(uint32_t k, uint32_t runs) { return (k & (kDies - 1)) * runs + k / kDies; }

// A word of the matrix and of the running counts: intervals << 20 | samples (a segment holds
// less than 4096 intervals of at most 255 samples).
__global__ __launch_bounds__(kThreads) void k_sort_hist(const uint32_t* __restrict__ iv_key,
                                                        const uint32_t* __restrict__ n_iv_dev,
                                                        uint32_t seg, uint32_t n_leaves,
                                                        uint32_t* __restrict__ mat) {
  extern __shared__ uint32_t sh[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  uint32_t* hist = sh + wave * n_leaves;
  const uint32_t n_iv = *n_iv_dev;
  const uint32_t nseg = (n_iv + seg - 1) / seg;
  const uint32_t runs = die_runs((nseg + waves - 1) / waves);
  for (uint32_t k = blockIdx.x; k < kDies * runs; k += gridDim.x) {
    const uint32_t s = die_block(k, runs) * waves + wave;
    if (s >= nseg) continue;
    for (uint32_t b = lane; b < n_leaves; b += 64) hist[b] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    uint64_t begin = (uint64_t)s * seg;
    uint64_t end = begin + seg < n_iv ? begin + seg : n_iv;
    for (uint64_t i = begin + lane; i < end; i += 64) {
      const uint32_t key = iv_key[i];
      atomicAdd(&hist[key_slot(key)], (1u << 20) | key_n(key));
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (uint32_t b = lane; b < n_leaves; b += 64) mat[(uint64_t)b * nseg + s] = hist[b];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Set bits of `mask` below this lane.
__device__ __forceinline__ uint32_t count_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// REC: the interval records are written too; WIN: and the MLP's windows.
template <bool REC, bool WIN>
__global__ __launch_bounds__(kThreads) void k_sort_scatter(IvSet iv, uint32_t seg, uint32_t n_leaves,
                                                           uint32_t key_bits, SortBufs out) {
  extern __shared__ uint32_t sh[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  uint32_t* run = sh + wave * n_leaves;   // the segment's intervals and samples of each slot so far
  const uint32_t n_iv = *iv.n_iv_dev;
  const uint32_t nseg = (n_iv + seg - 1) / seg;
  const uint32_t runs = die_runs((nseg + waves - 1) / waves);
  for (uint32_t k = blockIdx.x; k < kDies * runs; k += gridDim.x) {
    const uint32_t s = die_block(k, runs) * waves + wave;
    if (s >= nseg) continue;
    for (uint32_t b = lane; b < n_leaves; b += 64) run[b] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    uint64_t begin = (uint64_t)s * seg;
    uint64_t end = begin + seg < n_iv ? begin + seg : n_iv;
    // The next 64 intervals are read while these are placed (past the end the last one again):
    // key, matrix entries and records were three waits a turn for the eight turns of a wave
    // (800x800 frame, 4.4 M intervals: 104 -> 90 us; 64x64 tile 17 -> 13.5).
    uint32_t nx_key, nx_ray = 0, nx_base = 0;
    float nx_t0 = 0.f, nx_dt = 0.f;
    auto read = [&](uint64_t c) {
      const uint64_t i = c + lane < end ? c + lane : end - 1;
      nx_key = iv.key[i];
      if (REC) {
        nx_t0 = iv.t0[i];
        nx_dt = iv.dt[i];
        nx_ray = iv.ray[i];
        nx_base = iv.base[i];
      }
    };
    read(begin);
    for (uint64_t c = begin; c < end; c += 64) {
      const uint64_t i = c + lane;
      const bool valid = i < end;
      const uint32_t key = nx_key, ray = nx_ray, base = nx_base;
      const float t0 = nx_t0, dt = nx_dt;
      const uint32_t slot = key_slot(key), n = valid ? key_n(key) : 0u;
      uint32_t pos = out.mat[(uint64_t)slot * nseg + s], smp = out.mat_smp[(uint64_t)slot * nseg + s];
      uint32_t first = 0, tile = 0;
      if (WIN) {
        first = out.bucket_off[slot];
        tile = out.tile_off[slot];
      }
      read(c + 64);
      // lanes with the same slot: intersect one ballot per key bit
      uint64_t peers = __ballot(valid);
      for (uint32_t bit = 0; bit < key_bits; ++bit) {
        const uint64_t ones = __ballot(valid && ((slot >> bit) & 1u));
        peers &= ((slot >> bit) & 1u) ? ones : ~ones;
      }
      const uint32_t rank = count_below(peers);
      uint32_t before = 0;   // samples of the earlier lanes of this slot
#pragma unroll
      for (uint32_t bit = 0; bit < 8; ++bit) before += count_below(peers & __ballot((n >> bit) & 1u)) << bit;
      const uint32_t had = valid ? run[slot] : 0u;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // the highest lane of each group advances that slot's counts
      if (valid && (peers >> lane) == 1ull) run[slot] = had + ((rank + 1) << 20) + before + n;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (valid) {
        pos += (had >> 20) + rank;
        smp += (had & 0xFFFFFu) + before;
        out.sidx[pos] = (uint32_t)i;
        out.ssb[pos] = smp;
        if (REC) {
          *reinterpret_cast<float4*>(out.rec + pos) =
              make_float4(t0, dt / (float)n, __uint_as_float(ray), __uint_as_float(base));
          // the windows (64 rows of the leaf's bucket) whose first row is one of these samples
          if (WIN) {
            const uint32_t at = smp - first;
            for (uint32_t w = (at + 63u) / 64u; 64u * w < at + n; ++w) out.win[4u * tile + w] = pos;
          }
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// One block: leaf bucket offsets in sorted samples and MLP tile offsets.
__global__ __launch_bounds__(1024) void k_bucket_tiles(uint32_t seg, uint32_t n_leaves, SortBufs out,
                                                       const uint32_t* __restrict__ n_iv_dev, ChunkCounts* counts) {
  __shared__ uint32_t sh[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t n_iv = *n_iv_dev;
  const uint32_t nseg = (n_iv + seg - 1) / seg;
  const uint32_t n_smp = out.mat_smp[(uint64_t)n_leaves * nseg];
  uint32_t carry = 0;
  for (uint32_t c = 0; c < n_leaves; c += 1024) {
    uint32_t b = c + threadIdx.x;
    uint32_t lo = 0, hi = 0;
    if (b < n_leaves) {
      lo = out.mat_smp[(uint64_t)b * nseg];
      hi = out.mat_smp[(uint64_t)(b + 1) * nseg];
      out.bucket_off[b] = lo;
    }
    uint32_t nt = (hi - lo + kMlpTileRows - 1) / kMlpTileRows;
    uint32_t x = nt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      uint32_t y = __shfl_up(x, off, 64);
      if (lane >= off) x += y;
    }
    if (lane == 63) sh[wave] = x;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
    for (int w = 0; w < 16; ++w) {
      uint32_t s = sh[w];
      if (w < wave) pre += s;
      tot += s;
    }
    if (b < n_leaves) out.tile_off[b] = carry + pre + x - nt;
    carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out.bucket_off[n_leaves] = n_smp;
    out.tile_off[n_leaves] = carry;
    out.ssb[n_iv] = n_smp;
    counts->n_iv = n_iv;
    counts->n_smp = n_smp;
    counts->n_tiles = carry;
    *out.unexpanded = out.rec != nullptr;
  }
}

// One block per 256 consecutive sorted intervals: their records go to LDS, then each wave
// writes windows of 64 consecutive sorted samples (coalesced).  A sample's interval is
// found without a search: the intervals starting inside the window mark their first
// lane in a per-wave LDS row, and a prefix maximum over the row (seeded with the last
// interval of the previous window) gives every lane the latest interval started at or
// before it.
//
// REC: from the intervals' sorted records.  Otherwise each of five arrays is read at a sorted
// interval's own place, a whole sector for four bytes: 184 us for the 23 M samples (1.7 M
// intervals) of a training batch against 67, with the records' writing 39 -> 81 in the scatter.
template <bool REC>
__global__ __launch_bounds__(kThreads) void k_expand(
    const uint32_t* __restrict__ sidx, const SortRec* __restrict__ rec, const uint32_t* __restrict__ ssb, IvSet iv,
    int64_t r0, int jitter, uint64_t seed, uint32_t* __restrict__ srec_ray, float* __restrict__ srec_t,
    uint32_t* __restrict__ perm, const uint32_t* __restrict__ if_unexpanded) {
  __shared__ uint32_t sh_base[kThreads + 1];
  __shared__ uint32_t sh_ray[kThreads], sh_rm[kThreads];
  __shared__ float sh_t0[kThreads], sh_delta[kThreads], sh_u[kThreads];
  __shared__ int sh_mark[kWaves][64];
  if (if_unexpanded && *if_unexpanded == 0u) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t n_iv = *iv.n_iv_dev;
  const uint32_t n_groups = (n_iv + kThreads - 1) / kThreads;
  for (uint32_t grp = blockIdx.x; grp < n_groups; grp += gridDim.x) {
    const uint32_t p0 = grp * kThreads;
    const uint32_t cnt = n_iv - p0 < (uint32_t)kThreads ? n_iv - p0 : (uint32_t)kThreads;
    const uint32_t p = p0 + threadIdx.x;
    if (REC && threadIdx.x < cnt) {
      const float4 r = *reinterpret_cast<const float4*>(rec + p);
      sh_base[threadIdx.x] = ssb[p];
      sh_ray[threadIdx.x] = __float_as_uint(r.z);
      sh_rm[threadIdx.x] = __float_as_uint(r.w);
      sh_t0[threadIdx.x] = r.x;
      sh_delta[threadIdx.x] = r.y;
      sh_u[threadIdx.x] = 0.5f;
    } else if (threadIdx.x < cnt) {
      uint32_t i = sidx[p];
      uint32_t ray = iv.ray[i];
      uint32_t n = key_n(iv.key[i]);
      uint32_t k = i - iv.iv_off[ray];
      sh_base[threadIdx.x] = ssb[p];
      sh_ray[threadIdx.x] = ray;
      sh_rm[threadIdx.x] = iv.base[i];   // ray-major index of the first sample
      sh_t0[threadIdx.x] = iv.t0[i];
      sh_delta[threadIdx.x] = iv.dt[i] / (float)n;
      sh_u[threadIdx.x] = stratum_u(jitter, seed, (uint64_t)(r0 + ray), k);
    }
    if (threadIdx.x == 0) sh_base[cnt] = ssb[p0 + cnt];
    __syncthreads();
    const uint32_t q0 = sh_base[0], q1 = sh_base[cnt];
    // this lane's view of the staged intervals' first samples (intervals lane + 64 c)
    uint32_t st[kWaves];
#pragma unroll
    for (int c = 0; c < kWaves; ++c) {
      const uint32_t a = (uint32_t)lane + 64u * c;
      st[c] = a < cnt ? sh_base[a] : 0xFFFFFFFFu;
    }
    // windows of 64 samples: wave w takes windows w, w + 4, ...; the interval covering a
    // window's first sample is the last one starting at or before it
    for (uint32_t qw = q0 + 64u * wave; qw < q1; qw += 64u * kWaves) {
      sh_mark[wave][lane] = -1;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      int before = 0;   // intervals starting at or before qw (at least interval 0 does)
#pragma unroll
      for (int c = 0; c < kWaves; ++c) {
        const uint32_t a = (uint32_t)lane + 64u * c;
        if (st[c] != 0xFFFFFFFFu && st[c] >= qw && st[c] < qw + 64u) sh_mark[wave][st[c] - qw] = (int)a;
        if (st[c] <= qw) before = max(before, (int)a);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int first = wave_max_incl(before);                       // lane 63 holds the maximum
      const int seed_iv = __builtin_amdgcn_readlane(first, 63);
      const int lo = max(wave_max_incl(sh_mark[wave][lane]), seed_iv);
      const uint32_t q = qw + (uint32_t)lane;
      if (q < q1) {
        const uint32_t j = q - sh_base[lo];
        srec_ray[q] = sh_ray[lo];
        srec_t[q] = sample_t(sh_t0[lo], sh_delta[lo], j, sh_u[lo]);
        perm[q] = sh_rm[lo] + j;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
  }
}

}  // namespace

SortPlan make_sort_plan(uint64_t n_iv_max, uint32_t n_leaves, bool small) {
  SortPlan p;
  p.n_leaves = n_leaves;
  uint32_t bits = 0;
  while ((1u << bits) < n_leaves) ++bits;
  p.key_bits = bits;
  // a segment per wave, of 512 intervals, or 64 where few intervals would otherwise leave
  // most of the chip without a segment (2^18 intervals make 512 segments of 512); at least as
  // many intervals per segment as slots, so the count matrix (n_leaves x segments) has no more
  // entries than there are intervals; below 4096, which the packed counts allow
  uint64_t seg = small && n_iv_max <= (1u << 18) ? 64 : 512;
  seg = std::max<uint64_t>(seg, ((uint64_t)n_leaves + 63) / 64 * 64);
  p.seg = (uint32_t)std::min<uint64_t>(seg, 4032);
  p.nseg_max = (uint32_t)((n_iv_max + p.seg - 1) / p.seg);
  if (p.nseg_max == 0) p.nseg_max = 1;
  return p;
}

// Waves per block: a wave's counts take 4 bytes per slot of LDS, so with many slots a block is
// one wave (16 KiB at 4096: ten per compute unit against two blocks of four).
static int sort_waves(const SortPlan& p) { return p.n_leaves > 1024 ? 1 : kWaves; }

hipError_t launch_sort_hist(const SortPlan& p, const uint32_t* iv_key, const uint32_t* n_iv_dev,
                            uint32_t* mat, hipStream_t st) {
  const uint32_t w = (uint32_t)sort_waves(p);
  const uint32_t grid = std::min<uint32_t>(((p.nseg_max + w - 1) / w + kDies - 1) / kDies * kDies, kMaxGrid);
  hipLaunchKernelGGL(k_sort_hist, dim3(grid), dim3(64 * w), sizeof(uint32_t) * w * p.n_leaves, st, iv_key, n_iv_dev,
                     p.seg, p.n_leaves, mat);
  return hipGetLastError();
}

hipError_t launch_sort_scatter(const SortPlan& p, const SortBufs& b, const IvSet& iv, hipStream_t st) {
  const uint32_t w = (uint32_t)sort_waves(p);
  const uint32_t grid = std::min<uint32_t>(((p.nseg_max + w - 1) / w + kDies - 1) / kDies * kDies, kMaxGrid);
  auto kern = !b.rec ? k_sort_scatter<false, false> : (b.win ? k_sort_scatter<true, true> : k_sort_scatter<true, false>);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * w), sizeof(uint32_t) * w * p.n_leaves, st, iv, p.seg, p.n_leaves,
                     p.key_bits, b);
  return hipGetLastError();
}

hipError_t launch_bucket_tiles(const SortPlan& p, const SortBufs& b, const uint32_t* n_iv_dev, ChunkCounts* counts,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_bucket_tiles, dim3(1), dim3(1024), 0, st, p.seg, p.n_leaves, b, n_iv_dev, counts);
  return hipGetLastError();
}

hipError_t launch_expand(const uint32_t* sidx, const SortRec* rec, const uint32_t* ssb, const IvSet& iv, int64_t r0,
                         int jitter, uint64_t seed, uint32_t* srec_ray, float* srec_t, uint32_t* perm,
                         const uint32_t* if_unexpanded, hipStream_t st) {
  hipLaunchKernelGGL((rec ? k_expand<true> : k_expand<false>), dim3(4096), dim3(kThreads), 0, st, sidx, rec, ssb, iv, r0,
                     jitter, seed, srec_ray, srec_t, perm, if_unexpanded);
  return hipGetLastError();
}

}  // namespace amn
