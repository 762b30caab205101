// trav.hip -- ray / KD-tree traversal producing front-to-back leaf intervals
// (Section 3.5, Algorithm 1: Traverse), one lane per ray.
//
// Interval endpoints are carried as unevaluated float pairs (hi + lo): the plane
// crossing t = (s - o) / d is formed with an exact TwoSum of the numerator and an
// FMA-exact remainder of the division, so endpoints agree with a float64 evaluation to
// about 2^-46 relative.  Descent decisions therefore match a float64 traversal except on
// rays that graze a split edge, and interval lengths (which weight densities in the
// quadrature) keep float32 relative accuracy even far along the ray.
//
// The walk is a serial chain per ray (node -> crossing -> next node), so its latency is
// what a small launch waits for and its instruction count what a large one does.  The
// crossing therefore multiplies by a reciprocal taken once per ray and axis, with the same
// remainder step as a division (the pair keeps its accuracy whatever the quotient's last
// bit), both children of a node are read while its crossing is computed, and the side of the
// plane and the ray's component are chosen without branches.  4096 rays x 20 leaves of a
// 512-leaf tree, one traversal: 54 -> 36 us.
#include <algorithm>

#include <atomic>

#include "internal.hpp"
#include "devcommon.hpp"

namespace amn {
namespace {

struct DF {
  float hi, lo;
};

__device__ __forceinline__ DF two_sum(float a, float b) {
  float s = a + b;
  float bb = s - a;
  float e = (a - (s - bb)) + (b - bb);
  return {s, e};
}

// (s - o) / d as a normalised pair, inv the correctly rounded 1 / d: the quotient's
// estimate q0 is within 2 ulp, the fused remainder of it is exact to one more rounding, and
// the correction q1 carries the pair to about 2^-46 relative.  (No contraction: h - q0 must
// see the rounded product q0.)
__device__ __forceinline__ DF plane_t(float s, float o, float d, float inv) {
#pragma clang fp contract(off)
  DF num = two_sum(s, -o);
  float q0 = num.hi * inv;
  float r = fmaf(-q0, d, num.hi);
  r += num.lo;
  float q1 = r * inv;
  float h = q0 + q1;
  float l = q1 - (h - q0);
  return {h, l};
}

// The same by division, for directions with a component so small that 1 / d overflows.
__device__ __forceinline__ DF plane_t_div(float s, float o, float d) {
  DF num = two_sum(s, -o);
  float q0 = num.hi / d;
  float r = fmaf(-q0, d, num.hi);
  r += num.lo;
  float q1 = r / d;
  float h = q0 + q1;
  float l = q1 - (h - q0);
  return {h, l};
}

// (bitwise: three compares and two mask operations, no branch)
__device__ __forceinline__ bool df_lt(DF a, DF b) { return (a.hi < b.hi) | ((a.hi == b.hi) & (a.lo < b.lo)); }

constexpr int kBlock = 256;
// LDS per block: the node table (when staged), then the traversal stack of `stack_n` =
// tree depth + 1 8-byte entries per thread, strided by kBlock (a wave's entries of one level
// are consecutive): the node index (16 bits) packed with the exit parameter's low part
// rounded to bfloat16 (the pair then still carries about 2^-32 relative precision, far below
// the 1e-6 perturbation under which node ids are compared), and the exit parameter's high
// part.
constexpr int kLdsNodes = 2048;  // node tables up to this size are staged in LDS per block

// Component a of a vector as two selects.  (The axis differs from lane to lane, so a branch on
// it never pays; the components are scalars because an indexed array would go to scratch.)
struct V3 {
  float x, y, z;
};
__device__ __forceinline__ float axis_val(V3 v, int a) {
  const float yz = __builtin_unpredictable(a == 1) ? v.y : v.z;
  return __builtin_unpredictable(a == 0) ? v.x : yz;
}

// A node in one 8-byte read (both tables are 8-byte aligned).
__device__ __forceinline__ DevNode load_node(const DevNode* nodes, int i) {
  const uint2 w = reinterpret_cast<const uint2*>(nodes)[i];
  return {__uint_as_float(w.x), (int32_t)w.y};
}

// Hierarchical sampling (HCheck): the descent stops at an inner node when the ray enters
// it farther than the node's stopping distance t_stop = size / footprint (size: the node's
// longest side; footprint: the caller's sample footprint per unit distance), and the node's
// own MLP then takes the ray's whole segment in it.  Both the decision (float32 entry
// parameter against float32 t_stop) and t_stop (one correctly rounded float32 division)
// are fixed to the bit.  Two views of the per-node data: staged in LDS as (t_stop, slot)
// pairs, or read from memory with t_stop formed on the fly.
struct AhsNone {
  __device__ float tstop(int) const { return __builtin_inff(); }
  __device__ uint32_t slot(int) const { return 0u; }
};
struct AhsLds {
  const float2* p;
  __device__ float tstop(int i) const { return p[i].x; }
  __device__ uint32_t slot(int i) const { return __builtin_bit_cast(uint32_t, p[i].y); }
};
struct AhsMem {
  const DevNodeAhs* p;
  float footprint;
  __device__ float tstop(int i) const { return __fdiv_rn(p[i].size, footprint); }
  __device__ uint32_t slot(int i) const { return p[i].slot; }
};

// Traverses one ray.  EMIT = false: returns the interval count, stopping once it exceeds
// cap.  EMIT = true: writes the first `cap` intervals through the output pointers.  AHS:
// stop the descent by HCheck, and key intervals by the node's preorder slot.
__device__ __forceinline__ uint32_t push_word(int node, float lo) {
  return (uint32_t)node | ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)lo) << 16);
}
__device__ __forceinline__ float word_lo(uint32_t w) { return (float)__builtin_bit_cast(__bf16, (uint16_t)(w >> 16)); }

// TINY: crossings by division (see plane_t_div).
template <bool EMIT, bool AHS, bool TINY, typename Ahs, typename Put>
__device__ int traverse_one(const DevNode* nodes, const Ahs ahs, const V3 o, const V3 dir, int cap, uint32_t n_per,
                        uint2* st, Put put) {
  // root box [0,1]^3
  const V3 inv = {1.f / dir.x, 1.f / dir.y, 1.f / dir.z};
  auto cross = [&](float s, float oa, float da, float ia) {
    if constexpr (TINY) return plane_t_div(s, oa, da);
    else return plane_t(s, oa, da, ia);
  };
  DF tin = {0.f, 0.f}, tout = {__builtin_inff(), 0.f};
  bool hit = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float oa = a == 0 ? o.x : (a == 1 ? o.y : o.z), da = a == 0 ? dir.x : (a == 1 ? dir.y : dir.z);
    if (da == 0.f) {
      if (oa < 0.f || oa > 1.f) hit = false;
      continue;
    }
    const float ia = a == 0 ? inv.x : (a == 1 ? inv.y : inv.z);
    DF ta = cross(0.f, oa, da, ia);
    DF tb = cross(1.f, oa, da, ia);
    if (df_lt(tb, ta)) { DF t = ta; ta = tb; tb = t; }
    if (df_lt(tin, ta)) tin = ta;
    if (df_lt(tb, tout)) tout = tb;
  }
  hit = hit && df_lt(tin, tout);
  if (!hit) return 0;
  int m = 0, sp = 0, node = 0;
  DF t0 = tin, t1 = tout;
  while (true) {
    DevNode nd = load_node(nodes, node);
    while (nd.info >= 0) {
      if (AHS && t0.hi > ahs.tstop(node)) break;
      const int a = nd.info & 3;
      const int left = nd.info >> 2;
      // both children (adjacent) are read while the crossing is computed
      const DevNode c0 = load_node(nodes, left), c1 = load_node(nodes, left + 1);
      __builtin_amdgcn_sched_barrier(0);   // (the scheduler would place the read after it)
      const float oa = axis_val(o, a), da = axis_val(dir, a);
      DF ts = cross(nd.plane, oa, da, axis_val(inv, a));
      // a ray parallel to the plane never crosses it: it stays on its side
      const bool par = da == 0.f;
      ts.hi = par ? __builtin_inff() : ts.hi;
      ts.lo = par ? 0.f : ts.lo;
      const bool up = par ? oa >= nd.plane : !(da > 0.f);   // the upper child is entered first
      const int after = left + (up ? 0 : 1);
      const bool only_before = !df_lt(ts, t1);
      const bool only_after = !only_before & !df_lt(t0, ts);
      // the entry above the top is written in any case and kept only when both children are
      // crossed (at depth k at most k entries are held, so it exists)
      const bool both = !only_before & !only_after;
      st[sp * kBlock] = make_uint2(push_word(after, t1.lo), __float_as_uint(t1.hi));
      sp += both ? 1 : 0;
      t1.hi = both ? ts.hi : t1.hi;
      t1.lo = both ? ts.lo : t1.lo;
      const bool upper = only_after ? !up : up;
      node = left + (upper ? 1 : 0);
      nd.plane = upper ? c1.plane : c0.plane;
      nd.info = upper ? c1.info : c0.info;
    }
    const int info = nd.info;
    // interval [t0, t1] of a leaf (or, with AHS, of a node HCheck stopped at), t1 > t0 by
    // construction
    if (EMIT) {
      if (m < cap) {
        float dh = t1.hi - t0.hi;
        float dt = dh + (t1.lo - t0.lo);
        const uint32_t slot = AHS ? ahs.slot(node) : (uint32_t)(-(info + 1));
        put(m, t0.hi, dt, slot | (n_per << 16));
      }
    }
    ++m;
    if (m >= cap + (EMIT ? 0 : 1) || sp == 0) break;
    --sp;
    const uint2 w = st[sp * kBlock];
    node = (int)(w.x & 0xFFFFu);
    t0 = t1;
    t1 = {__uint_as_float(w.y), word_lo(w.x)};
  }
  return m;
}

template <bool EMIT, bool AHS, typename Ahs, typename Put>
__device__ __forceinline__ int traverse(const DevNode* nodes, const Ahs ahs, const V3 o, const V3 dir, int cap,
                                        uint32_t n_per, uint2* st, Put put) {
  // some ray of the wave has a nonzero component whose reciprocal overflows
  auto tiny = [](float v) { return v != 0.f && fabsf(v) < 1.1754944e-38f; };
  if (__ballot(tiny(dir.x) || tiny(dir.y) || tiny(dir.z)) != 0)
    return traverse_one<EMIT, AHS, true>(nodes, ahs, o, dir, cap, n_per, st, put);
  return traverse_one<EMIT, AHS, false>(nodes, ahs, o, dir, cap, n_per, st, put);
}

// The block's copy of the node table (LDS = true) or the table in memory, the per-node
// hierarchical-sampling data (staged with the table when AHS), and the stack.
struct TravLds {
  const DevNode* nodes;
  const float2* ahs;
  uint2* st;
};

template <bool LDS, bool AHS>
__device__ __forceinline__ TravLds stage(const DevNode* __restrict__ nodes, const DevNodeAhs* __restrict__ ahs,
                                         float footprint, uint32_t n_nodes, int stack_n, uint8_t* dyn) {
  TravLds t;
  uint8_t* p = dyn;
  t.ahs = nullptr;
  if (LDS) {
    DevNode* s = reinterpret_cast<DevNode*>(p);
    for (uint32_t i = threadIdx.x; i < n_nodes; i += kBlock) s[i] = nodes[i];
    p += sizeof(DevNode) * n_nodes;
    t.nodes = s;
    if (AHS) {
      float2* a = reinterpret_cast<float2*>(p);
      for (uint32_t i = threadIdx.x; i < n_nodes; i += kBlock) {
        const DevNodeAhs v = ahs[i];
        a[i] = make_float2(__fdiv_rn(v.size, footprint), __builtin_bit_cast(float, v.slot));
      }
      p += sizeof(float2) * n_nodes;
      t.ahs = a;
    }
  } else {
    t.nodes = nodes;
  }
  t.st = reinterpret_cast<uint2*>(p) + threadIdx.x;
  if (LDS) __syncthreads();
  return t;
}

__host__ __device__ constexpr uint32_t trav_lds_bytes(bool lds, bool ahs, uint32_t n_nodes, int stack_n) {
  return (lds ? (uint32_t)(sizeof(DevNode) + (ahs ? sizeof(float2) : 0u)) * n_nodes : 0u) +
         8u * (uint32_t)stack_n * kBlock;
}

// Runs `f` with the hierarchical-sampling view that matches the staging.
template <bool LDS, bool AHS, typename F>
__device__ __forceinline__ int with_ahs(const TravLds& tl, const DevNodeAhs* ahs, float footprint, F f) {
  if constexpr (!AHS) return f(AhsNone{});
  else if constexpr (LDS) return f(AhsLds{tl.ahs});
  else return f(AhsMem{ahs, footprint});
}

// Counts.  Samples per interval follow the ray's leaf-interval count m (s_max / m, or 1
// when m > s_max); with AHS the intervals are those of the HCheck traversal, so a node that
// stops the descent gets one interval's share however many leaves it covers.
template <bool LDS, bool AHS>
__global__ __launch_bounds__(kBlock) void k_trav_count(const DevNode* __restrict__ nodes,
                                                       const DevNodeAhs* __restrict__ ahs, float footprint,
                                                       uint32_t n_nodes,
                                                       int stack_n, const float* __restrict__ o,
                                                       const float* __restrict__ d,
                                                       int64_t stride, int64_t r0, uint32_t nr,
                                                       int s_max, uint32_t* __restrict__ cnt_iv,
                                                       uint32_t* __restrict__ cnt_smp) {
  extern __shared__ __align__(16) uint8_t dyn[];
  const TravLds tl = stage<LDS, AHS>(nodes, ahs, footprint, n_nodes, stack_n, dyn);
  uint32_t r = blockIdx.x * kBlock + threadIdx.x;
  bool live = r < nr;
  V3 oo = {0.f, 0.f, 0.f}, dd = {0.f, 0.f, 1.f};
  if (live) {
    const int64_t ri = r0 + r;
    oo = {o[ri], o[stride + ri], o[2 * stride + ri]};
    dd = {d[ri], d[stride + ri], d[2 * stride + ri]};
  }
  int m = 0, mi = 0;
  // skip the descent for a wave whose rays are all out of range
  if (__ballot(live) != 0 && live) {
    auto none = [](int, float, float, uint32_t) {};
    m = traverse<false, false>(tl.nodes, AhsNone{}, oo, dd, s_max, 0, tl.st, none);
    mi = m;
    if (AHS && m > 0)
      mi = with_ahs<LDS, AHS>(tl, ahs, footprint, [&](auto av) {
        return traverse<false, AHS>(tl.nodes, av, oo, dd, s_max, 0, tl.st, none);
      });
  }
  if (live) {
    uint32_t meff = mi <= s_max ? (uint32_t)mi : (uint32_t)s_max;
    uint32_t nper = m == 0 ? 0u : (m <= s_max ? (uint32_t)(s_max / m) : 1u);
    cnt_iv[r] = meff;
    cnt_smp[r] = meff * nper;
  }
}

// Emission: the block's rays are consecutive, so its intervals fill one contiguous range of
// the output.  Each lane puts its intervals into an LDS copy of the first `stage_n` entries
// of that range (entries past it go straight to memory), and the block then writes the
// staged entries out with consecutive threads on consecutive entries, so every cache line
// is written whole at once instead of piecewise by lanes that finish at different times.
template <bool LDS, bool AHS>
__global__ __launch_bounds__(kBlock) void k_trav_emit(const DevNode* __restrict__ nodes,
                                                      const DevNodeAhs* __restrict__ ahs, float footprint,
                                                      uint32_t n_nodes,
                                                      int stack_n, uint32_t stage_n, const float* __restrict__ o,
                                                      const float* __restrict__ d, int64_t stride,
                                                      int64_t r0, uint32_t nr,
                                                      const uint32_t* __restrict__ cnt_iv,
                                                      const uint32_t* __restrict__ cnt_smp,
                                                      const uint32_t* __restrict__ iv_off,
                                                      const uint32_t* __restrict__ smp_off,
                                                      float* __restrict__ iv_t0,
                                                      float* __restrict__ iv_dt,
                                                      uint32_t* __restrict__ iv_key,
                                                      uint32_t* __restrict__ iv_ray,
                                                      uint32_t* __restrict__ iv_base,
                                                      ChunkCounts* __restrict__ counts) {
  extern __shared__ __align__(16) uint8_t dyn[];
  const TravLds tl = stage<LDS, AHS>(nodes, ahs, footprint, n_nodes, stack_n, dyn);
  uint8_t* sp = dyn + trav_lds_bytes(LDS, AHS, n_nodes, stack_n);
  float* s_t0 = reinterpret_cast<float*>(sp);
  float* s_dt = s_t0 + stage_n;
  uint32_t* s_key = reinterpret_cast<uint32_t*>(s_dt + stage_n);
  uint32_t* s_ray = s_key + stage_n;
  uint32_t* s_base = s_ray + stage_n;
  const uint32_t rb = blockIdx.x * kBlock;                      // first ray of the block
  const uint32_t re = rb + kBlock < nr ? rb + kBlock : nr;      // one past its last ray
  const uint32_t b0 = iv_off[rb], b1 = iv_off[re];              // the block's output range
  const uint32_t r = rb + threadIdx.x;
  const uint32_t meff = r < nr ? cnt_iv[r] : 0u;
  if (__ballot(meff != 0) != 0 && meff != 0) {
    const int64_t ri = r0 + r;
    const V3 oo = {o[ri], o[stride + ri], o[2 * stride + ri]}, dd = {d[ri], d[stride + ri], d[2 * stride + ri]};
    const uint32_t nper = cnt_smp[r] / meff;
    const uint32_t pos0 = iv_off[r] - b0;
    const uint32_t base = smp_off[r];
    auto put = [&](int m, float t0, float dt, uint32_t key) {
      const uint32_t q = pos0 + (uint32_t)m;
      const uint32_t smp = base + (uint32_t)m * nper;
      if (q < stage_n) {
        s_t0[q] = t0; s_dt[q] = dt; s_key[q] = key; s_ray[q] = r; s_base[q] = smp;
      } else {
        iv_t0[b0 + q] = t0; iv_dt[b0 + q] = dt; iv_key[b0 + q] = key; iv_ray[b0 + q] = r;
        iv_base[b0 + q] = smp;
      }
    };
    const int got = with_ahs<LDS, AHS>(tl, ahs, footprint, [&](auto av) {
      return traverse<true, AHS>(tl.nodes, av, oo, dd, (int)meff, nper, tl.st, put);
    });
    // The count pass walks the same way, so `got` equals meff.  Should a walk ever end
    // early, the rest of the ray's range still gets well-formed entries (zero length,
    // slot 0), so later stages never read an unwritten key, and the filled entries are
    // counted (reported by the render statistics; every test requires 0).
    if ((uint32_t)got < meff) {
      for (uint32_t q = (uint32_t)got; q < meff; ++q) put((int)q, 0.f, 0.f, nper << 16);
      atomicAdd(reinterpret_cast<unsigned long long*>(&counts->unreached), (unsigned long long)(meff - (uint32_t)got));
    }
  }
  __syncthreads();
  const uint32_t n = b1 - b0 < stage_n ? b1 - b0 : stage_n;
  for (uint32_t q = threadIdx.x; q < n; q += kBlock) {
    iv_t0[b0 + q] = s_t0[q];
    iv_dt[b0 + q] = s_dt[q];
    iv_key[b0 + q] = s_key[q];
    iv_ray[b0 + q] = s_ray[q];
    iv_base[b0 + q] = s_base[q];
  }
}

}  // namespace

static hipError_t allow_lds(const void* kern) {
  return hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
}

template <bool AHS>
static hipError_t trav_setup_one() {
  hipError_t e = allow_lds((const void*)k_trav_count<true, AHS>);
  if (e == hipSuccess) e = allow_lds((const void*)k_trav_count<false, AHS>);
  if (e == hipSuccess) e = allow_lds((const void*)k_trav_emit<true, AHS>);
  if (e == hipSuccess) e = allow_lds((const void*)k_trav_emit<false, AHS>);
  return e;
}

// Once per device (the attribute is set on the current device).
static hipError_t trav_setup() {
  static std::atomic<uint64_t> done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < 64 ? 1ull << dev : 0ull;
  if (bit && (done.load() & bit)) return hipSuccess;
  e = trav_setup_one<false>();
  if (e == hipSuccess) e = trav_setup_one<true>();
  if (e == hipSuccess) done.fetch_or(bit);
  return e;
}

template <bool LDS, bool AHS>
static void count_launch(uint32_t grid, uint32_t bytes, hipStream_t st, const DevNode* nodes, const DevNodeAhs* ahs,
                         float footprint, uint32_t n_nodes, int stack_n, const float* o, const float* d,
                         int64_t ray_stride, int64_t r0, uint32_t nr, int s_max, uint32_t* cnt_iv, uint32_t* cnt_smp) {
  hipLaunchKernelGGL((k_trav_count<LDS, AHS>), dim3(grid), dim3(kBlock), bytes, st, nodes, ahs, footprint, n_nodes,
                     stack_n, o, d, ray_stride, r0, nr, s_max, cnt_iv, cnt_smp);
}

hipError_t launch_trav_count(const DevNode* nodes, const DevNodeAhs* ahs, float footprint, uint32_t n_nodes, int depth,
                             const float* o, const float* d, int64_t ray_stride, int64_t r0, uint32_t nr, int s_max,
                             uint32_t* cnt_iv, uint32_t* cnt_smp, hipStream_t st) {
  if (nr == 0) return hipSuccess;
  hipError_t e = trav_setup();
  if (e != hipSuccess) return e;
  const int stack_n = depth + 1;
  const uint32_t grid = (nr + kBlock - 1) / kBlock;
  const bool lds = n_nodes <= (uint32_t)kLdsNodes, hs = ahs != nullptr;
  const uint32_t bytes = trav_lds_bytes(lds, hs, n_nodes, stack_n);
  auto go = [&](auto fn) { fn(grid, bytes, st, nodes, ahs, footprint, n_nodes, stack_n, o, d, ray_stride, r0, nr, s_max,
                              cnt_iv, cnt_smp); };
  if (lds && hs) go(count_launch<true, true>);
  else if (lds) go(count_launch<true, false>);
  else if (hs) go(count_launch<false, true>);
  else go(count_launch<false, false>);
  return hipGetLastError();
}

template <bool LDS, bool AHS>
static void emit_launch(uint32_t grid, uint32_t bytes, hipStream_t st, const DevNode* nodes, const DevNodeAhs* ahs,
                        float footprint, uint32_t n_nodes, int stack_n, uint32_t stage_n, const float* o,
                        const float* d, int64_t ray_stride, int64_t r0, uint32_t nr, const uint32_t* cnt_iv,
                        const uint32_t* cnt_smp, const uint32_t* iv_off, const uint32_t* smp_off, float* iv_t0,
                        float* iv_dt, uint32_t* iv_key, uint32_t* iv_ray, uint32_t* iv_base, ChunkCounts* counts) {
  hipLaunchKernelGGL((k_trav_emit<LDS, AHS>), dim3(grid), dim3(kBlock), bytes, st, nodes, ahs, footprint, n_nodes,
                     stack_n, stage_n, o, d, ray_stride, r0, nr, cnt_iv, cnt_smp, iv_off, smp_off, iv_t0, iv_dt,
                     iv_key, iv_ray, iv_base, counts);
}

hipError_t launch_trav_emit(const DevNode* nodes, const DevNodeAhs* ahs, float footprint, uint32_t n_nodes, int depth,
                            const float* o, const float* d, int64_t ray_stride, int64_t r0, uint32_t nr,
                            const uint32_t* cnt_iv, const uint32_t* cnt_smp, const uint32_t* iv_off,
                            const uint32_t* smp_off, float* iv_t0, float* iv_dt, uint32_t* iv_key, uint32_t* iv_ray,
                            uint32_t* iv_base, ChunkCounts* counts, hipStream_t st) {
  if (nr == 0) return hipSuccess;
  hipError_t e = trav_setup();
  if (e != hipSuccess) return e;
  const int stack_n = depth + 1;
  const uint32_t grid = (nr + kBlock - 1) / kBlock;
  const bool lds = n_nodes <= (uint32_t)kLdsNodes, hs = ahs != nullptr;
  // staging sized so that two blocks still fit in a CU's 160 KiB of LDS (the traversal
  // needs the occupancy), at most 2048 entries of 20 bytes
  const uint32_t fixed = trav_lds_bytes(lds, hs, n_nodes, stack_n);
  const uint32_t budget = 80u * 1024u;
  uint32_t stage_n = fixed + 20u * 256u <= budget ? (budget - fixed) / 20u : 256u;
  stage_n = std::min<uint32_t>(stage_n, 2048u) & ~63u;
  const uint32_t bytes = fixed + 20u * stage_n;
  auto go = [&](auto fn) { fn(grid, bytes, st, nodes, ahs, footprint, n_nodes, stack_n, stage_n, o, d, ray_stride, r0,
                              nr, cnt_iv, cnt_smp, iv_off, smp_off, iv_t0, iv_dt, iv_key, iv_ray, iv_base, counts); };
  if (lds && hs) go(emit_launch<true, true>);
  else if (lds) go(emit_launch<true, false>);
  else if (hs) go(emit_launch<false, true>);
  else go(emit_launch<false, false>);
  return hipGetLastError();
}

}  // namespace amn
