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
// crossing therefore multiplies by a reciprocal taken once per ray and axis, with a residual
// step that gives a division's bits, both children of a node are read while its crossing is
// computed, and the side of the plane and the ray's component are chosen without branches.
// 4096 rays x 20 leaves of a 512-leaf tree, one traversal: 54 -> 36 us.
#include <algorithm>

#include <atomic>

#include "internal.hpp"
#include "chain.hpp"
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

// a / d from the correctly rounded reciprocal inv: one residual step makes the product's quotient
// (within 2 ulp) the correctly rounded one (Markstein, "Computation of elementary functions on the
// IBM RISC System/6000 processor", 1990), as long as nothing under- or overflows.
__device__ __forceinline__ float quotient(float a, float d, float inv) {
  const float q = a * inv;
  return fmaf(fmaf(-q, d, a), inv, q);
}

// (s - o) / d as a normalised pair, inv the correctly rounded 1 / d: the quotient, the fused
// (exact) remainder of it, and that remainder's quotient: the bits of the same steps with
// divisions.  (With bare products for quotients the pair's error was three times that, 2^-45.2
// against 2^-47, and the traversal of a 64x64 tile took 46 us instead of 48, of an 800x800 frame
// 126 instead of 129.)  No contraction: h - q0 must see the rounded q0.
__device__ __forceinline__ DF plane_t(float s, float o, float d, float inv) {
#pragma clang fp contract(off)
  DF num = two_sum(s, -o);
  float q0 = quotient(num.hi, d, inv);
  float r = fmaf(-q0, d, num.hi);
  r += num.lo;
  float q1 = quotient(r, d, inv);
  float h = q0 + q1;
  float l = q1 - (h - q0);
  return {h, l};
}

// The same by division, for components that are so small that the quotient may overflow, or so
// large that the reciprocal is no normal number.  Small ones are scaled by 2^64 (exact) and the
// pair scaled back: t is then an infinity of the right sign where it exceeds the float range,
// instead of the NaN of an infinity's remainder.
__device__ __forceinline__ DF plane_t_div(float s, float o, float d) {
#pragma clang fp contract(off)
  const float sc = fabsf(d) < 0x1p-100f ? 0x1p64f : 1.f, ds = d * sc;
  DF num = two_sum(s, -o);
  float q0 = num.hi / ds;
  if (isinf(q0)) return {q0, 0.f};
  float r = fmaf(-q0, ds, num.hi);
  r += num.lo;
  float q1 = r / ds;
  float h = q0 + q1;
  float l = q1 - (h - q0);
  h *= sc;
  return {h, isinf(h) ? 0.f : l * sc};
}

// (bitwise: three compares and two mask operations, no branch)
__device__ __forceinline__ bool df_lt(DF a, DF b) { return (a.hi < b.hi) | ((a.hi == b.hi) & (a.lo < b.lo)); }

// Blocks of kBlock rays, or of kBlockSmall (one wave) for launches that would otherwise leave
// compute units without a block.
constexpr int kBlock = 256, kBlockSmall = 64;
constexpr uint32_t kSmallRays = 65536;   // 256 compute units x 256 rays
// LDS per block: the node table (when staged), then the traversal stack of `stack_n` =
// tree depth + 1 8-byte entries per thread, strided by the block size (a wave's entries of one level
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

// Traverses one ray: hands its first `cap` intervals to put(m, t0, dt, slot) and returns the
// interval count, stopping once it exceeds cap.  AHS: stop the descent by HCheck, and key
// intervals by the node's preorder slot.  B: the block size (the stack's stride).
__device__ __forceinline__ uint32_t push_word(int node, float lo) {
  return (uint32_t)node | ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)lo) << 16);
}
__device__ __forceinline__ float word_lo(uint32_t w) { return (float)__builtin_bit_cast(__bf16, (uint16_t)(w >> 16)); }

// TINY: crossings by division (see plane_t_div).
template <int B, bool AHS, bool TINY, typename Ahs, typename Put>
__device__ int traverse_one(const DevNode* nodes, const Ahs ahs, const V3 o, const V3 dir, int cap, uint2* st,
                            Put put) {
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
      st[sp * B] = make_uint2(push_word(after, t1.lo), __float_as_uint(t1.hi));
      sp += both ? 1 : 0;
      t1.hi = both ? ts.hi : t1.hi;
      t1.lo = both ? ts.lo : t1.lo;
      const bool upper = only_after ? !up : up;
      node = left + (upper ? 1 : 0);
      nd.plane = upper ? c1.plane : c0.plane;
      nd.info = upper ? c1.info : c0.info;
    }
    // interval [t0, t1] of a leaf (or, with AHS, of a node HCheck stopped at), t1 > t0 by
    // construction
    if (m < cap) {
      float dh = t1.hi - t0.hi;
      float dt = dh + (t1.lo - t0.lo);
      put(m, t0.hi, dt, AHS ? ahs.slot(node) : (uint32_t)(-(nd.info + 1)));
    }
    ++m;
    if (m > cap || sp == 0) break;
    --sp;
    const uint2 w = st[sp * B];
    node = (int)(w.x & 0xFFFFu);
    t0 = t1;
    t1 = {__uint_as_float(w.y), word_lo(w.x)};
  }
  return m;
}

template <int B, bool AHS, typename Ahs, typename Put>
__device__ __forceinline__ int traverse(const DevNode* nodes, const Ahs ahs, const V3 o, const V3 dir, int cap,
                                        uint2* st, Put put) {
  // some ray of the wave has a nonzero component for plane_t_div (origins within 2^27 cannot
  // make the quotient of one of 2^-100 overflow)
  auto odd = [](float v) { return v != 0.f && !(fabsf(v) >= 0x1p-100f && fabsf(v) <= 0x1p126f); };
  if (__ballot(odd(dir.x) || odd(dir.y) || odd(dir.z)) != 0)
    return traverse_one<B, AHS, true>(nodes, ahs, o, dir, cap, st, put);
  return traverse_one<B, AHS, false>(nodes, ahs, o, dir, cap, st, put);
}

// The block's copy of the node table (LDS = true) or the table in memory, the per-node
// hierarchical-sampling data (staged with the table when AHS), and the stack.
struct TravLds {
  const DevNode* nodes;
  const float2* ahs;
  uint2* st;
};

template <int B, bool LDS, bool AHS>
__device__ __forceinline__ TravLds stage(const DevNode* __restrict__ nodes, const DevNodeAhs* __restrict__ ahs,
                                         float footprint, uint32_t n_nodes, int stack_n, uint8_t* dyn) {
  TravLds t;
  uint8_t* p = dyn;
  t.ahs = nullptr;
  if (LDS) {
    DevNode* s = reinterpret_cast<DevNode*>(p);
    for (uint32_t i = threadIdx.x; i < n_nodes; i += B) s[i] = nodes[i];
    p += sizeof(DevNode) * n_nodes;
    t.nodes = s;
    if (AHS) {
      float2* a = reinterpret_cast<float2*>(p);
      for (uint32_t i = threadIdx.x; i < n_nodes; i += B) {
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
  return t;   // (the caller synchronises the block)
}

__host__ __device__ constexpr uint32_t trav_lds_bytes(int block, bool lds, bool ahs, uint32_t n_nodes, int stack_n) {
  return (lds ? (uint32_t)(sizeof(DevNode) + (ahs ? sizeof(float2) : 0u)) * n_nodes : 0u) +
         8u * (uint32_t)stack_n * (uint32_t)block;
}

// Runs `f` with the hierarchical-sampling view that matches the staging.
template <bool LDS, bool AHS, typename F>
__device__ __forceinline__ int with_ahs(const TravLds& tl, const DevNodeAhs* ahs, float footprint, F f) {
  if constexpr (!AHS) return f(AhsNone{});
  else if constexpr (LDS) return f(AhsLds{tl.ahs});
  else return f(AhsMem{ahs, footprint});
}

// Traversal in one pass.  Samples per interval follow the ray's leaf-interval count m (s_max /
// m, or 1 when m > s_max); with AHS the intervals are those of the HCheck traversal, so a node
// that stops the descent gets one interval's share however many leaves it covers (the leaves
// are counted by a walk of their own first).
//
// Where a ray's intervals go depends on the counts of every ray before it.  Each wave puts its
// intervals, as it finds them, into scratch rows of its own (row m = the m-th interval of its
// rays, so a row is one coalesced write); the block's totals then go through the chained scan,
// and the wave writes its part of the ray-major arrays with consecutive lanes on consecutive
// entries, reading its rows back while they are still in cache.  Walking twice (a counting
// pass, three scan launches and an emitting pass) cost the whole chain a second time; whole
// renders: 4096-ray tile 153 -> 125 us, 800x800 planned frame 1.82 -> 1.72 ms, 1920x1080 frame
// of 4096 leaves 9.02 -> 8.01 ms.
template <int B, bool LDS, bool AHS>
__global__ __launch_bounds__(B) void k_trav(
    const DevNode* __restrict__ nodes, const DevNodeAhs* __restrict__ ahs, float footprint, uint32_t n_nodes,
    int stack_n, const float* __restrict__ o, const float* __restrict__ d, int64_t stride, int64_t r0, uint32_t nr,
    int s_max, uint32_t iv_cap, float2* scratch_t, uint32_t* scratch_slot, uint64_t* __restrict__ state,
    uint32_t* __restrict__ iv_off, uint32_t* __restrict__ smp_off, float* __restrict__ iv_t0,
    float* __restrict__ iv_dt, uint32_t* __restrict__ iv_key, uint32_t* __restrict__ iv_ray,
    uint32_t* __restrict__ iv_base) {
  extern __shared__ __align__(16) uint8_t dyn[];
  constexpr int W = B / 64;
  __shared__ uint32_t s_blk;
  __shared__ uint64_t s_sum[W], s_before;
  __shared__ int s_mark[W][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) s_blk = chain_ticket(state);
  const TravLds tl = stage<B, LDS, AHS>(nodes, ahs, footprint, n_nodes, stack_n, dyn);
  __syncthreads();
  const uint32_t blk = __builtin_amdgcn_readfirstlane(s_blk);
  const uint32_t rw = blk * B + 64u * (uint32_t)wave;   // the wave's first ray
  const uint32_t r = rw + (uint32_t)lane;
  const uint32_t width = rw < nr ? (nr - rw < 64u ? nr - rw : 64u) : 0u;   // its rays = its rows' length
  float2* const row_t = scratch_t + (uint64_t)rw * iv_cap;
  uint32_t* const row_slot = scratch_slot + (uint64_t)rw * iv_cap;
  int m = 0, mi = 0;
  if ((uint32_t)lane < width) {
    const int64_t ri = r0 + r;
    const V3 oo = {o[ri], o[stride + ri], o[2 * stride + ri]}, dd = {d[ri], d[stride + ri], d[2 * stride + ri]};
    auto put = [&](int k, float t0, float dt, uint32_t slot) {
      row_t[(uint32_t)k * width + lane] = make_float2(t0, dt);
      row_slot[(uint32_t)k * width + lane] = slot;
    };
    if constexpr (AHS) {
      m = traverse<B, false>(tl.nodes, AhsNone{}, oo, dd, s_max, tl.st, [](int, float, float, uint32_t) {});
      if (m > 0)
        mi = with_ahs<LDS, AHS>(tl, ahs, footprint,
                                [&](auto av) { return traverse<B, AHS>(tl.nodes, av, oo, dd, s_max, tl.st, put); });
    } else {
      mi = m = traverse<B, false>(tl.nodes, AhsNone{}, oo, dd, s_max, tl.st, put);
    }
  }
  const uint32_t meff = mi <= s_max ? (uint32_t)mi : (uint32_t)s_max;
  const uint32_t nper = m == 0 ? 0u : (m <= s_max ? (uint32_t)(s_max / m) : 1u);
  // intervals in the high and samples in the low part of one sum (both stay below 2^31)
  const uint64_t own = ((uint64_t)meff << 31) | (meff * nper);
  uint64_t incl = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t y = __shfl_up(incl, off, 64);
    if (lane >= off) incl += y;
  }
  if (lane == 63) s_sum[wave] = incl;
  __syncthreads();
  uint64_t sum = 0, first = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    if (w < wave) first += s_sum[w];
    sum += s_sum[w];
  }
  if (wave == 0) {
    const uint64_t before = chain_prefix(state + 1, blk, sum, lane);
    if (lane == 0) s_before = before;
  }
  __syncthreads();
  const uint64_t at_wave = s_before + first, at = at_wave + (incl - own);
  constexpr uint32_t kLow = 0x7FFFFFFFu;
  const uint32_t base = (uint32_t)at & kLow;
  if ((uint32_t)lane < width) {
    iv_off[r] = (uint32_t)(at >> 31);
    smp_off[r] = base;
  }
  if (r + 1 == nr) {   // (the last ray of the launch)
    iv_off[nr] = (uint32_t)((at + own) >> 31);
    smp_off[nr] = (uint32_t)(at + own) & kLow;
  }
  // the wave's intervals, ray-major: entry q belongs to the last ray that starts at or before
  // it (rays mark their first entry in a 64-entry window, a prefix maximum spreads the marks)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  const uint32_t iv_w = (uint32_t)(at_wave >> 31);
  const uint32_t pos = (uint32_t)(at >> 31) - iv_w;   // this ray's first entry among the wave's
  const uint32_t n_w = (uint32_t)(__shfl(incl, 63, 64) >> 31);
  for (uint32_t q0 = 0; q0 < n_w; q0 += 64) {
    s_mark[wave][lane] = -1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (meff != 0 && pos >= q0 && pos < q0 + 64u) s_mark[wave][pos - q0] = lane;
    const uint64_t started = __ballot(meff != 0 && pos <= q0);   // ray 0 of them at least
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int src = max(wave_max_incl(s_mark[wave][lane]), 63 - (int)__builtin_clzll(started));
    const uint32_t k = q0 + (uint32_t)lane - __shfl(pos, src, 64);
    const uint32_t np = __shfl(nper, src, 64), sb = __shfl(base, src, 64);
    if (q0 + (uint32_t)lane < n_w) {
      const float2 t = row_t[k * width + (uint32_t)src];
      const uint32_t slot = row_slot[k * width + (uint32_t)src];
      const uint32_t q = iv_w + q0 + (uint32_t)lane;
      iv_t0[q] = t.x;
      iv_dt[q] = t.y;
      iv_key[q] = slot | (np << 16);
      iv_ray[q] = rw + (uint32_t)src;
      iv_base[q] = sb + k * np;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

template <int B, bool AHS>
hipError_t trav_setup_one() {
  auto allow = [](const void* k) {
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
  };
  hipError_t e = allow((const void*)k_trav<B, true, AHS>);
  if (e == hipSuccess) e = allow((const void*)k_trav<B, false, AHS>);
  return e;
}

// Once per device (the attribute is set on the current device).
hipError_t trav_setup() {
  static std::atomic<uint64_t> done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev < 64 ? 1ull << dev : 0ull;
  if (bit && (done.load() & bit)) return hipSuccess;
  e = trav_setup_one<kBlock, false>();
  if (e == hipSuccess) e = trav_setup_one<kBlock, true>();
  if (e == hipSuccess) e = trav_setup_one<kBlockSmall, false>();
  if (e == hipSuccess) e = trav_setup_one<kBlockSmall, true>();
  if (e == hipSuccess) done.fetch_or(bit);
  return e;
}

}  // namespace

uint64_t trav_state_words(uint64_t nr) {
  // enough for any launch of at most nr rays (the last pass of a call is a smaller one)
  const uint64_t small = (std::min<uint64_t>(nr, kSmallRays) + kBlockSmall - 1) / kBlockSmall;
  return 1 + std::max<uint64_t>(small, (nr + kBlock - 1) / kBlock);
}

hipError_t launch_trav(const DevNode* nodes, const DevNodeAhs* ahs, float footprint, uint32_t n_nodes, int depth,
                       const float* o, const float* d, int64_t ray_stride, int64_t r0, uint32_t nr, int s_max,
                       uint32_t iv_cap, float* scratch, uint64_t* state, uint32_t* iv_off, uint32_t* smp_off,
                       float* iv_t0, float* iv_dt, uint32_t* iv_key, uint32_t* iv_ray, uint32_t* iv_base,
                       hipStream_t st) {
  if (nr == 0) return hipSuccess;
  hipError_t e = trav_setup();
  if (e != hipSuccess) return e;
  const int stack_n = depth + 1;
  const bool lds = n_nodes <= (uint32_t)kLdsNodes, hs = ahs != nullptr, small = nr < kSmallRays;
  const int block = small ? kBlockSmall : kBlock;
  const uint32_t grid = (nr + (uint32_t)block - 1) / (uint32_t)block;
  const uint32_t bytes = trav_lds_bytes(block, lds, hs, n_nodes, stack_n);
  float2* const scratch_t = reinterpret_cast<float2*>(scratch);
  uint32_t* const scratch_slot = reinterpret_cast<uint32_t*>(scratch + 2 * (uint64_t)nr * iv_cap);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(grid), dim3(block), bytes, st, nodes, ahs, footprint, n_nodes, stack_n, o, d,
                       ray_stride, r0, nr, s_max, iv_cap, scratch_t, scratch_slot, state, iv_off, smp_off, iv_t0, iv_dt,
                       iv_key, iv_ray, iv_base);
  };
  if (small) {
    if (lds && hs) go(k_trav<kBlockSmall, true, true>);
    else if (lds) go(k_trav<kBlockSmall, true, false>);
    else if (hs) go(k_trav<kBlockSmall, false, true>);
    else go(k_trav<kBlockSmall, false, false>);
  } else {
    if (lds && hs) go(k_trav<kBlock, true, true>);
    else if (lds) go(k_trav<kBlock, true, false>);
    else if (hs) go(k_trav<kBlock, false, true>);
    else go(k_trav<kBlock, false, false>);
  }
  return hipGetLastError();
}

}  // namespace amn
