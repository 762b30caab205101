// scan.hip -- exclusive prefix sums of uint32 arrays whose length may live on the device, in
// one pass (chain.hpp): used for ray offsets, the sort's count matrix and the rounds' selection.
//
// A tile is 2048 elements (256 threads x 8, in registers between its sum and its output), or
// 8192 (1024 threads) from 2^19 on, so every element is read and written once.  What bounds a
// long scan is the chain, which passes from tile to tile at 25 to 35 ns: with small tiles, and
// with blocks that took a second ticket to learn that nothing was left, 5 M elements took 60 us
// and 18 now, the 1.7 M of a training batch's matrix 43 and 17.  Reduce, scan of the block sums
// and rescan read everything twice and took three launches: 21 us for those 5 M, and 12 us of
// launches for a 64x64 tile's matrix and intervals, where this takes 6.
#include "internal.hpp"
#include "chain.hpp"

namespace amn {
namespace {

constexpr int kPer = 8;
constexpr int kSmallThreads = kScanItems / kPer;   // 256
constexpr int kLargeThreads = 1024;
constexpr uint64_t kLargeFrom = 1ull << 19;

// What an element holds and where its prefix goes.
enum ScanMode {
  kSingle,   // one array to one
  kPair,     // two arrays of the same length to two
  kPacked    // count << 20 | samples in one word: the counts' prefix in place, the samples' to out2
};

// Both halves of a sum stay below 2^31 (a pass holds at most 2^28 samples).
__device__ __forceinline__ uint64_t pack2(uint32_t a, uint32_t b) { return ((uint64_t)a << 31) | b; }

template <int MODE>
__device__ __forceinline__ uint64_t element(uint32_t a, uint32_t b) {
  if (MODE == kPair) return pack2(a, b);
  if (MODE == kPacked) return pack2(a >> 20, a & 0xFFFFFu);
  return a;
}

template <int MODE>
__device__ __forceinline__ void split2(uint64_t v, uint32_t& a, uint32_t& b) {
  a = MODE == kSingle ? (uint32_t)v : (uint32_t)(v >> 31);
  b = (uint32_t)v & 0x7FFFFFFFu;
}

// n = n_cap, or mul * ceil(*n_dev / div) (at most n_cap) when n_dev is given.
template <int MODE, int kThreads>
__global__ __launch_bounds__(kThreads) void k_scan(const uint32_t* in, const uint32_t* __restrict__ in2, uint32_t* out,
                                                   uint32_t* __restrict__ out2, uint64_t n_cap,
                                                   const uint32_t* __restrict__ n_dev, uint32_t mul, uint32_t div,
                                                   uint64_t* __restrict__ state) {
  constexpr uint32_t kItems = kThreads * kPer;
  __shared__ uint32_t s_tile;
  __shared__ uint64_t s_wave[kThreads / 64], s_before;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t n = n_cap;
  if (n_dev) {
    n = (uint64_t)mul * (((uint64_t)*n_dev + div - 1) / div);
    if (n > n_cap) n = n_cap;
  }
  if (n == 0 && blockIdx.x == 0 && threadIdx.x == 0) {
    out[0] = 0u;
    if (MODE != kSingle) out2[0] = 0u;
  }
  // one block per tile; those past a shorter array leave without a ticket
  if ((uint64_t)blockIdx.x * kItems >= n) return;
  if (threadIdx.x == 0) s_tile = chain_ticket(state);
  __syncthreads();
  const uint32_t tile = __builtin_amdgcn_readfirstlane(s_tile);
  const uint64_t first = (uint64_t)tile * kItems;
  const uint64_t base = first + (uint64_t)threadIdx.x * kPer;
  uint32_t a[kPer], b[kPer];
  if (base + kPer <= n) {
#pragma unroll
    for (int i = 0; i < kPer; i += 4) {
      const uint4 v = *reinterpret_cast<const uint4*>(in + base + i);
      a[i] = v.x; a[i + 1] = v.y; a[i + 2] = v.z; a[i + 3] = v.w;
      if (MODE == kPair) {
        const uint4 w = *reinterpret_cast<const uint4*>(in2 + base + i);
        b[i] = w.x; b[i + 1] = w.y; b[i + 2] = w.z; b[i + 3] = w.w;
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      a[i] = base + i < n ? in[base + i] : 0u;
      b[i] = MODE == kPair && base + i < n ? in2[base + i] : 0u;
    }
  }
  uint64_t own = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) own += element<MODE>(a[i], b[i]);
  uint64_t incl = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t y = __shfl_up(incl, off, 64);
    if (lane >= off) incl += y;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  uint64_t pre = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) {
    if (w < wave) pre += s_wave[w];
    tot += s_wave[w];
  }
  if (wave == 0) {
    const uint64_t before = chain_prefix(state + 1, tile, tot, lane);
    if (lane == 0) s_before = before;
  }
  __syncthreads();
  uint64_t run = s_before + pre + (incl - own);
  uint32_t x[kPer], y[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    split2<MODE>(run, x[i], y[i]);
    run += element<MODE>(a[i], b[i]);
  }
  if (base + kPer <= n) {
#pragma unroll
    for (int i = 0; i < kPer; i += 4) {
      *reinterpret_cast<uint4*>(out + base + i) = make_uint4(x[i], x[i + 1], x[i + 2], x[i + 3]);
      if (MODE != kSingle) *reinterpret_cast<uint4*>(out2 + base + i) = make_uint4(y[i], y[i + 1], y[i + 2], y[i + 3]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (base + i < n) {
        out[base + i] = x[i];
        if (MODE != kSingle) out2[base + i] = y[i];
      }
  }
  if (first + kItems >= n && threadIdx.x == 0) {   // the last tile: the totals
    uint32_t ta, tb;
    split2<MODE>(s_before + tot, ta, tb);
    out[n] = ta;
    if (MODE != kSingle) out2[n] = tb;
  }
}

template <int MODE>
hipError_t launch(const uint32_t* in, const uint32_t* in2, uint32_t* out, uint32_t* out2, uint64_t n_cap,
                  const uint32_t* n_dev, uint32_t mul, uint32_t div, uint64_t* state, hipStream_t st) {
  const uint32_t threads = n_cap < kLargeFrom ? kSmallThreads : kLargeThreads;
  const uint64_t nb = (n_cap + threads * kPer - 1) / (threads * kPer);
  const uint32_t grid = (uint32_t)(nb > 0 ? nb : 1);
  hipLaunchKernelGGL((threads == kSmallThreads ? k_scan<MODE, kSmallThreads> : k_scan<MODE, kLargeThreads>), dim3(grid),
                     dim3(threads), 0, st, in, in2, out, out2, n_cap, n_dev, mul, div, state);
  return hipGetLastError();
}

}  // namespace

// A ticket and a word per (small) tile.
uint64_t scan_state_words(uint64_t n_cap) { return 1 + (n_cap + kScanItems - 1) / kScanItems; }

hipError_t launch_scan_u32(const uint32_t* in, uint32_t* out, uint64_t n_cap, const uint32_t* n_dev,
                           uint64_t* state, hipStream_t st) {
  return launch<kSingle>(in, nullptr, out, nullptr, n_cap, n_dev, 1u, 1u, state, st);
}

hipError_t launch_scan_u32_pair(const uint32_t* in_a, uint32_t* out_a, const uint32_t* in_b, uint32_t* out_b,
                                uint64_t n_cap, uint64_t* state, hipStream_t st) {
  return launch<kPair>(in_a, in_b, out_a, out_b, n_cap, nullptr, 1u, 1u, state, st);
}

hipError_t launch_scan_packed(uint32_t* mat, uint32_t* out_smp, uint64_t n_cap, const uint32_t* n_dev, uint32_t mul,
                              uint32_t div, uint64_t* state, hipStream_t st) {
  return launch<kPacked>(mat, nullptr, mat, out_smp, n_cap, n_dev, mul, div, state, st);
}

}  // namespace amn
