// mlp32.hip -- float32 inference of the grouped per-leaf MLPs on the bfloat16 matrix cores.
//
// The float32 matrix instructions (16x16x4) run at a sixteenth of the bfloat16 rate, and the
// float32 leaf MLP was bound by them (0.75 of what they reach).  A float32 value is exactly
// the sum of three bfloat16 values of 8 significant bits each (the split of Henry, Tang and
// Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision
// computations", 2019), and a product of two such values is exact in float32.  Activations are
// split by truncation, |x2| < 2^-7 |x| and |x3| < 2^-15 |x|, weights to nearest, |w2| <= 2^-8 |w|
// and |w3| <= 2^-17 |w|.  Of the nine partial products w x takes eight; w3 x3 alone is left out,
// below 2^-32 |w x|.  The leading products w1 x1 have an accumulator of their own, the seven
// small ones another, whose roundings are 2^-6 of one in the main sum at most and which is added
// to it once: a 64-wide layer then rounds its main sum 5 times (4 steps of 16 and the addition)
// where the float32 instruction rounds it 16 times.
//
// Error against float64: a single product's is the float32 instruction's (largest 2^-24.01, rms
// 2^-24.6 over values with all low bits set; without w2 x3 and w3 x2 they were 2^-22.3 and
// 2^-23.5), a sample's lower at every shape (1..7 layers of 32 and 64): 1.44e-7 -> 1.04e-7 of the
// output's rms at 4x64.  (A main sum within 2^-8 of the largest float may overflow early.)
//
// Instruction: 32x32x16 (it sustains 1.6 times the rate of 16x16x32, and here the order of a
// sum is free).  Its accumulator leaves lane (h = lane / 32, c = lane % 32) rows 8 j + 4 h + i
// (j, i = 0..3) of sample c; taken 8 at a time in that order these are the lane's next B
// operand, with the weights' columns permuted to match, so activations stay in registers and
// each lane splits its own.
//
// Work: the 256-row tiles of mlp.hip, 8 waves of 32 rows per block (the split weights of a
// 4x64 leaf take 87 KB of LDS, so a compute unit holds one block: two waves per SIMD, one
// splitting while the other multiplies).  The output layer (4 rows) runs on the vector units:
// a 32-row matrix step would be seven eighths padding.
// Measured on the 61 M samples of an 800x800 frame, 4x64: 15.2 -> 11.1 ms (30 720 executed FLOP
// per sample and product: 1.35 PFLOP/s of bfloat16 products, matrix cores busy 65 % of 20.7 M
// cycles; 9.4 ms with six products, 12 with nine).  What is left: about 1 400 vector
// instructions per 32 samples, half of them the splits, which the matrix time hides in part
// (a wave's raised priority during its products gained 3 %; interleaving one output block's
// splits with the other's products, and a static priority between a SIMD's two waves, nothing).
#include "internal.hpp"
#include "devcommon.hpp"
#include "mlp_layout.hpp"
#include "rows.hpp"

namespace amn {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kFragBytes = 3 * 1024;   // one A fragment: three parts of 64 lanes x 16 bytes
static_assert(kWaves * 32 == kMlpTileRows, "a wave takes 32 rows of a tile");

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Fragment order: layer 0 (H / 32 output blocks x 2 steps of 16 inputs), then the hidden
// layers (H / 32 x H / 16 each).
__host__ __device__ constexpr int frag0(int H) { return H / 32 * 2; }
__host__ __device__ constexpr int frags_hidden(int H) { return H / 32 * (H / 16); }
__host__ __device__ constexpr int frags(int H, int nh) { return frag0(H) + (nh - 1) * frags_hidden(H); }
// LDS: fragments, biases (n_hidden * H floats), output weights [H][4], output biases [4], the
// waves' row marks
__host__ __device__ constexpr uint32_t lds_bytes(int H, int nh) {
  return (uint32_t)(frags(H, nh) * kFragBytes + nh * H * 4 + H * 16 + 16 + kWaves * 64);
}

__device__ __forceinline__ uint32_t high_halves(float a, float b) {   // low: a's, high: b's
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}
__device__ __forceinline__ float high_part(float a) { return __uint_as_float(__float_as_uint(a) & 0xFFFF0000u); }

// Eight values as three bfloat16 fragments, by truncation: each part takes the leading 8
// significant bits of what the parts before it left (exact).
__device__ __forceinline__ void split8(const float v[8], bf16x8 part[3]) {
  uint32_t w[3][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = v[2 * i], b = v[2 * i + 1];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      w[p][i] = high_halves(a, b);
      if (p < 2) {
        a -= high_part(a);
        b -= high_part(b);
      }
    }
  }
#pragma unroll
  for (int p = 0; p < 3; ++p) part[p] = __builtin_bit_cast(bf16x8, w[p]);
}

// The same for weights, each part rounded to nearest (a finite value that would round to infinity
// keeps its truncated leading part; an infinity or a NaN is its leading part alone).
__device__ __forceinline__ void split_weight(float w, __bf16 part[3]) {
  const bool finite = fabsf(w) < __builtin_inff();
  __bf16 h = (__bf16)w;
  if (finite && !(fabsf((float)h) < __builtin_inff())) h = (__bf16)high_part(w);
  const float r = w - (float)h;
  part[0] = h;
  part[1] = finite ? (__bf16)r : (__bf16)0.f;
  part[2] = finite ? (__bf16)(r - (float)part[1]) : (__bf16)0.f;
}

// Leaf b's float32 block (mlp_layout.hpp) into LDS as split fragments: fragment (layer, ob,
// ks), lane (h, c), elements 0..3 and 4..7 are unit (layer, 2 ob + c / 16, ks), lanes (h, c %
// 16) and (h + 2, c % 16) of the block, in layer 0 as well.
template <int H>
__device__ __forceinline__ void stage_leaf32(const Layout& L, const uint8_t* __restrict__ blk, uint8_t* lds, int tid) {
  constexpr int KS = H / 16;
  const uint8_t* units = blk + L.bias_bytes;
  const int n = frags(H, L.nh) * 64;
  for (int i = tid; i < n; i += kThreads) {
    const int f = i >> 6, lane = i & 63, h = lane >> 5, c = lane & 31;
    int layer = 0, ob = f / 2, ks = f % 2;
    if (f >= frag0(H)) {
      const int q = f - frag0(H);
      layer = 1 + q / frags_hidden(H);
      ob = q % frags_hidden(H) / KS;
      ks = q % KS;
    }
    const uint8_t* u = units + L.unit_index(layer, 2 * ob + (c >> 4), ks) * kUnitBytes + (c & 15) * 16;
    const f32x4 lo = *reinterpret_cast<const f32x4*>(u + h * 256);
    const f32x4 hi = *reinterpret_cast<const f32x4*>(u + (h + 2) * 256);
    bf16x8 part[3];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      __bf16 p[3];
      split_weight(e < 4 ? lo[e & 3] : hi[e & 3], p);
#pragma unroll
      for (int k = 0; k < 3; ++k) part[k][e] = p[k];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) *reinterpret_cast<bf16x8*>(lds + f * kFragBytes + k * 1024 + lane * 16) = part[k];
  }
  const float* src = reinterpret_cast<const float*>(blk);
  float* bias = reinterpret_cast<float*>(lds + frags(H, L.nh) * kFragBytes);
  for (int i = tid; i < L.nh * H; i += kThreads) bias[i] = src[i];
  float* wo = bias + L.nh * H;
  for (int i = tid; i < H * 4; i += kThreads) {   // wo[k][out]: unit (nh, 0, k / 16), lane (k % 16 / 4, out)
    const int k = i >> 2, out = i & 3;
    wo[i] = *reinterpret_cast<const float*>(units + L.unit_index(L.nh, 0, k >> 4) * kUnitBytes +
                                            (((k & 15) >> 2) * 16 + out) * 16 + (k & 3) * 4);
  }
  if (tid < 4) wo[4 * H + tid] = src[L.nh * H + tid];
}

// One layer from the split inputs B[0 .. KS) to the next layer's (written back to B), or, for
// the last hidden layer, into this lane's half of the output layer's sums r.
template <int H, int KS, bool LAST>
__device__ __forceinline__ void layer32(const uint8_t* frag, const float* bias, const float* wo, int lane, int h,
                                        bf16x8 (&B)[H / 16][3], f32x4& r) {
  constexpr int OB = H / 32;
  f32x16 big[OB], small[OB];
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4 bv = *reinterpret_cast<const f32x4*>(bias + 32 * ob + 8 * j + 4 * h);
#pragma unroll
      for (int i = 0; i < 4; ++i) big[ob][4 * j + i] = bv[i];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) small[ob][i] = 0.f;
  }
  __builtin_amdgcn_s_setprio(1);   // products go ahead of the other wave's splits
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    bf16x8 A[OB][3];
#pragma unroll
    for (int ob = 0; ob < OB; ++ob)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        A[ob][p] = *reinterpret_cast<const bf16x8*>(frag + (ob * KS + ks) * kFragBytes + p * 1024 + lane * 16);
    // the products (part of the weights, part of the inputs, sum), smallest first and the leading
    // one last, alternating between blocks
    constexpr int kProducts = 8;
    constexpr int pa[kProducts] = {1, 2, 0, 2, 1, 0, 1, 0}, pb[kProducts] = {2, 1, 2, 0, 1, 1, 0, 0};
#pragma unroll
    for (int q = 0; q < kProducts; ++q)
#pragma unroll
      for (int ob = 0; ob < OB; ++ob) {
        f32x16& acc = q == kProducts - 1 ? big[ob] : small[ob];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[ob][pa[q]], B[ks][pb[q]], acc, 0, 0, 0);
      }
  }
  __builtin_amdgcn_s_setprio(0);
#pragma unroll
  for (int ob = 0; ob < OB; ++ob) {
    // ReLU.  An infinite weight or input makes the small products infinities and NaNs of any kind
    // (inf x 0, w2 inf of the other sign), but every such product has its leading one in the main
    // sum, which is then what the float32 sum is: +inf must come out as +inf, -inf and NaN as 0.
    // So the ReLU's maximum takes a third operand, which is +inf for a main sum of +inf and at
    // most 0 for a finite one.
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
      v[i] = fmaxf(fmaxf(big[ob][i] + small[ob][i], 0.f), big[ob][i] - 3.402823466e38f);
    if constexpr (LAST) {
#pragma unroll
      for (int q = 0; q < 16; q += 8) {
        f32x4 w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
          w[i] = *reinterpret_cast<const f32x4*>(wo + 4 * (32 * ob + 8 * ((q + i) / 4) + 4 * h + i % 4));
        __builtin_amdgcn_sched_barrier(0);   // (eight reads in flight, not one at a time)
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int k = 0; k < 4; ++k) r[k] = fmaf(w[i][k], v[q + i], r[k]);
      }
    } else {
#pragma unroll
      for (int s = 0; s < 2; ++s) split8(&v[8 * s], B[2 * ob + s]);
    }
  }
}

template <int H, bool FUSED>
__global__ __launch_bounds__(kThreads, H == 64 ? 2 : 4) void k_mlp32(
    Layout L, const uint8_t* __restrict__ packed, uint32_t n_leaves, const uint32_t* __restrict__ bucket_off,
    const uint32_t* __restrict__ tile_off, const ChunkCounts* __restrict__ counts,
    const SortRec* __restrict__ sv_rec, const uint32_t* __restrict__ sv_ssb, const uint32_t* __restrict__ sv_win,
    const uint32_t* __restrict__ sm_ray, const float* __restrict__ sm_t, const uint32_t* __restrict__ sm_perm,
    const float* __restrict__ o, const float* __restrict__ d, int64_t stride, int64_t r0, float* __restrict__ out) {
  extern __shared__ __align__(16) uint8_t lds[];
  constexpr int KS = H / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, c = lane & 31;
  const float* bias = reinterpret_cast<const float*>(lds + frags(H, L.nh) * kFragBytes);
  const float* wo = bias + L.nh * H;
  const uint32_t T = counts->n_tiles;
  const uint32_t tb = (uint32_t)(((uint64_t)blockIdx.x * T) / gridDim.x);
  const uint32_t te = (uint32_t)(((uint64_t)(blockIdx.x + 1) * T) / gridDim.x);
  if (tb >= te) return;
  uint32_t lo = 0, hi = n_leaves;   // leaf of the first tile: largest b with tile_off[b] <= tb
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (tile_off[mid] <= tb) lo = mid; else hi = mid;
  }
  uint32_t b = lo;
  int cur = -1;
  // the next tile's row of this lane (both halves of the wave hold row c), found and loaded
  // during the current tile
  uint8_t* mark = lds + lds_bytes(H, L.nh) - (kWaves - wave) * 64;
  const uint32_t n_iv = counts->n_iv;
  const RowSource rows = {sv_rec, sv_ssb, sv_win, sm_ray, sm_t, sm_perm};
  RowFetch<FUSED, 32> q;
  q.init(rows, lo, tb, wave);
  q.locate(rows, bucket_off, tile_off, tb, te - 1, wave, lane, n_iv);
  q.fetch(rows, mark, o, d, stride, r0, lane);
  q.gather(o, d, stride, r0);
  for (uint32_t t = tb; t < te; ++t) {
    while (tile_off[b + 1] <= t) ++b;
    if ((int)b != cur) {
      __syncthreads();
      stage_leaf32<H>(L, packed + (uint64_t)b * L.bytes, lds, tid);
      __syncthreads();
      cur = (int)b;
    }
    const bool valid = q.row0 + (uint32_t)c < q.end;
    const bool any = q.row0 < q.end;
    const uint32_t dst = q.perm;
    float p[3], dd[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      dd[a] = q.d[a];
      p[a] = 2.f * fmaf(q.t, q.d[a], q.o[a]) - 1.f;
    }
    q.locate(rows, bucket_off, tile_off, min(t + 1, te - 1), te - 1, wave, lane, n_iv);
    if (!any) {
      q.fetch(rows, mark, o, d, stride, r0, lane);
      q.gather(o, d, stride, r0);
      q.settle();
      continue;
    }
    // inputs: frequency groups g = h and h + 2 of mlp_layout.hpp's float32 order, slots 4 ks + e
    bf16x8 B[KS][3];
    {
      float f[2][8];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float sc = (float)(1 << (h + 2 * q));
#pragma unroll
        for (int a = 0; a < 3; ++a) sincospif(p[a] * sc, &f[q][a], &f[q][3 + a]);
      }
      f[0][6] = h == 0 ? p[0] : p[2];
      f[0][7] = h == 0 ? p[1] : dd[0];
      f[1][6] = h == 0 ? dd[1] : 0.f;
      f[1][7] = h == 0 ? dd[2] : 0.f;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = f[e / 4][4 * ks + e % 4];
        split8(v, B[ks]);
      }
    }
    // (the output layer's bias enters the half sums of lanes h = 0)
    f32x4 r = h == 0 ? *reinterpret_cast<const f32x4*>(wo + 4 * H) : f32x4{0.f, 0.f, 0.f, 0.f};
    if (L.nh == 1) {
      layer32<H, 2, true>(lds, bias, wo, lane, h, B, r);
      q.fetch(rows, mark, o, d, stride, r0, lane);
      q.gather(o, d, stride, r0);
    } else {
      layer32<H, 2, false>(lds, bias, wo, lane, h, B, r);
      __builtin_amdgcn_sched_barrier(0);
      q.fetch(rows, mark, o, d, stride, r0, lane);
      __builtin_amdgcn_sched_barrier(0);
      const uint8_t* frag = lds + frag0(H) * kFragBytes;
      const float* lb = bias + H;
      for (int layer = 1; layer + 1 < L.nh; ++layer) {
        layer32<H, KS, false>(frag, lb, wo, lane, h, B, r);
        frag += frags_hidden(H) * kFragBytes;
        lb += H;
      }
      __builtin_amdgcn_sched_barrier(0);
      q.gather(o, d, stride, r0);
      __builtin_amdgcn_sched_barrier(0);
      layer32<H, KS, true>(frag, lb, wo, lane, h, B, r);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] += __shfl_xor(r[k], 32, 64);
    if (h == 0 && valid) *reinterpret_cast<f32x4*>(out + 4 * (uint64_t)dst) = r;
  }
}

template <int H, bool FUSED>
hipError_t launch_rows32(const Layout& L, const void* packed, uint32_t n_leaves, const uint32_t* bucket_off,
                         const uint32_t* tile_off, const ChunkCounts* counts, const RowSource& rows, const float* o,
                         const float* d, int64_t stride, int64_t r0, float* out, hipStream_t st) {
  auto kern = k_mlp32<H, FUSED>;
  const uint32_t lds = lds_bytes(H, L.nh);
  int grid = 0;
  hipError_t e = persistent_grid((const void*)kern, kThreads, lds, &grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, st, L, (const uint8_t*)packed, n_leaves, bucket_off,
                     tile_off, counts, rows.rec, rows.ssb, rows.win, rows.ray, rows.t,
                     rows.perm, o, d, stride, r0, out);
  return hipGetLastError();
}

template <int H>
hipError_t launch_typed32(const Layout& L, const void* packed, uint32_t n_leaves, const uint32_t* bucket_off,
                          const uint32_t* tile_off, const ChunkCounts* counts, const RowSource& rows, const float* o,
                          const float* d, int64_t stride, int64_t r0, float* out, hipStream_t st) {
  return rows.rec ? launch_rows32<H, true>(L, packed, n_leaves, bucket_off, tile_off, counts, rows, o, d, stride, r0, out, st)
                  : launch_rows32<H, false>(L, packed, n_leaves, bucket_off, tile_off, counts, rows, o, d, stride, r0, out, st);
}

}  // namespace

bool mlp32_fits(int n_hidden, int hidden) { return lds_bytes(hidden, n_hidden) <= 160u * 1024u; }

hipError_t launch_mlp32(int n_hidden, int hidden, const void* packed, uint32_t n_leaves, const uint32_t* bucket_off,
                        const uint32_t* tile_off, const ChunkCounts* counts, const RowSource& rows, const float* o,
                        const float* d, int64_t stride, int64_t r0, float* out, hipStream_t st) {
  const Layout L = make_layout(n_hidden, hidden, AMNERF_F32);
  return hidden == 64 ? launch_typed32<64>(L, packed, n_leaves, bucket_off, tile_off, counts, rows, o, d, stride, r0, out, st)
                      : launch_typed32<32>(L, packed, n_leaves, bucket_off, tile_off, counts, rows, o, d, stride, r0, out, st);
}

}  // namespace amn
