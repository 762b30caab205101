// mlp_bwd.hip -- backward pass of the grouped per-leaf MLP (bfloat16 operands, float32
// accumulation), the differentiable counterpart of the grouped forward in mlp.hip.
//
// Work item: a segment of at most seg_tiles consecutive 256-row tiles of one leaf, each
// processed by a block of 8 waves (2 per SIMD: one block fills a compute unit), 32 rows per
// wave in two column blocks that share every weight read.  Every wave recomputes its forward
// activations (none are stored between the forward and backward passes) and keeps each layer's
// bfloat16 input in registers in B-operand order.  Then, from the output layer down:
//   * dZ_l (gradient at layer l's pre-activation) and the layer's input H_{l-1} are staged
//     in LDS, a row per sample, and the waves accumulate dW_l = sum_samples dZ_l H_{l-1}^T on
//     MFMA with K = samples (and db_l = sum_samples dZ_l against a ones operand), their
//     operands coming from transposed LDS reads;
//   * dH_{l-1} = W_l^T dZ_l runs on MFMA in registers (transposed weights packed in the
//     same register-chained order as the forward), then dZ_{l-1} = dH_{l-1} where the
//     forward activation was positive.
// Each segment writes its partial dW, db (master layout) to its own slot; a separate
// kernel sums the slots of each leaf in order, so the gradient is deterministic.
//
// What bounds it is the chain of a tile's phases (the matrix cores are busy a third of the
// time): a layer's staging, its dW blocks on half of the waves, and dH wait for each other, two
// waves per SIMD being what the registers allow.  262 144-ray training batch (23 M samples, 4
// layers of 64), every sum in the same order throughout: 16 waves of 16 rows that staged
// feature-major (2-byte writes, every weight fragment read twice as often) 4.70 ms; rows staged
// as they are 3.67; LDS reads issued ahead of the matrix instructions 3.15.  16 waves of 16 rows
// on this staging spill (3.8 ms or more).
#include "internal.hpp"
#include "devcommon.hpp"
#include "mlp_layout.hpp"

namespace amn {
namespace {

constexpr int kThreads = 256;                    // the float32 kernel's block
constexpr int kWavesB = 8;                       // waves of a bfloat16 block (2 per SIMD)
constexpr int kThreadsB = 64 * kWavesB;
constexpr int kNCB = 2;                          // 16-sample column blocks per wave
constexpr int kTileRows = kMlpTileRows;          // 256-row tiles of the forward pass, one
static_assert(kWavesB * 16 * kNCB == kTileRows, "a tile is one step of the block");   // step each
constexpr int kRowBytes = 128;                   // staged sample (bf16 features)
constexpr int kWeightsAhead = 6;                 // weight fragments read ahead of their use

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Weight-gradient ownership, fixed so that every sum is taken in one order.  Below the
// output layer, dW_l is cut into 32x32 blocks (rows: outputs; columns: staged inputs),
// accumulated with 32x32x16 MFMAs over the tile's samples.  The blocks of the layers in the
// order 1, 2, .., NH - 1, 0 are dealt to the waves in turn, (H/32)^2 a layer, so a wave holds
// at most two and never two of one layer.  db_l's 16-row blocks go to 16x16x32 MFMAs against
// a ones operand, dealt in turn too, to waves that hold no dW block of the layer and at most
// two a wave.  The output layer (its outputs padded to 16 rows) keeps 16x16 blocks: column
// block ci on wave ci, its db on the last wave.
__device__ __forceinline__ constexpr int bwd_slot(int NH, int l) { return l >= 1 ? l - 1 : NH - 1; }
__device__ __forceinline__ constexpr int bwd_first_block(int H, int NH, int l) {
  return bwd_slot(NH, l) * (H / 32) * (H / 32);
}

// Staged samples are rows of kRowBytes whose sixteen 8-byte pieces are permuted by an exclusive
// or with the low bits of the sample's number, reordered to s1 s3 s2 s0.  A wave's 8-byte write
// takes 16 lanes at a time (32 banks): 16 samples, the same piece, which all four bits spread.  A
// transposed read takes 32 lanes (64 banks): eight pieces of four samples in a row, which s0
// (a row is half the banks) and s1 spread, or four pieces of samples 0..3 and 8..11, which s0,
// s1 and s3 spread.  Neither has a bank conflict; with 32-byte pieces permuted the writes took
// 16 cycles instead of 4.
__device__ __forceinline__ uint32_t stage_swz(uint32_t s) {
  return (s & 2u) << 5 ^ (s & 8u) << 2 ^ (s & 4u) << 2 ^ (s & 1u) << 3;
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Eight samples of one feature from two transposed reads: each lane group of 16 reads a
// 4-sample x 16-feature block, lane i receiving feature i of the four samples.
__device__ __forceinline__ bf16x8 read_tr(const uint8_t* p0, const uint8_t* p1) {
  typedef __attribute__((address_space(3))) s16x4* lds_ptr;
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p0);
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)p1);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

__device__ __forceinline__ bool pos_bf16(__bf16 v) {
  return __builtin_bit_cast(short, v) > 0;
}

template <int H, int NH>
__global__ __launch_bounds__(kThreadsB, 2) void k_mlp_bwd(
    Layout L, const uint8_t* __restrict__ packed_fwd, const uint8_t* __restrict__ packed_bwd,
    uint32_t n_leaves, const uint32_t* __restrict__ bucket_off,
    const uint32_t* __restrict__ tile_off, const uint32_t* __restrict__ seg_off,
    const uint32_t* __restrict__ srec_ray, const float* __restrict__ srec_t,
    const uint32_t* __restrict__ perm, const float* __restrict__ o, const float* __restrict__ d,
    int64_t stride, int64_t r0, const float* __restrict__ gpre, float* __restrict__ part, int P,
    uint32_t* __restrict__ seg_queue, uint32_t seg_tiles) {
  extern __shared__ __align__(16) uint8_t lds[];
  constexpr int RB = H / 16;
  constexpr int KUh = H / 32;
  constexpr int kBig = (4 * (H / 32) * (H / 32) + kWavesB - 1) / kWavesB;   // blocks a wave holds at most
  constexpr int kBias = (4 * (H / 16) + kWavesB - 1) / kWavesB;
  uint8_t* w_fwd = lds;
  uint8_t* w_bwd = lds + L.bytes;
  uint8_t* s_dz = w_bwd + L.bwd_bytes;                       // H = 32: gradients and inputs share rows
  uint32_t& s_seg = *reinterpret_cast<uint32_t*>(s_dz + (H == 64 ? 2 : 1) * kTileRows * kRowBytes);   // the segment taken
  const float* bias = reinterpret_cast<const float*>(w_fwd);
  const uint8_t* units = w_fwd + L.bias_bytes;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, m = lane & 15;
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.f;
  // this wave's blocks (see above)
  const int h32 = lane >> 5, c32 = lane & 31;
  int big_l[kBig], big_ri[kBig], big_cj[kBig], bias_l[kBias], bias_j[kBias];
#pragma unroll
  for (int q = 0; q < kBig; ++q) big_l[q] = -1, big_ri[q] = 0, big_cj[q] = 0;
#pragma unroll
  for (int q = 0; q < kBias; ++q) bias_l[q] = -1, bias_j[q] = 0;
#pragma unroll
  for (int l = 0; l < NH; ++l) {
    const int ncol = l == 0 ? 1 : H / 32;
    const int first = bwd_first_block(H, NH, l);
    const int n_big = (H / 32) * ncol;
#pragma unroll
    for (int q = 0; q < kBig; ++q) {
      const int bi = wave + q * kWavesB - first;
      if (bi >= 0 && bi < n_big) { big_l[q] = l; big_ri[q] = bi / ncol; big_cj[q] = bi % ncol; }
    }
    const int bj = (wave - (H / 16) * (bwd_slot(NH, l) + 1)) & (kWavesB - 1);
    if (bj < H / 16) {
      bias_l[bwd_slot(NH, l) * (H / 16) / kWavesB] = l;
      bias_j[bwd_slot(NH, l) * (H / 16) / kWavesB] = bj;
    }
  }
  // byte offsets, the same for every layer: this wave's writes (sample row, 16-feature block rb)
  uint32_t wr[4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
    wr[rb] = (uint32_t)(wave * 16 * kNCB + m) * kRowBytes + ((32u * rb + 8u * g) ^ stage_swz(m));
  // and the transposed reads: 32-wide operands (+ 2048 bytes per 16 samples; feature block j of
  // the gradients, of the inputs) and 16-wide ones (+ 4096 bytes per 32 samples)
  auto rd32 = [&](int j, uint32_t area, int t) {
    const uint32_t smp = 8u * h32 + 4u * t + (m >> 2);
    return smp * kRowBytes + ((area + 64u * j + 32u * (g & 1) + 8u * (m & 3)) ^ stage_swz(smp));
  };
  auto rd16 = [&](int j, uint32_t area, int t) {
    const uint32_t smp = 8u * g + 4u * t + (m >> 2);
    return smp * kRowBytes + ((area + 32u * j + 8u * (m & 3)) ^ stage_swz(smp));
  };
  constexpr uint32_t kHIn = H == 64 ? 0u : 64u;              // the inputs' place in a row
  uint8_t* s_in = H == 64 ? s_dz + kTileRows * kRowBytes : s_dz;

  const uint32_t n_seg = seg_off[n_leaves];
  int cur = -1;
  // segments are taken from a queue (segments differ in length, so a fixed stride over them
  // leaves blocks unevenly loaded); each writes its own partial slot, so the order is free
  if (tid == 0) s_seg = atomicAdd(seg_queue, 1u);
  __syncthreads();
  uint32_t seg = __builtin_amdgcn_readfirstlane(s_seg);
  while (seg < n_seg) {
    uint32_t lo = 0, hi = n_leaves;
    while (hi - lo > 1) {
      uint32_t mid = (lo + hi) >> 1;
      if (seg_off[mid] <= seg) lo = mid; else hi = mid;
    }
    const uint32_t b = lo;
    const uint32_t t_first = tile_off[b] + (seg - seg_off[b]) * seg_tiles;
    const uint32_t t_last = t_first + seg_tiles < tile_off[b + 1] ? t_first + seg_tiles : tile_off[b + 1];
    if ((int)b != cur) {
      __syncthreads();
      const f32x4* s1 = reinterpret_cast<const f32x4*>(packed_fwd + (uint64_t)b * L.bytes);
      for (uint32_t i = tid; i < L.bytes / 16; i += kThreadsB) reinterpret_cast<f32x4*>(w_fwd)[i] = s1[i];
      const f32x4* s2 = reinterpret_cast<const f32x4*>(packed_bwd + (uint64_t)b * L.bwd_bytes);
      for (uint32_t i = tid; i < L.bwd_bytes / 16; i += kThreadsB) reinterpret_cast<f32x4*>(w_bwd)[i] = s2[i];
      __syncthreads();
      cur = (int)b;
    }
    f32x16 accW32[kBig];       // this wave's 32x32 blocks of dW_l (l < NH)
    f32x4 accB16[kBias];       // its 16-row blocks of db_l (l < NH)
#pragma unroll
    for (int q = 0; q < kBig; ++q)
#pragma unroll
      for (int i = 0; i < 16; ++i) accW32[q][i] = 0.f;
#pragma unroll
    for (int q = 0; q < kBias; ++q) accB16[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 accWo = {0.f, 0.f, 0.f, 0.f};    // its 16x16 block of the output layer's dW
    f32x4 accBo = {0.f, 0.f, 0.f, 0.f};    // the output layer's db (last wave)

    // Rows are read a tile ahead, in two steps (the record, then what it points at), each
    // issued well before its use; past the leaf's last row the last one is read again.
    const uint32_t row_first = bucket_off[b] + (t_first - tile_off[b]) * kTileRows;
    const uint32_t row_end = bucket_off[b + 1];
    const uint32_t row_lane = wave * (16 * kNCB) + m;
    uint32_t n_ray[kNCB], n_dst[kNCB];
    float n_ts[kNCB], n_ray6[kNCB][6];
    f32x4 n_gz[kNCB];
    auto read_rec = [&](uint32_t row0) {
#pragma unroll
      for (int cb = 0; cb < kNCB; ++cb) {
        const uint32_t row = min(row0 + row_lane + 16u * cb, row_end - 1u);
        n_ray[cb] = srec_ray[row];
        n_ts[cb] = srec_t[row];
        n_dst[cb] = perm[row];
      }
    };
    auto read_row = [&]() {
#pragma unroll
      for (int cb = 0; cb < kNCB; ++cb) {
        const int64_t ri = r0 + n_ray[cb];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          n_ray6[cb][a] = o[a * stride + ri];
          n_ray6[cb][3 + a] = d[a * stride + ri];
        }
        n_gz[cb] = *reinterpret_cast<const f32x4*>(gpre + 4 * (uint64_t)n_dst[cb]);
      }
    };
    read_rec(row_first);
    read_row();

    for (uint32_t tile = t_first; tile < t_last; ++tile) {
      const uint32_t row0 = row_first + (tile - t_first) * kTileRows;
      // ---- forward recompute: layer inputs in B-operand order ----
      bf16x8 X0[kNCB];
      bf16x8 Hs[NH + 1][kNCB][KUh];    // Hs[l] = input of layer l (l >= 1), after ReLU
      f32x4 dz[kNCB][RB];
#pragma unroll
      for (int cb = 0; cb < kNCB; ++cb) {
        const bool valid = row0 + row_lane + 16u * cb < row_end;
        const float ts = n_ts[cb];
        const float dx = n_ray6[cb][3], dy = n_ray6[cb][4], dzz = n_ray6[cb][5];
        const float px = 2.f * fmaf(ts, dx, n_ray6[cb][0]) - 1.f;
        const float py = 2.f * fmaf(ts, dy, n_ray6[cb][1]) - 1.f;
        const float pz = 2.f * fmaf(ts, dzz, n_ray6[cb][2]) - 1.f;
        float feat[8];
        const float v = g == 1 ? py : (g == 2 ? pz : px);
        float sn = __builtin_amdgcn_sinf(0.5f * v);
        float cs = __builtin_amdgcn_cosf(0.5f * v);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          feat[2 * k] = sn;
          feat[2 * k + 1] = cs;
          const float t2 = sn + sn;
          const float s2 = t2 * cs;
          cs = fmaf(-t2, sn, 1.f);
          sn = s2;
        }
        if (g == 3) {
          feat[0] = px; feat[1] = py; feat[2] = pz;
          feat[3] = dx; feat[4] = dy; feat[5] = dzz;
          feat[6] = 0.f; feat[7] = 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) X0[cb][e] = (__bf16)feat[e];
        // output-layer gradient: lanes of group 0 hold (dsigma^, dr^, dg^, db^)
        f32x4 gz = {0.f, 0.f, 0.f, 0.f};
        if (g == 0 && valid) gz = n_gz[cb];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) dz[cb][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
        dz[cb][0] = gz;
      }
      read_rec(row0 + kTileRows);
#pragma unroll
      for (int l = 0; l < NH; ++l) {
        f32x4 acc[kNCB][RB];
        const int n_ku = l == 0 ? 1 : KUh;
        bf16x8 A[RB * KUh];
        f32x4 bv[RB];
        read_ahead<RB * KUh, kWeightsAhead>(
            [&](int i) {
              const int rb = i / KUh, ku = i % KUh;
              if (ku >= n_ku) return;
              if (ku == 0) bv[rb] = *reinterpret_cast<const f32x4*>(bias + l * H + 16 * rb + 4 * g);
              A[i] = *reinterpret_cast<const bf16x8*>(units + L.unit_index(l, rb, ku) * kUnitBytes + lane * 16);
            },
            [&](int i) {
              const int rb = i / KUh, ku = i % KUh;
              if (ku >= n_ku) return;
#pragma unroll
              for (int cb = 0; cb < kNCB; ++cb)
                acc[cb][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[i], l == 0 ? X0[cb] : Hs[l][cb][ku],
                                                                      ku == 0 ? bv[rb] : acc[cb][rb], 0, 0, 0);
            });
#pragma unroll
        for (int cb = 0; cb < kNCB; ++cb)
#pragma unroll
          for (int ku = 0; ku < KUh; ++ku) {
            float vv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) vv[e] = acc[cb][2 * ku + e / 4][e % 4];
            Hs[l + 1][cb][ku] = relu_bf16x8(vv);
          }
      }

      read_row();

      // ---- backward, output layer first ----
#pragma unroll
      for (int l = NH; l >= 0; --l) {
        const int rbo = l == NH ? 1 : RB;          // row blocks of this layer's outputs
        // dZ_l in bfloat16: the operand of dH below, and what is staged
        const int ku_n = l == NH ? 1 : KUh;
        bf16x8 Bz[kNCB][KUh];
#pragma unroll
        for (int cb = 0; cb < kNCB; ++cb)
#pragma unroll
          for (int ku = 0; ku < KUh; ++ku) {
            if (ku >= ku_n) break;
            float vv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const int rbs = 2 * ku + e / 4;
              vv[e] = rbs < rbo ? dz[cb][rbs][e % 4] : 0.f;
            }
            Bz[cb][ku] = cvt_bf16x8(vv);
          }
        // stage dZ_l and the layer input, a row per sample
        __syncthreads();
#pragma unroll
        for (int cb = 0; cb < kNCB; ++cb) {
          auto put = [&](uint8_t* base, int rb, bf16x8 v, int half) {
            *reinterpret_cast<bf16x4*>(base + wr[rb] + cb * 16 * kRowBytes) =
                half ? __builtin_shufflevector(v, v, 4, 5, 6, 7) : __builtin_shufflevector(v, v, 0, 1, 2, 3);
          };
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            if (rb >= rbo) break;
            put(s_dz, rb, Bz[cb][rb / 2], rb & 1);
          }
          if (l == 0) {
#pragma unroll
            for (int half = 0; half < 2; ++half)
              *reinterpret_cast<bf16x4*>(s_in + (wave * 16 * kNCB + cb * 16 + m) * kRowBytes +
                                         ((kHIn + 16u * g + 8u * half) ^ stage_swz(m))) =
                  half ? __builtin_shufflevector(X0[cb], X0[cb], 4, 5, 6, 7) : __builtin_shufflevector(X0[cb], X0[cb], 0, 1, 2, 3);
          } else {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
              put(s_in, (int)(kHIn / 32u) + rb, Hs[l][cb][rb / 2], rb & 1);
          }
        }
        __syncthreads();
        // dW_l += dZ_l H^T, db_l += dZ_l 1 over the tile's samples
        if (l == NH) {
          const uint8_t *a0 = s_dz + rd16(0, 0u, 0), *a1 = s_dz + rd16(0, 0u, 1);
          bf16x8 A[kTileRows / 32], Bm[kTileRows / 32];
          if (wave < RB) {
            const uint8_t *b0 = s_in + rd16(wave, kHIn, 0), *b1 = s_in + rd16(wave, kHIn, 1);
            read_ahead<kTileRows / 32, 3>(
                [&](int kb) {
                  A[kb] = read_tr(a0 + 4096 * kb, a1 + 4096 * kb);
                  Bm[kb] = read_tr(b0 + 4096 * kb, b1 + 4096 * kb);
                },
                [&](int kb) { accWo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[kb], Bm[kb], accWo, 0, 0, 0); });
          } else if (wave == kWavesB - 1) {
            read_ahead<kTileRows / 32, 5>(
                [&](int kb) { A[kb] = read_tr(a0 + 4096 * kb, a1 + 4096 * kb); },
                [&](int kb) { accBo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[kb], ones, accBo, 0, 0, 0); });
          }
        } else {
          // A: lane (h, c) holds dZ feature 32 ri + c of samples 16 ks + 8 h ..; B: the input
          // feature 32 cj + c of the same samples
#pragma unroll
          for (int q = 0; q < kBig; ++q) {
            if (bwd_first_block(H, NH, l) + (H / 32) * (l == 0 ? 1 : H / 32) <= q * kWavesB ||
                bwd_first_block(H, NH, l) >= (q + 1) * kWavesB)
              continue;
            if (big_l[q] != l) continue;
            const uint8_t *a0 = s_dz + rd32(big_ri[q], 0u, 0), *a1 = s_dz + rd32(big_ri[q], 0u, 1);
            const uint8_t *b0 = s_in + rd32(big_cj[q], kHIn, 0), *b1 = s_in + rd32(big_cj[q], kHIn, 1);
            bf16x8 A[kTileRows / 16], Bm[kTileRows / 16];
            read_ahead<kTileRows / 16, 3>(
                [&](int ks) {
                  A[ks] = read_tr(a0 + 2048 * ks, a1 + 2048 * ks);
                  Bm[ks] = read_tr(b0 + 2048 * ks, b1 + 2048 * ks);
                },
                [&](int ks) { accW32[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[ks], Bm[ks], accW32[q], 0, 0, 0); });
          }
          const int q = bwd_slot(NH, l) * (H / 16) / kWavesB;
          if (bias_l[q] == l) {
            const uint8_t *a0 = s_dz + rd16(bias_j[q], 0u, 0), *a1 = s_dz + rd16(bias_j[q], 0u, 1);
            bf16x8 A[kTileRows / 32];
            read_ahead<kTileRows / 32, 5>(
                [&](int kb) { A[kb] = read_tr(a0 + 4096 * kb, a1 + 4096 * kb); },
                [&](int kb) { accB16[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[kb], ones, accB16[q], 0, 0, 0); });
          }
        }
        if (l == 0) break;
        // dH = W_l^T dZ_l, then the ReLU mask of the forward activation
        f32x4 dh[kNCB][RB];
        bf16x8 A[RB * KUh];
        read_ahead<RB * KUh, kWeightsAhead>(
            [&](int i) {
              const int rb = i / KUh, ku = i % KUh;
              if (ku >= ku_n) return;
              A[i] = *reinterpret_cast<const bf16x8*>(w_bwd + L.bwd_unit_index(l, rb, ku) * kUnitBytes + lane * 16);
            },
            [&](int i) {
              const int rb = i / KUh, ku = i % KUh;
              if (ku >= ku_n) return;
#pragma unroll
              for (int cb = 0; cb < kNCB; ++cb)
                dh[cb][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    A[i], Bz[cb][ku], ku == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : dh[cb][rb], 0, 0, 0);
            });
#pragma unroll
        for (int cb = 0; cb < kNCB; ++cb)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              dz[cb][rb][i] = pos_bf16(Hs[l][cb][rb / 2][4 * (rb % 2) + i]) ? dh[cb][rb][i] : 0.f;
      }
    }

    // ---- this segment's partial gradient, master layout ----
    // (every weight and bias of the leaf is written by exactly one wave)
    float* dst = part + (uint64_t)seg * P;
    {
      int din, dout, off_w, off_b;
      master_offsets(NH, H, NH, din, dout, off_w, off_b);
      const int c = 16 * wave + m;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int out = 4 * g + i;
        if (wave < RB && out < dout) dst[off_w + out * din + c] = accWo[i];
        if (wave == kWavesB - 1 && m == 0 && out < dout) dst[off_b + out] = accBo[i];
      }
    }
#pragma unroll
    for (int q = 0; q < kBig; ++q) {
      if (big_l[q] < 0) continue;
      int din, dout, off_w, off_b;
      master_offsets(NH, H, big_l[q], din, dout, off_w, off_b);
      const int cc = 32 * big_cj[q] + c32;
      const int col = big_l[q] == 0 ? first_layer_col_bf16(cc / 8, cc % 8) : cc;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int out = 32 * big_ri[q] + 8 * (r / 4) + 4 * h32 + (r % 4);   // accumulator row of register r
        if (out < dout && col >= 0) dst[off_w + out * din + col] = accW32[q][r];
      }
    }
#pragma unroll
    for (int q = 0; q < kBias; ++q) {
      if (bias_l[q] < 0 || m != 0) continue;
      int din, dout, off_w, off_b;
      master_offsets(NH, H, bias_l[q], din, dout, off_w, off_b);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int out = 16 * bias_j[q] + 4 * g + i;
        if (out < dout) dst[off_b + out] = accB16[q][i];
      }
    }
    __syncthreads();   // every wave has read s_seg
    if (tid == 0) s_seg = atomicAdd(seg_queue, 1u);
    __syncthreads();
    seg = __builtin_amdgcn_readfirstlane(s_seg);
  }
}

// ---- float32 operands: v_mfma_f32_16x16x4_f32.  An MFMA takes A[m][k] from lane
// (k, m) and B[k][n] from lane (k, n) (one float each) and leaves C rows 4g..4g+3 of column
// n in lane (g, n).  The same work split as the bfloat16 kernel (segments of one leaf's
// tiles, partial gradients per segment), with 64-row sub-tiles of 16 rows per wave; the
// leaf's float32 forward block (the layout k_mlp reads) is staged in LDS and serves both
// the forward recomputation and, read transposed, dH = W^T dZ.
constexpr int kSub32 = 64;                 // rows of a float32 sub-tile (4 waves x 16)
constexpr int kRowF = kSub32 + 4;          // staged feature row (floats) + padding

// W_l[row][col] of a hidden or output layer inside the float32 forward block: unit
// (l, row / 16, col / 16), lane ((col % 16) / 4) * 16 + row % 16, element col % 4.
__device__ __forceinline__ float w_at(const Layout& L, const uint8_t* units, int l, int row, int col) {
  const int u = L.unit_index(l, row >> 4, col >> 4);
  return *reinterpret_cast<const float*>(units + u * kUnitBytes + ((((col & 15) >> 2) << 4) + (row & 15)) * 16 +
                                         (col & 3) * 4);
}

template <int H, int NH>
__global__ __launch_bounds__(kThreads) void k_mlp_bwd_f32(
    Layout L, const uint8_t* __restrict__ packed, uint32_t n_leaves, const uint32_t* __restrict__ bucket_off,
    const uint32_t* __restrict__ tile_off, const uint32_t* __restrict__ seg_off,
    const uint32_t* __restrict__ srec_ray, const float* __restrict__ srec_t, const uint32_t* __restrict__ perm,
    const float* __restrict__ o, const float* __restrict__ d, int64_t stride, int64_t r0,
    const float* __restrict__ gpre, float* __restrict__ part, int P, uint32_t seg_tiles) {
  extern __shared__ __align__(16) uint8_t lds[];
  constexpr int RB = H / 16;
  const float* bias = reinterpret_cast<const float*>(lds);
  const uint8_t* units = lds + L.bias_bytes;
  float* sZ = reinterpret_cast<float*>(lds + L.bytes);   // [H][kRowF]: dZ_l, feature-major
  float* sH = sZ + H * kRowF;                            // [H][kRowF]: layer input, feature-major
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, m = lane & 15;
  const uint32_t n_seg = seg_off[n_leaves];
  int cur = -1;
  for (uint32_t seg = blockIdx.x; seg < n_seg; seg += gridDim.x) {
    uint32_t lo = 0, hi = n_leaves;
    while (hi - lo > 1) {
      uint32_t mid = (lo + hi) >> 1;
      if (seg_off[mid] <= seg) lo = mid; else hi = mid;
    }
    const uint32_t b = lo;
    const uint32_t t_first = tile_off[b] + (seg - seg_off[b]) * seg_tiles;
    const uint32_t t_last = t_first + seg_tiles < tile_off[b + 1] ? t_first + seg_tiles : tile_off[b + 1];
    if ((int)b != cur) {
      __syncthreads();
      const f32x4* src = reinterpret_cast<const f32x4*>(packed + (uint64_t)b * L.bytes);
      for (uint32_t i = tid; i < L.bytes / 16; i += kThreads) reinterpret_cast<f32x4*>(lds)[i] = src[i];
      __syncthreads();
      cur = (int)b;
    }
    f32x4 accW[NH + 1][4];
    f32x4 accB[NH + 1];
#pragma unroll
    for (int l = 0; l <= NH; ++l) {
      accB[l] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 4; ++q) accW[l][q] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    constexpr int kSubPerTile = kMlpTileRows / kSub32;
    for (uint32_t sub = kSubPerTile * t_first; sub < kSubPerTile * t_last; ++sub) {
      const uint32_t row_end = bucket_off[b + 1];
      const uint32_t row = bucket_off[b] + (sub - kSubPerTile * tile_off[b]) * kSub32 + wave * 16 + m;
      const bool valid = row < row_end;
      // ---- this lane's sample (column m of the wave's block): inputs as in the forward ----
      uint32_t ray = 0, dst = 0;
      float ts = 0.f;
      if (valid) {
        ray = srec_ray[row];
        ts = srec_t[row];
        dst = perm[row];
      }
      const int64_t ri = r0 + ray;
      const float ox = o[ri], oy = o[stride + ri], oz = o[2 * stride + ri];
      const float dx = d[ri], dy = d[stride + ri], dz_ = d[2 * stride + ri];
      const float px = 2.f * fmaf(ts, dx, ox) - 1.f;
      const float py = 2.f * fmaf(ts, dy, oy) - 1.f;
      const float pz = 2.f * fmaf(ts, dz_, oz) - 1.f;
      float feat[8];
      {
        const float sc = (float)(1 << g);
        feat[0] = sinpif(px * sc); feat[1] = sinpif(py * sc); feat[2] = sinpif(pz * sc);
        feat[3] = cospif(px * sc); feat[4] = cospif(py * sc); feat[5] = cospif(pz * sc);
        feat[6] = g == 0 ? px : (g == 1 ? pz : (g == 2 ? dy : 0.f));
        feat[7] = g == 0 ? py : (g == 1 ? dx : (g == 2 ? dz_ : 0.f));
      }
      // ---- forward recompute: Hs[l] = ReLU output of layer l (accumulator layout) ----
      f32x4 Hs[NH][RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        f32x4 z = *reinterpret_cast<const f32x4*>(bias + 16 * rb + 4 * g);
#pragma unroll
        for (int ku = 0; ku < 2; ++ku) {
          const f32x4 A = *reinterpret_cast<const f32x4*>(units + L.unit_index(0, rb, ku) * kUnitBytes + lane * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) z = __builtin_amdgcn_mfma_f32_16x16x4f32(A[e], feat[4 * ku + e], z, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) Hs[0][rb][i] = fmaxf(z[i], 0.f);
      }
#pragma unroll
      for (int l = 1; l < NH; ++l) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          f32x4 z = *reinterpret_cast<const f32x4*>(bias + l * H + 16 * rb + 4 * g);
#pragma unroll
          for (int ku = 0; ku < RB; ++ku) {
            const f32x4 A = *reinterpret_cast<const f32x4*>(units + L.unit_index(l, rb, ku) * kUnitBytes + lane * 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) z = __builtin_amdgcn_mfma_f32_16x16x4f32(A[e], Hs[l - 1][ku][e], z, 0, 0, 0);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) Hs[l][rb][i] = fmaxf(z[i], 0.f);
        }
      }
      // ---- backward from the output layer: lanes of group 0 hold dL/d(sigma^, r^, g^, b^) ----
      f32x4 dz[RB];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) dz[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (g == 0 && valid) dz[0] = *reinterpret_cast<const f32x4*>(gpre + 4 * (uint64_t)dst);
#pragma unroll
      for (int l = NH; l >= 0; --l) {
        const int rbo = l == NH ? 1 : RB;          // row blocks of this layer's outputs
        const int cbi = l == 0 ? 2 : RB;           // 16-column blocks of its inputs
        const int n_items = rbo * cbi;
        const int per = (n_items + 3) / 4;
        __syncthreads();
        const int col = wave * 16 + m;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          if (rb >= rbo) break;
#pragma unroll
          for (int i = 0; i < 4; ++i) sZ[(16 * rb + 4 * g + i) * kRowF + col] = dz[rb][i];
        }
        if (l == 0) {
#pragma unroll
          for (int i = 0; i < 8; ++i) sH[(8 * g + i) * kRowF + col] = feat[i];
        } else {
#pragma unroll
          for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) sH[(16 * rb + 4 * g + i) * kRowF + col] = Hs[l - 1][rb][i];
        }
        __syncthreads();
        // dW_l += dZ_l X_l^T and db_l += dZ_l 1 over the sub-tile's 64 samples (K = samples)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int item = wave * per + q;
          if (q >= per || item >= n_items) break;
          const int rb = item / cbi, ci = item % cbi;
#pragma unroll 4
          for (int kk = 0; kk < kSub32 / 4; ++kk) {
            const float a = sZ[(16 * rb + m) * kRowF + 4 * kk + g];
            const float bb = sH[(16 * ci + m) * kRowF + 4 * kk + g];
            accW[l][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, bb, accW[l][q], 0, 0, 0);
            if (ci == 0) accB[l] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, 1.f, accB[l], 0, 0, 0);
          }
        }
        if (l == 0) break;
        // dH = W_l^T dZ_l (rows: the layer's inputs; K: its outputs), then the ReLU mask
        f32x4 dh[RB];
#pragma unroll
        for (int rbi = 0; rbi < RB; ++rbi) {
          dh[rbi] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ku = 0; ku < RB; ++ku) {
            if (ku >= rbo) break;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float a = w_at(L, units, l, 16 * ku + 4 * g + e, 16 * rbi + m);
              dh[rbi] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, dz[ku][e], dh[rbi], 0, 0, 0);
            }
          }
        }
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
          for (int i = 0; i < 4; ++i) dz[rb][i] = Hs[l - 1][rb][i] > 0.f ? dh[rb][i] : 0.f;
      }
    }

    // ---- this segment's partial gradient, master layout ----
    float* dstp = part + (uint64_t)seg * P;
#pragma unroll
    for (int l = 0; l <= NH; ++l) {
      const int rbo = l == NH ? 1 : RB;
      const int cbi = l == 0 ? 2 : RB;
      const int n_items = rbo * cbi;
      const int per = (n_items + 3) / 4;
      int din, dout, off_w, off_b;
      master_offsets(NH, H, l, din, dout, off_w, off_b);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int item = wave * per + q;
        if (q >= per || item >= n_items) break;
        const int rb = item / cbi, ci = item % cbi;
        const int c = 16 * ci + m;
        const int colm = l == 0 ? first_layer_col(c >> 3, c & 7) : c;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int out = 16 * rb + 4 * g + i;
          if (out < dout && colm >= 0) dstp[off_w + out * din + colm] = accW[l][q][i];
          if (ci == 0 && m == 0 && out < dout) dstp[off_b + out] = accB[l][i];
        }
      }
    }
  }
}

template <int H, int NH>
hipError_t launch_bwd_f32_typed(const Layout& L, const void* packed, uint32_t n_leaves,
                                const uint32_t* bucket_off, const uint32_t* tile_off,
                                const uint32_t* seg_off, const uint32_t* srec_ray, const float* srec_t,
                                const uint32_t* perm, const float* o, const float* d, int64_t stride,
                                int64_t r0, const float* gpre, float* part, uint32_t seg_tiles, hipStream_t st) {
  auto kern = k_mlp_bwd_f32<H, NH>;
  const uint32_t lds = L.bytes + 2u * H * kRowF * 4u;
  int grid = 0;
  hipError_t e = persistent_grid((const void*)kern, kThreads, lds, &grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, st, L, (const uint8_t*)packed, n_leaves,
                     bucket_off, tile_off, seg_off, srec_ray, srec_t, perm, o, d, stride, r0, gpre, part,
                     master_param_count(NH, H), seg_tiles);
  return hipGetLastError();
}

template <int H, int NH>
hipError_t launch_bwd_typed(const Layout& L, const void* packed, uint32_t n_leaves,
                            const uint32_t* bucket_off, const uint32_t* tile_off,
                            uint32_t* seg_off, const uint32_t* srec_ray, const float* srec_t,
                            const uint32_t* perm, const float* o, const float* d, int64_t stride,
                            int64_t r0, const float* gpre, float* part, uint32_t seg_tiles, hipStream_t st) {
  auto kern = k_mlp_bwd<H, NH>;
  const uint32_t lds = L.bytes + L.bwd_bytes + (H == 64 ? 2u : 1u) * kTileRows * kRowBytes + 16u;   // + the queue word
  int grid = 0;
  hipError_t e = persistent_grid((const void*)kern, kThreadsB, lds, &grid);
  if (e != hipSuccess) return e;
  const uint8_t* pf = (const uint8_t*)packed;
  const uint8_t* pb = pf + (uint64_t)n_leaves * L.bytes;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreadsB), lds, st, L, pf, pb, n_leaves, bucket_off, tile_off,
                     seg_off, srec_ray, srec_t, perm, o, d, stride, r0, gpre, part,
                     master_param_count(NH, H), seg_off + n_leaves + 1, seg_tiles);
  return hipGetLastError();
}

}  // namespace

bool mlp_bwd_supported(int n_hidden, int hidden) {
  return n_hidden >= 1 && n_hidden <= 4 && (hidden == 32 || hidden == 64);
}

hipError_t launch_mlp_bwd(const MlpGeom& g, const void* packed, uint32_t n_leaves,
                          const uint32_t* bucket_off, const uint32_t* tile_off, uint32_t* seg_off,
                          const uint32_t* srec_ray, const float* srec_t, const uint32_t* perm,
                          const float* o, const float* d, int64_t ray_stride, int64_t r0,
                          const float* gpre, float* part, uint32_t seg_tiles, hipStream_t st) {
  Layout L = make_layout(g.n_hidden, g.hidden, g.dtype);
#define AMN_BWD(HH, NN)                                                                                \
  if (g.hidden == HH && g.n_hidden == NN) {                                                            \
    if (g.dtype == AMNERF_F32)                                                                         \
      return launch_bwd_f32_typed<HH, NN>(L, packed, n_leaves, bucket_off, tile_off, seg_off, srec_ray, \
                                          srec_t, perm, o, d, ray_stride, r0, gpre, part, seg_tiles, st); \
    return launch_bwd_typed<HH, NN>(L, packed, n_leaves, bucket_off, tile_off, seg_off, srec_ray,       \
                                    srec_t, perm, o, d, ray_stride, r0, gpre, part, seg_tiles, st);   \
  }
  AMN_BWD(64, 4)
  AMN_BWD(64, 3)
  AMN_BWD(64, 2)
  AMN_BWD(64, 1)
  AMN_BWD(32, 4)
  AMN_BWD(32, 3)
  AMN_BWD(32, 2)
  AMN_BWD(32, 1)
#undef AMN_BWD
  return hipErrorInvalidValue;
}

}  // namespace amn
