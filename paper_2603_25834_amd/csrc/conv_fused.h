// conv_fused.h -- the actor-critic's convolutional encoder in one kernel (gfx950).
//
// conv1 (1 -> 16) and conv2 (16 -> 32), both 3x3 with stride 2 and padding 1
// and ReLU, for one sample at a time per workgroup, with the 32x32x16 conv1
// activation kept in LDS: HBM sees only the 64x64 int16 crop coming in and the
// 8192 BF16 features going out.  Both convolutions run on MFMA
// (v_mfma_f32_16x16x32_bf16, FP32 accumulation) with the same rounding points
// as the layer-by-layer path: crop L/256, weights and activations in BF16.
//
// conv1 is written as C'[co][px] = sum_k W'[co][k] P[k][px] over a 4x4 input
// window per output pixel: the crop is stored in LDS space-to-depth (2x2
// blocks of 8 bytes), so the window of pixel (y, x) is the four blocks at
// block rows y-1, y and block columns x-1, x, and a lane's eight k values are
// two adjacent blocks (two 8-byte reads).  k = 8r + 4c + 2dy + dx addresses
// block row r, block column c and the element (dy, dx) inside it, which is
// input row 2y - 2 + 2r + dy, i.e. tap ky = 2r + dy - 1 (likewise kx); taps
// outside 0..2 carry a zero weight.  The transposed product hands each lane
// four consecutive channels of one pixel, one 8-byte LDS store.
//
// conv2 is C[pos][co] = sum_k col[pos][k] W2[k][co] with k = tap*16 + ci
// (K = 144 padded to 160): a lane's eight k values are eight channels of one
// a1 pixel, one 16-byte LDS read; the weights stay in registers for the
// workgroup's lifetime.  Each lane then holds four consecutive positions of
// one output channel, one 8-byte store into a2[b][co*256 + pos].
//
// Split precision (PREC): every operand v of both convolutions is carried as
// two BF16 numbers, hi = bf16(v) and lo = bf16(v - hi) (16 significant bits;
// the crop L/256 is exact), and each product is hi*hi + hi*lo + lo*hi on
// MFMA (the lo*lo term is below FP32 resolution of the sum), so the ReLU
// pre-activations are FP32-accurate and a ReLU sees the sign the exact
// network gives; the outputs (a1 and the FC1 input) are stored as hi and lo.
#pragma once

#include "policy_kernels.h"

namespace aslam {
namespace pol {

using gemm::bf16x8;
using gemm::f32x4;

constexpr int kBlk = 33;                 // crop 2x2 blocks per row and column, plus the zero block -1
constexpr int kCropLds = kBlk * kBlk * 4;            // BF16 elements

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {   // one conversion of two
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)lo, (__bf16)hi});
}

// hi = bf16(v), or with LO the remainder bf16(v - hi).
template <bool LO>
__device__ __forceinline__ uint16_t bf16_part(float v) {
  const uint16_t h = f2bf(v);
  return LO ? f2bf(v - bf2f(h)) : h;
}

// conv1 weights as the A operand: lane supplies W'[co = lane % 16][k = 8 (lane / 16) + j].
template <bool LO = false>
__device__ __forceinline__ bf16x8 conv1_weight_frag(const float* w1, int lr, int lg) {
  uint16_t v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int k = 8 * lg + j;
    const int r = k >> 3, c = (k >> 2) & 1, dy = (k >> 1) & 1, dx = k & 1;
    const int ky = 2 * r + dy - 1, kx = 2 * c + dx - 1;
    v[j] = (lg < 2 && ky >= 0 && kx >= 0) ? bf16_part<LO>(w1[lr * 9 + ky * 3 + kx]) : (uint16_t)0;
  }
  uint4 u;
  u.x = v[0] | ((uint32_t)v[1] << 16);
  u.y = v[2] | ((uint32_t)v[3] << 16);
  u.z = v[4] | ((uint32_t)v[5] << 16);
  u.w = v[6] | ((uint32_t)v[7] << 16);
  return __builtin_bit_cast(bf16x8, u);
}

// conv2 weights as the B operand: lane supplies W2[k = 32 s + 8 (lane / 16) + j][co], k = tap*16 + ci.
template <bool LO = false>
__device__ __forceinline__ bf16x8 conv2_weight_frag(const float* w2, int co, int s, int lg) {
  uint16_t v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int k = 32 * s + 8 * lg + j, tap = k >> 4, ci = k & 15;
    v[j] = tap < 9 ? bf16_part<LO>(w2[(co * kC1 + ci) * 9 + tap]) : (uint16_t)0;
  }
  uint4 u;
  u.x = v[0] | ((uint32_t)v[1] << 16);
  u.y = v[2] | ((uint32_t)v[3] << 16);
  u.z = v[4] | ((uint32_t)v[5] << 16);
  u.w = v[6] | ((uint32_t)v[7] << 16);
  return __builtin_bit_cast(bf16x8, u);
}

// The forward's weight fragments, formed once per parameter update: fragment f < 11 of lane l at
// frag[64 f + l]; f = 0 is conv1's A operand, f = 1 + 5 nt + s is conv2's B operand for output
// channels 16 nt .. 16 nt + 15 and k slice s (the values conv1_weight_frag / conv2_weight_frag give).
// With LO the same fragments of the weights' lo parts, written from frag[64 kConvLoFrag] on.
constexpr int kConvFrags = 11;

template <bool LO = false>
__device__ __forceinline__ void conv_frag_elem(const float* prm, const Offsets& o, uint4* frag, int idx) {
  const int f = idx >> 6, lane = idx & 63, lr = lane & 15, lg = lane >> 4;
  bf16x8 v;
  if (f == 0) {
    v = conv1_weight_frag<LO>(prm + o.c1w, lr, lg);
  } else {
    const int nt = (f - 1) / 5, s = (f - 1) % 5;
    v = conv2_weight_frag<LO>(prm + o.c2w, 16 * nt + lr, s, lg);
  }
  frag[idx] = __builtin_bit_cast(uint4, v);
}

__global__ __launch_bounds__(64 * kConvFrags) void k_conv_frags(const float* prm, Offsets o, uint4* frag) {
  conv_frag_elem(prm, o, frag, threadIdx.x);
}

// A 64x64 int16 crop is 512 vectors of eight cells (row y = v / 8, columns
// 8 (v % 8) .. + 7); a workgroup of NT threads holds 512 / NT of them per
// thread in registers, so the next sample's crop can be in flight while the
// current one is processed.
template <int NT>
struct CropRegs {
  static constexpr int kPer = kCrop * kCrop / 8 / NT;
  int4 v[kPer];
};

template <int NT>
__device__ __forceinline__ void load_crop(const int16_t* src, CropRegs<NT>& r) {
  const int4* s4 = reinterpret_cast<const int4*>(src);
#pragma unroll
  for (int i = 0; i < CropRegs<NT>::kPer; ++i) r.v[i] = s4[threadIdx.x + i * NT];
}

// The lo parts of the crop registers' BF16(L / 256) into LDS, space-to-depth.  Block (Y, X)
// sits at ((Y + 1) * 33 + X + 1) * 4; the row and column of index 0 are the
// zero padding and are never written here.
template <int NT>
__device__ __forceinline__ void store_crop_lo(const CropRegs<NT>& r, uint16_t* s_crop) {
#pragma unroll
  for (int i = 0; i < CropRegs<NT>::kPer; ++i) {
    const int v = threadIdx.x + i * NT;
    const int y = v >> 3, x0 = (v & 7) * 8;
    const int32_t w[4] = {r.v[i].x, r.v[i].y, r.v[i].z, r.v[i].w};
    const int Y = y >> 1, dy = y & 1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float lo = (float)(int16_t)(w[q] & 0xffff) * (1.0f / 256.0f);
      const float hi = (float)(int16_t)(w[q] >> 16) * (1.0f / 256.0f);
      const int X = (x0 >> 1) + q;
      *reinterpret_cast<uint32_t*>(s_crop + ((Y + 1) * kBlk + X + 1) * 4 + 2 * dy) =
          (uint32_t)bf16_part<true>(lo) | ((uint32_t)bf16_part<true>(hi) << 16);
    }
  }
}

// Four ReLU outputs packed as BF16 (hi parts, or with LO the lo parts).
template <bool LO>
__device__ __forceinline__ uint2 pack_relu4(const f32x4& acc, const float b[4]) {
  uint16_t h[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) h[e] = bf16_part<LO>(fmaxf(acc[e] + b[e], 0.0f));
  return make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
}

// Bit e: the e-th of four packed ReLU outputs is > 0.
__device__ __forceinline__ uint32_t positive4(const uint2& h) {
  return ((h.x & 0x7fffu) ? 1u : 0u) | ((h.x & 0x7fff0000u) ? 2u : 0u) | ((h.y & 0x7fffu) ? 4u : 0u) |
         ((h.y & 0x7fff0000u) ? 8u : 0u);
}

// Encoder forward: a2[b * lda2 + co*256 + oy*16 + ox] = bf16(relu(conv2(relu(conv1(crop_b))))), and
// the rest of the FC1 input row: a2[b * lda2 + 8192 + j] = bf16(scan_b[j]), then bf16(state_b), then
// zeros up to lda2.  Input row b is rows[b] of crop / scan / state (b itself when rows is NULL).
// The workgroup loops over samples; the next sample's crop and the first 512 elements of its
// scan / state tail are loaded into registers while the current one is processed, so no global read
// is waited on inside a sample (a longer tail, R > 500, reads its remainder directly).
// MASK: amask receives conv2's ReLU mask for the backward, bit ox of word [b][co][oy] (bit n % 8 of byte
// n / 8 of the row's features n).
// PREC: a2lo receives the lo parts of the same row (conv features and the scan / state tail), the
// products are split as described at the top, and the workgroup holds the crop and a1 twice.
//
// What bounds it: a sample is a chain of two phases with a barrier behind each (conv1 reads the crop and
// writes a1, conv2 reads a1 while the next crop is stored), so a CU needs workgroups at different places
// of it.  Without border pixels the LDS of a sample is 40 KB (80 KB with PREC): four (two) workgroups of four
// waves per CU; the borders' zeros are put into the operands instead.  The tiles' LDS offsets are one
// base and immediate strides.  With borders (43.6 and 87 KB: three workgroups, one of eight waves) the
// kernel took 170 us on 9000 split-precision samples and 126 us on 16384 BF16 ones; it takes 152 and 122
// (109 without the mask).
constexpr int kConvFwdTailPre = 2;   // tail elements per thread held in registers

// The lo fragments of the split-precision path start at fragment kConvLoFrag (after the backward's).
constexpr int kConvLoFrag = 20;

constexpr int kConvFwdThreads = 256;
constexpr int kCropFwd = kA1 * kA1 * 4;      // BF16 elements: block (Y, X) at (Y * 32 + X) * 4
constexpr int kA1Fwd = kA1 * kA1 * kC1;
// a1 pixel (y, x) at (y * 32 + (x % 2) * 16 + x / 2) * 16, its two channel halves swapped when y / 2 is odd:
// conv2's stride-2 reads of four columns in each of two rows hit different banks.

// Crop registers into the forward's LDS copy (and, PREC, its lo parts), space-to-depth, as BF16(L / 256).
template <bool PREC>
__device__ __forceinline__ void store_crop_fwd(const CropRegs<kConvFwdThreads>& r, uint16_t* s_crop, uint16_t* s_cropl) {
#pragma unroll
  for (int i = 0; i < CropRegs<kConvFwdThreads>::kPer; ++i) {
    const int v = threadIdx.x + i * kConvFwdThreads;
    const int y = v >> 3, X0 = (v & 7) * 4;
    const int32_t w[4] = {r.v[i].x, r.v[i].y, r.v[i].z, r.v[i].w};
    const int at = ((y >> 1) * kA1 + X0) * 4 + 2 * (y & 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float lo = (float)(int16_t)(w[q] & 0xffff) * (1.0f / 256.0f);
      const float hi = (float)(w[q] >> 16) * (1.0f / 256.0f);
      *reinterpret_cast<uint32_t*>(s_crop + at + 4 * q) = (uint32_t)f2bf(lo) | ((uint32_t)f2bf(hi) << 16);
      if (PREC)
        *reinterpret_cast<uint32_t*>(s_cropl + at + 4 * q) =
            (uint32_t)bf16_part<true>(lo) | ((uint32_t)bf16_part<true>(hi) << 16);
    }
  }
}

template <bool PREC, bool MASK>
__global__ __launch_bounds__(kConvFwdThreads, PREC ? 2 : 4) void k_conv_fwd(
    const float* __restrict__ prm, Offsets o, const uint4* __restrict__ frag, const int16_t* __restrict__ crop,
    const float* __restrict__ scan, const float* __restrict__ state, int R, const int32_t* __restrict__ rows,
    uint16_t* __restrict__ a2, uint16_t* __restrict__ a2lo, int64_t lda2, int B, uint16_t* __restrict__ amask) {
  constexpr int NT = kConvFwdThreads, NW = NT / 64, kCopies = PREC ? 2 : 1;
  __shared__ __align__(16) uint16_t s_all[kCopies * (kCropFwd + kA1Fwd)];
  uint16_t* const s_a1 = s_all;
  uint16_t* const s_a1l = s_a1 + (PREC ? kA1Fwd : 0);
  uint16_t* const s_crop = s_all + kCopies * kA1Fwd;
  uint16_t* const s_cropl = s_crop + (PREC ? kCropFwd : 0);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const bf16x8 w1f = __builtin_bit_cast(bf16x8, frag[lane]);
  const bf16x8 w1fl = PREC ? __builtin_bit_cast(bf16x8, frag[64 * kConvLoFrag + lane]) : w1f;
  float b1[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) b1[i] = prm[o.c1b + 4 * lg + i];
  bf16x8 w2f[2][5], w2fl[2][5];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt)
#pragma unroll
    for (int s = 0; s < 5; ++s) {
      w2f[nt][s] = __builtin_bit_cast(bf16x8, frag[64 * (1 + 5 * nt + s) + lane]);
      if (PREC) w2fl[nt][s] = __builtin_bit_cast(bf16x8, frag[64 * (kConvLoFrag + 1 + 5 * nt + s) + lane]);
    }
  const float b2[2] = {prm[o.c2b + lr], prm[o.c2b + 16 + lr]};
  const int tail = (int)(lda2 - kFeat);
  auto src = [&](int b) -> int64_t { return rows ? (int64_t)rows[b] : (int64_t)b; };
  auto tail_value = [&](int64_t sb, int j) -> float {
    return j < R ? scan[sb * R + j] : (j < R + 12 ? state[sb * 12 + (j - R)] : 0.0f);
  };
  CropRegs<NT> cr;
  float tv[kConvFwdTailPre];
  auto load_sample = [&](int b) {
    const int64_t sb = src(b);
    load_crop<NT>(crop + sb * kCrop * kCrop, cr);
#pragma unroll
    for (int i = 0; i < kConvFwdTailPre; ++i) {
      const int j = threadIdx.x + NT * i;
      tv[i] = j < tail ? tail_value(sb, j) : 0.0f;
    }
  };
  auto store_sample = [&](int b) {   // the loaded sample's crop into LDS, its tail into the output row
    store_crop_fwd<PREC>(cr, s_crop, s_cropl);
    uint16_t* row = a2 + (int64_t)b * lda2 + kFeat;
    uint16_t* rowl = PREC ? a2lo + (int64_t)b * lda2 + kFeat : row;
#pragma unroll
    for (int i = 0; i < kConvFwdTailPre; ++i) {
      const int j = threadIdx.x + NT * i;
      if (j < tail) {
        row[j] = j < R + 12 ? f2bf(tv[i]) : (uint16_t)0;
        if (PREC) rowl[j] = j < R + 12 ? bf16_part<true>(tv[i]) : (uint16_t)0;
      }
    }
    for (int j = threadIdx.x + NT * kConvFwdTailPre; j < tail; j += NT) {
      const float v = j < R + 12 ? tail_value(src(b), j) : 0.0f;
      row[j] = f2bf(v);
      if (PREC) rowl[j] = bf16_part<true>(v);
    }
  };
  // conv1: the wave's tile j covers the 16 pixels of row y = 8 wave + j / 2 from column 16 (j % 2); its window
  // operand is the blocks (y - 1 + lg, x - 1) and (.., x) for the lanes with lg < 2, zeros for the rest, above
  // the first row and left of the first column
  const int y0 = kA1 / NW * wave;
  const int win0 = ((y0 - 1 + lg) * kA1 + lr) * 4, slot0 = (y0 * kA1 + (lr & 1) * 16 + (lr >> 1)) * kC1 + 4 * lg;
  static_assert((kA1 / NW) % 4 == 0, "the halves' swap of a wave's row y0 + q is that of row q");
  auto window = [&](const uint16_t* c, int j) -> uint4 {
    if (lg >= 2 || (lg == 0 && y0 + (j >> 1) == 0)) return make_uint4(0u, 0u, 0u, 0u);
    const uint16_t* q = c + win0 + ((j >> 1) * kA1 + (j & 1) * 16) * 4;
    const uint2 d = *reinterpret_cast<const uint2*>(q);
    uint2 a = make_uint2(0u, 0u);
    if ((j & 1) || lr > 0) a = *reinterpret_cast<const uint2*>(q - 4);
    return make_uint4(a.x, a.y, d.x, d.y);
  };
  // conv2: the wave's four output rows, as four tiles: row m = 4 q + e of tile i is the output (oy = 4 wave + q,
  // ox = 4 i + e), so that a lane ends up with the 16 outputs of one row of its channel.  Operand of k slice s
  // for this lane (a tap and a channel half); rows above and columns left of the image are zeros.
  static_assert(kA2 / NW == 4, "a wave's four output rows");
  int c2_off[5];
  bool c2_ok[5], c2_first[5];   // inside; inside also in the first tile
#pragma unroll
  for (int s = 0; s < 5; ++s) {
    const int k0 = 32 * s + 8 * lg, tap = k0 >> 4, half = (k0 >> 3) & 1;
    const int y = 2 * (4 * wave + (lr >> 2)) + tap / 3 - 1, x = 2 * (lr & 3) + tap % 3 - 1;
    c2_ok[s] = tap < 9 && y >= 0;
    c2_first[s] = c2_ok[s] && x >= 0;
    c2_off[s] = (y * kA1 + (x & 1) * 16 + (x >> 1)) * kC1 + 8 * (half ^ ((y >> 1) & 1));
  }
  auto col_frag = [&](const uint16_t* a, int i, int s) -> bf16x8 {
    uint4 u = make_uint4(0u, 0u, 0u, 0u);
    if (i > 0 ? c2_ok[s] : c2_first[s]) u = *reinterpret_cast<const uint4*>(a + c2_off[s] + i * 4 * kC1);
    return __builtin_bit_cast(bf16x8, u);
  };
  if (blockIdx.x < B) {
    load_sample(blockIdx.x);
    store_sample(blockIdx.x);
    if (blockIdx.x + gridDim.x < B) load_sample(blockIdx.x + gridDim.x);
  }
  __syncthreads();
  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    // conv1 + ReLU into a1, four tiles at a time so that their operand reads are in flight together
#pragma unroll
    for (int j0 = 0; j0 < kA1 * kA1 / 16 / NW; j0 += 4) {
      uint4 u[4], ul[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        u[i] = window(s_crop, j0 + i);
        if (PREC) ul[i] = window(s_cropl, j0 + i);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1f, __builtin_bit_cast(bf16x8, u[i]),
                                                           f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        if (PREC) {
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1f, __builtin_bit_cast(bf16x8, ul[i]), acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1fl, __builtin_bit_cast(bf16x8, u[i]), acc, 0, 0, 0);
        }
        const int q = (j0 + i) >> 1;
        const int at = (slot0 + (q * kA1 + ((j0 + i) & 1) * 8) * kC1) ^ ((q & 2) ? 8 : 0);
        *reinterpret_cast<uint2*>(s_a1 + at) = pack_relu4<false>(acc, b1);
        if (PREC) *reinterpret_cast<uint2*>(s_a1l + at) = pack_relu4<true>(acc, b1);
      }
    }
    __syncthreads();
    // the next sample's crop takes the place of the one just used, the one after is loaded
    if (b + (int)gridDim.x < B) {
      store_sample(b + gridDim.x);
      if (b + 2 * (int)gridDim.x < B) load_sample(b + 2 * gridDim.x);
    }
    f32x4 acc[2][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[0][i] = acc[1][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 5; ++s) {
        const bf16x8 af = col_frag(s_a1, i, s);
        acc[0][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, w2f[0][s], acc[0][i], 0, 0, 0);
        acc[1][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, w2f[1][s], acc[1][i], 0, 0, 0);
        if (PREC) {
          const bf16x8 afl = col_frag(s_a1l, i, s);
          acc[0][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, w2fl[0][s], acc[0][i], 0, 0, 0);
          acc[1][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, w2fl[1][s], acc[1][i], 0, 0, 0);
          acc[0][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afl, w2f[0][s], acc[0][i], 0, 0, 0);
          acc[1][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afl, w2f[1][s], acc[1][i], 0, 0, 0);
        }
      }
    }
    // row oy = 4 wave + lg of channels lr and 16 + lr: 32 bytes a lane, the wave's rows of a channel one line
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float bb[4] = {b2[h], b2[h], b2[h], b2[h]};
      const int64_t off = (int64_t)b * lda2 + (16 * h + lr) * 256 + (4 * wave + lg) * kA2;
      uint2 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = pack_relu4<false>(acc[h][i], bb);
      reinterpret_cast<uint4*>(a2 + off)[0] = make_uint4(v[0].x, v[0].y, v[1].x, v[1].y);
      reinterpret_cast<uint4*>(a2 + off)[1] = make_uint4(v[2].x, v[2].y, v[3].x, v[3].y);
      if (MASK)
        amask[((int64_t)b * kC2 + 16 * h + lr) * kA2 + 4 * wave + lg] =
            (uint16_t)(positive4(v[0]) | (positive4(v[1]) << 4) | (positive4(v[2]) << 8) | (positive4(v[3]) << 12));
      if (PREC) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = pack_relu4<true>(acc[h][i], bb);
        reinterpret_cast<uint4*>(a2lo + off)[0] = make_uint4(v[0].x, v[0].y, v[1].x, v[1].y);
        reinterpret_cast<uint4*>(a2lo + off)[1] = make_uint4(v[2].x, v[2].y, v[3].x, v[3].y);
      }
    }
    __syncthreads();
  }
}

}  // namespace pol
}  // namespace aslam

namespace aslam {
namespace pol {

// ------------------------------------------------------------ encoder backward
//
// One kernel for everything below the FC1 input gradient, per sample b:
//   conv1 is recomputed from the crop; with dz2 = dL/d(conv2 pre-activation)
//   (BF16 [b][co][pos], already masked by conv2's ReLU),
//   dW2[co][ci][tap] += sum_pos dz2[co][pos] a1[ci][pixel(pos, tap)]
//   da1[ci][y][x]     = sum_{co, tap} W2[co][ci][tap] dz2[co][pos(y, x, tap)]
//   dz1 = bf16(da1) * [a1 > 0]
//   dW1[co][tap]     += sum_px dz1[co][px] in[pixel(px, tap)]
//   db1 += sum dz1,  db2 += sum dz2.
// The workgroup (four waves) keeps its gradient sums over all its samples and
// writes them once, as partials [gridDim.x][kConvPart], reduced afterwards in
// a fixed order.
//
// What bounds it: a sample is a chain of three phases (stage the crop and dz2; conv1; the products) with a
// barrier behind each, so a CU holds two workgroups that are at different places of it (77 KB of LDS; 68 in
// BF16), and the vector instructions: the operands come from LDS in the layout that they arrive in, transposed by the
// read where the product contracts over the other index (ds_read_b64_tr_b16: of a group's 16 lanes, lane
// 4 r + c reads four elements of row r, lane i receives element i of the four rows), and the bias sums are
// products with ones.  One workgroup of eight waves with transposed copies in LDS (three shifted planes of a1,
// five of the crop, two of dz2: 127 KB, 560 vector instructions a wave and sample) took 187 us on 9000
// split-precision samples, 267 on 16384 BF16 ones and 36 on 96; this takes 111, 171 and 11.
//
// LDS layouts (BF16):
//   crop   cell (y, x) at row y + 2 (rows of 128 bytes, rows 0 and 1 zero), column x of copy A and column x + 2
//          of copy B (its columns 0 and 1 zero): four consecutive cells from any even column are eight aligned
//          bytes of one copy.  The 64-byte halves of row r are swapped when r / 2 is odd, and B starts 128 bytes
//          past A's last row, so that conv1's and dW1's reads of two row pairs and both copies cover all banks.
//   a1     pixel (y, x), 16 channels of 32 bytes, at row y + 1 (row 0 zero): the even columns, 48 bytes of zeros,
//          the odd columns: a product's reads of 8 positions along x are 256 contiguous bytes, and conv1's stores
//          of 16 pixels' channel halves cover all banks.
//   dz     [co][pos], rows of 512 bytes; the 32-byte blocks oy of a channel's row at oy ^ f(co), f = co % 4 +
//          4 (co / 8 % 2): the transposing read of channels 8 g .. 8 g + 3 covers all banks.
// dW2: K = 32 positions, k = 8 lg + 4 h + r <-> (oy = 4 wave + 2 s + h, ox = 4 lg + r), s the wave's k-step.
// da1 is computed one sub-pixel phase (y % 2, x % 2) at a time: the input
// pixels of a phase form a 16 x 16 grid that receives taps ky = 1 (y even) or
// ky in {0, 2} (y odd), likewise kx, each from the output position
// (qy + (py + 1 - ky) / 2, qx + (px + 1 - kx) / 2).  K = 32 channels per tap.  The operands of the positions
// one to the right are those of the positions moved by a lane.
// dz1 = bf16(da1) * [a1 > 0] never leaves registers: a lane holds channel
// lr at the pixels 4 lg + i of the phase rows qy = wave + 4 rr, and
// those of two rows are exactly its A operand of one dW1 MFMA, so dW1 is accumulated right after each
// phase's da1 products.  dW1's columns are 4 ky + kx + 1.
constexpr int kConvPartW2 = kC2 * 144;          // [co][tap*16 + ci]
constexpr int kConvPartW1 = kC1 * 16;           // [co][tap], taps padded to 16
constexpr int kConvPart = kConvPartW2 + kConvPartW1 + kC1 + kC2;
constexpr int kBwdThreads = 256;
constexpr int kCropRow = 2 * kCrop, kCropB = (kCrop + 3) * kCropRow;   // bytes: a row, copy B
constexpr int kCropBytes = kCropB + (kCrop + 3) * kCropRow;            // (a row past the end for dW1's unused columns)
constexpr int kA1Pix = 2 * kC1, kA1Odd = 17 * kA1Pix + 16, kA1RowB = kA1Odd + 16 * kA1Pix, kA1Bytes = 33 * kA1RowB;
constexpr int kDzRowB = 512, kDzBytes = kC2 * kDzRowB;

struct PhaseTaps {
  int n;                 // taps of the phase (1, 2 or 4)
  int ky[4], kx[4], dy[4], dx[4];
};

__device__ __forceinline__ PhaseTaps phase_taps(int py, int px) {
  PhaseTaps t;
  const int nky = py ? 2 : 1, nkx = px ? 2 : 1;
  t.n = nky * nkx;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int iy = j / nkx, ix = j % nkx;
    const int ky = py ? 2 * iy : 1, kx = px ? 2 * ix : 1;
    t.ky[j] = ky; t.kx[j] = kx;
    t.dy[j] = (py + 1 - ky) / 2; t.dx[j] = (px + 1 - kx) / 2;
  }
  return t;
}

// B operand of the phase product for k-step (phase, j): lane supplies
// W2[co = 8 lg + e][ci = lr][ky_j][kx_j], e < 8.
__device__ __forceinline__ bf16x8 phase_weight_frag(const float* w2, int ky, int kx, int lr, int lg) {
  uint16_t v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = f2bf(w2[((8 * lg + e) * kC1 + lr) * 9 + ky * 3 + kx]);
  uint4 u;
  u.x = v[0] | ((uint32_t)v[1] << 16);
  u.y = v[2] | ((uint32_t)v[3] << 16);
  u.z = v[4] | ((uint32_t)v[5] << 16);
  u.w = v[6] | ((uint32_t)v[7] << 16);
  return __builtin_bit_cast(bf16x8, u);
}

// The backward's phase weight fragments, formed once per parameter update after the forward's
// kConvFrags: fragment kConvFrags + q of lane l at frag[64 (kConvFrags + q) + l], q enumerating the
// (phase, tap) pairs in phase order (9 in all).
constexpr int kConvPhaseFrags = 9;
static_assert(kConvLoFrag == kConvFrags + kConvPhaseFrags, "lo fragments follow the backward's");

__device__ __forceinline__ void conv_bwd_frag_elem(const float* prm, const Offsets& o, uint4* frag, int idx) {
  const int f = idx >> 6, lane = idx & 63, lr = lane & 15, lg = lane >> 4;
  int q = 0;
#pragma unroll
  for (int ph = 0; ph < 4; ++ph) {
    const PhaseTaps t = phase_taps(ph >> 1, ph & 1);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (j < t.n) {
        if (q == f)
          frag[64 * (kConvFrags + q) + lane] =
              __builtin_bit_cast(uint4, phase_weight_frag(prm + o.c2w, t.ky[j], t.kx[j], lr, lg));
        ++q;
      }
    }
  }
}

__global__ __launch_bounds__(64 * kConvPhaseFrags) void k_conv_bwd_frags(const float* prm, Offsets o, uint4* frag) {
  conv_bwd_frag_elem(prm, o, frag, threadIdx.x);
}

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4_t lds_short4;

__device__ __forceinline__ uint2 read_tr(const unsigned char* p) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)p));
}

// Each lane of 16 gets the next one's value, the last one zero.
__device__ __forceinline__ uint32_t next_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x101, 0xf, 0xf, true);
}

// Two gradients as BF16 where the two activations a (BF16, not negative) are not zero.
__device__ __forceinline__ uint32_t masked2(uint32_t a, float lo, float hi) {
  // two 16-bit operations each (in C++ they become a compare and a select per value); the matrix cores must
  // not read an asm's result directly, the wait that takes is the compiler's to insert
  uint32_t on, mask;
  asm("v_pk_min_u16 %0, %1, %2" : "=v"(on) : "v"(a & 0x7fff7fffu), "v"(0x00010001u));
  asm("v_pk_mul_lo_u16 %0, %1, %2" : "=v"(mask) : "v"(on), "v"(0xffffffffu));
  return mask & pack_bf16x2(lo, hi);
}

// PREC: conv1 is recomputed with split operands (the crop's lo part staged beside it), so its ReLU
// mask is the one the split forward applied; the products of the backward stay BF16.
template <bool PREC>
__global__ __launch_bounds__(kBwdThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_conv_bwd(
    const float* __restrict__ prm, Offsets o, const uint4* __restrict__ frag, const int16_t* __restrict__ crop,
    const int32_t* __restrict__ rows, const uint16_t* __restrict__ dz2c, int B, float* __restrict__ part) {
  __shared__ __align__(256) unsigned char s_crop[kCropBytes];
  __shared__ __align__(256) unsigned char s_a1[kA1Bytes];
  __shared__ __align__(256) unsigned char s_dz[kDzBytes];
  __shared__ __align__(16) uint16_t s_cropl[PREC ? (kCropLds + 7) / 8 * 8 : 8];   // space-to-depth, with its border
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  {
    uint4* z = reinterpret_cast<uint4*>(s_crop);
    for (int i = threadIdx.x; i < kCropBytes / 16; i += kBwdThreads) z[i] = make_uint4(0u, 0u, 0u, 0u);
    z = reinterpret_cast<uint4*>(s_a1);
    for (int i = threadIdx.x; i < kA1Bytes / 16; i += kBwdThreads) z[i] = make_uint4(0u, 0u, 0u, 0u);
    if (PREC) {
      z = reinterpret_cast<uint4*>(s_cropl);
      for (int i = threadIdx.x; i < (kCropLds + 7) / 8; i += kBwdThreads) z[i] = make_uint4(0u, 0u, 0u, 0u);
    }
  }
  // registers that live for the whole workgroup
  // conv1's weights with k in the order of the window's reads, 4 dy + 2 c + dx (the sum is the same, bit for bit)
  auto w1_frag = [&](int f) {
    const uint4 w = frag[64 * f + lane];
    return __builtin_bit_cast(bf16x8, make_uint4(w.x, w.z, w.y, w.w));
  };
  const bf16x8 w1f = w1_frag(0), w1fl = PREC ? w1_frag(kConvLoFrag) : w1f;
  float b1[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) b1[i] = prm[o.c1b + 4 * lg + i];
  bf16x8 wph[kConvPhaseFrags];
#pragma unroll
  for (int q = 0; q < kConvPhaseFrags; ++q) wph[q] = __builtin_bit_cast(bf16x8, frag[64 * (kConvFrags + q) + lane]);
  const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  // sums over the workgroup's samples: dW2 [tap][output-channel half], dW1, the biases (the same in every column)
  f32x4 gw2[9][2], gw1 = zero4, gb1 = zero4, gb2[2] = {zero4, zero4};
#pragma unroll
  for (int a = 0; a < 9; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c) gw2[a][c] = zero4;
  f32x4 c0 = zero4;   // in registers of its own: as a constant it is written before each product that starts from it
  asm("" : "+v"(c0));
  // the sample's crop and dz2 in registers; the next sample's are loaded while this one is processed
  CropRegs<kBwdThreads> cr;
  gemm::u32x4 dzr[4];
  auto load_sample = [&](int bb) {
    load_crop<kBwdThreads>(crop + (rows ? (int64_t)rows[bb] : (int64_t)bb) * kCrop * kCrop, cr);
    const gemm::u32x4* src = reinterpret_cast<const gemm::u32x4*>(dz2c + (int64_t)bb * kFeat);
#pragma unroll
    for (int i = 0; i < 4; ++i) dzr[i] = src[threadIdx.x + i * kBwdThreads];
  };
  // staging: the thread's crop vectors are eight cells of rows y and y + 32, its dz2 vectors eight positions
  // (half a block) of channels co, co + 8, ..
  const int q8 = threadIdx.x & 7, row = (int)(threadIdx.x >> 3) + 2, swap = ((row >> 1) & 1) * 64;
  unsigned char* const st_a = s_crop + row * kCropRow + ((16 * q8) ^ swap);
  unsigned char* const st_b = s_crop + kCropB + row * kCropRow;
  const int co = threadIdx.x >> 5;   // 0 .. 7
  const int st_dz = co * kDzRowB + (((((int)threadIdx.x & 31) >> 1) ^ (co & 3)) << 5) + 16 * (threadIdx.x & 1);
  // conv1's windows: odd columns from copy A, even ones from copy B; lanes with lg >= 2 read what lg - 2 reads
  // (finite values; their weights are zero)
  const int l1 = lg & 1;
  const unsigned char* const win = s_crop + ((lr & 1) ? 4 * lr - 4 : kCropB + 4 * lr) + (16 * wave + 2 * l1) * kCropRow;
  const unsigned char* const win2[2] = {win + 64 * l1, win + 64 * (l1 ^ 1)};
  const uint16_t* const winl = s_cropl + ((8 * wave + l1) * kBlk + lr) * 4;
  unsigned char* const st_a1 = s_a1 + (8 * wave + 1) * kA1RowB + (lr & 1) * kA1Odd + (lr >> 1) * kA1Pix + 8 * lg;
  // transposing reads: this lane's row (lr / 4) and four elements (lr % 4)
  const int tr = lr >> 2, tc = lr & 3;
  const unsigned char* const px0 = s_a1 + (4 * lg + tr) * kA1Pix + 8 * tc;           // positions 4 lg + r along x
  const uint32_t dzt = (8 * lg + tr) * kDzRowB + ((tr | (l1 << 2)) << 5) + 8 * tc;   // channels 8 lg + r, block ^ oy
  const uint32_t dza = lr * kDzRowB + (((lr & 3) | ((lr >> 3) << 2)) << 5) + 8 * lg;   // channel lr, positions 4 lg ..
  const unsigned char* in2[2];   // dW1's cells at phase row py: rows 4 wave + ky - 1 (+ 2 py), columns 16 lg + 4 r ..
#pragma unroll
  for (int py = 0; py < 2; ++py)
    in2[py] = s_crop + (4 * wave + tc + 1 + 2 * py) * kCropRow + ((32 * lg + 8 * tr) ^ (64 * (py ^ ((tc + 1) >> 1 & 1))));
  if (blockIdx.x < B) load_sample(blockIdx.x);
  __syncthreads();

  for (int b = blockIdx.x; b < B; b += gridDim.x) {
    // ---- stage the crop and dz2
    if (PREC) store_crop_lo(cr, s_cropl);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int32_t w[4] = {cr.v[i].x, cr.v[i].y, cr.v[i].z, cr.v[i].w};
      uint32_t c[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        c[j] = pack_bf16x2((float)(int16_t)(w[j] & 0xffff) * (1.0f / 256.0f), (float)(w[j] >> 16) * (1.0f / 256.0f));
      const int at = i * 32 * kCropRow;
      *reinterpret_cast<uint4*>(st_a + at) = make_uint4(c[0], c[1], c[2], c[3]);
      *reinterpret_cast<uint32_t*>(st_b + at + ((16 * q8 + 4) ^ swap)) = c[0];
      *reinterpret_cast<uint2*>(st_b + at + ((16 * q8 + 8) ^ swap)) = make_uint2(c[1], c[2]);
      if (q8 < 7) *reinterpret_cast<uint32_t*>(st_b + at + ((16 * q8 + 16) ^ swap)) = c[3];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)   // channel co + 8 i: block bit 2 flips with i
      *reinterpret_cast<gemm::u32x4*>(s_dz + ((st_dz ^ ((i & 1) * 128)) + i * 8 * kDzRowB)) = dzr[i];
    __syncthreads();
    if (b + (int)gridDim.x < B) load_sample(b + gridDim.x);
    // ---- conv1 recompute: C'[co][px], the wave's tile j the 16 pixels of row y = 8 wave + j / 2 from column
    // 16 (j % 2), four tiles at a time so that their operand reads overlap
#pragma unroll
    for (int j0 = 0; j0 < 16; j0 += 4) {
      bf16x8 u[4], ul[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = j0 + i;
        // bit 6 of the column is (j ^ l1 ^ j / 2) % 2
        const unsigned char* q = win2[(j ^ (j >> 1)) & 1] + (j >> 1) * 2 * kCropRow;
        const uint2 a = *reinterpret_cast<const uint2*>(q), c = *reinterpret_cast<const uint2*>(q + kCropRow);
        u[i] = __builtin_bit_cast(bf16x8, make_uint4(a.x, a.y, c.x, c.y));
        if (PREC) {
          const uint16_t* ql = winl + ((j >> 1) * kBlk + 16 * (j & 1)) * 4;
          const uint2 e = *reinterpret_cast<const uint2*>(ql), f = *reinterpret_cast<const uint2*>(ql + 4);
          ul[i] = __builtin_bit_cast(bf16x8, make_uint4(e.x, f.x, e.y, f.y));
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = j0 + i;
        f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1f, u[i], c0, 0, 0, 0);
        if (PREC) {
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1f, ul[i], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1fl, u[i], acc, 0, 0, 0);
        }
        *reinterpret_cast<uint2*>(st_a1 + (j >> 1) * kA1RowB + (j & 1) * 8 * kA1Pix) = pack_relu4<false>(acc, b1);
      }
    }
    __syncthreads();
    // ---- dW2: the wave's two k-steps of 32 positions for all nine taps; db2
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8 af[2];
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        uint2 v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
          v[h] = *reinterpret_cast<const uint2*>(s_dz + (dza ^ (uint32_t)((4 * wave + 2 * s + h) << 5)) + mt * 16 * kDzRowB);
        af[mt] = __builtin_bit_cast(bf16x8, make_uint4(v[0].x, v[0].y, v[1].x, v[1].y));
        gb2[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[mt], ones, gb2[mt], 0, 0, 0);
      }
#pragma unroll
      for (int nt = 0; nt < 9; ++nt) {
        const int ky = nt / 3, kx = nt % 3;
        uint2 v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)   // row 2 oy + ky - 1, columns 2 ox + kx - 1
          v[h] = read_tr(px0 + (8 * wave + 4 * s + 2 * h + ky) * kA1RowB + (kx == 1 ? 0 : kx == 2 ? kA1Odd : kA1Odd - kA1Pix));
        const bf16x8 bf = __builtin_bit_cast(bf16x8, make_uint4(v[0].x, v[0].y, v[1].x, v[1].y));
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
          gw2[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[mt], bf, gw2[nt][mt], 0, 0, 0);
      }
    }
    // ---- da1 by phases -> dz1 (masked, BF16, in registers); db1; dW1.  Two of the wave's rows qy = wave + 4 rr
    // at a time
#pragma unroll
    for (int r2 = 0; r2 < 2; ++r2) {
      bf16x8 pos[2][2][2];   // [row of the pair][dy][dx]
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int dy = 0; dy < 2; ++dy) {
          const int oy = wave + 4 * (2 * r2 + k) + dy;
          uint4 v = make_uint4(0u, 0u, 0u, 0u);
          if (oy < kA2) {
            const unsigned char* q = s_dz + (dzt ^ (uint32_t)(oy << 5));
            const uint2 a = read_tr(q), c = read_tr(q + 4 * kDzRowB);
            v = make_uint4(a.x, a.y, c.x, c.y);
          }
          pos[k][dy][0] = __builtin_bit_cast(bf16x8, v);
          pos[k][dy][1] = __builtin_bit_cast(bf16x8, make_uint4(next_lane(v.x), next_lane(v.y), next_lane(v.z), next_lane(v.w)));
        }
      int q = 0;
#pragma unroll
      for (int ph = 0; ph < 4; ++ph) {
        const int py = ph >> 1, px = ph & 1;
        const PhaseTaps t = phase_taps(py, px);
        uint2 d[2], in[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int rr = 2 * r2 + k;
          f32x4 acc = c0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (j >= t.n) break;
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pos[k][t.dy[j]][t.dx[j]], wph[q + j], acc, 0, 0, 0);
          }
          // lane: input pixels (2 qy + py, 2 (4 lg + i) + px), channel lr
          const uint2 m = read_tr(px0 + (2 * wave + 8 * rr + py + 1) * kA1RowB + px * kA1Odd);
          d[k] = make_uint2(masked2(m.x, acc[0], acc[1]), masked2(m.y, acc[2], acc[3]));
          in[k] = read_tr(in2[py] + 16 * rr * kCropRow + (px ? 0 : kCropB));
        }
        q += t.n;
        const bf16x8 df = __builtin_bit_cast(bf16x8, make_uint4(d[0].x, d[0].y, d[1].x, d[1].y));
        gw1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            df, __builtin_bit_cast(bf16x8, make_uint4(in[0].x, in[0].y, in[1].x, in[1].y)), gw1, 0, 0, 0);
        gb1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(df, ones, gb1, 0, 0, 0);
      }
    }
    __syncthreads();
  }

  // ---- write the workgroup's partial sums (fixed order everywhere), the waves' summed in wave order through LDS
  constexpr int NW = kBwdThreads / 64;
  float* out = part + (int64_t)blockIdx.x * kConvPart;
  float* st = reinterpret_cast<float*>(s_a1);   // free after the sample loop
  static_assert(NW * 3 * 512 * 4 <= kA1Bytes && NW * (256 + kC1 + kC2) * 4 <= kDzBytes, "the sums' staging");
  // dW2 [co][nt*16 + ci]: lane value C[4 lg + i][lr] of tile (nt, mt) = (co = 16 mt + 4 lg + i, ci = lr), three taps
  // at a time
#pragma unroll
  for (int g = 0; g < 3; ++g) {
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) st[((wave * 3 + j) * 32 + 16 * mt + 4 * lg + i) * 16 + lr] = gw2[3 * g + j][mt][i];
    __syncthreads();
    for (int e = threadIdx.x; e < 3 * 512; e += kBwdThreads) {
      const int j = e >> 9, r = e & 511;
      float sum = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) sum += st[(w * 3 + j) * 512 + r];
      out[(r >> 4) * 144 + (3 * g + j) * 16 + (r & 15)] = sum;
    }
    __syncthreads();
  }
  // dW1 [co][tap] and the biases
  float* sb = reinterpret_cast<float*>(s_dz) + wave * (256 + kC1 + kC2);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int c = 4 * lg + i;
    if ((lr & 3) > 0 && lr < 12) sb[c * 16 + (lr >> 2) * 3 + (lr & 3) - 1] = gw1[i];
    else sb[c * 16 + (lr < 12 ? 9 + (lr >> 2) : lr)] = 0.0f;   // taps 9 .. 15
    if (lr == 0) {
      sb[256 + c] = gb1[i];
      sb[256 + kC1 + c] = gb2[0][i];
      sb[256 + kC1 + 16 + c] = gb2[1][i];
    }
  }
  __syncthreads();
  static_assert(kConvPartW1 == 256, "dW1, db1 and db2 are consecutive in the partials");
  for (int e = threadIdx.x; e < 256 + kC1 + kC2; e += kBwdThreads) {
    const float* q = reinterpret_cast<const float*>(s_dz) + e;
    float sum = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) sum += q[w * (256 + kC1 + kC2)];
    out[kConvPartW2 + e] = sum;
  }
}

}  // namespace pol
}  // namespace aslam
