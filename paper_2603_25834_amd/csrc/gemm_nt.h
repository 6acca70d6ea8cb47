// gemm_nt.h -- BF16 GEMM with both operands contiguous along k, for gfx950 (library-internal).
//
// C[m][n] = sum_k X[m][k] W[n][k] (FP32 accumulation), X the activations [M][K], W the weights [N][K], K and
// the leading dimensions multiples of 64, rows on 128-byte boundaries (a row that starts inside a cache
// line costs a second one per 128 bytes: 133 -> 92 us at M = 16384, K = 8576).  NP = 1: one product.
// NP = 3: the split-precision products X_hi W_hi, X_hi W_lo, X_lo W_hi, each into an accumulator of its own
// (the caller adds them in a fixed order).  K may be split over z.
//
// What bounds the 128 x 128 tile this takes the place of for the wide products: four waves of 64 x 64
// read as many LDS bytes per cycle as the LDS delivers, twice the operand bytes for three products in
// turn, and stage through registers.  Here a workgroup of eight waves owns 128 x 256 of C (64 x 64 a
// wave), one per CU; a stage of 48 KB holds 64 k (NP = 1), or 32 k of the hi and the lo parts (NP = 3: the
// three products share one staging, 16 fragment reads feed 48 MFMAs), three stages in LDS.  Global reads
// go straight to LDS (16 bytes a lane), two stages ahead, one barrier a stage; the wait counts exactly the
// newest stage's reads.  The 16-byte chunks of a row are permuted by the choice of the chunk each lane
// reads, so that the eight lanes of a fragment read's cycle cover all banks.  What bounds it now is the
// way from L2 and HBM: without the reads the same loop takes 48 us (1.5 PFLOP/s), the reads alone 75-84 us
// of the 86 us at M = 16384, K = 8576, two K slices (138 us before); NP = 3 at M = 9000, three slices:
// 229 -> 154 us (kernel alone).
//
// The fragments of W are the MFMA's row operand: a lane ends up with four consecutive n of one m (16-byte
// stores).  Products and their order along k are those of gemm_bf16.h's engine.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "gemm_bf16.h"

namespace aslam {
namespace gemm_nt {

using gemm::bf16x8;
using gemm::f32x4;

constexpr int kBM = 128, kBN = 256, kThreads = 512;
constexpr int kSubX = kBM * 64, kSubW = kBN * 64;          // bytes of a sub-tile (32 k)
constexpr int kStageBytes = 2 * (kSubX + kSubW);

struct Operands {
  const uint16_t *x, *x_lo;   // [M][ldx] (x_lo: NP = 3)
  const uint16_t *w, *w_lo;   // [N][ldw]
  int64_t ldx, ldw;
  int M, N, K;
};

typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) char* glb_bytes;

__device__ __forceinline__ void to_lds(glb_bytes base, uint32_t off, void* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base + off), (lds_void*)dst, 16, 0, 0);
}

// Eight waves' reads of one stage into LDS.  NP = 1: rows of 128 bytes (64 k); wave w takes rows 8 w .. and
// 64 + 8 w .. of X and 8 w + 64 q .. of W, lane l the chunk (l % 8) ^ ((l / 8) % 8) of row l / 8.
// NP = 3: rows of 64 bytes, the hi sub-tile then the lo one; wave w takes rows 16 w .. of both parts of X
// and 16 w .. and 128 + 16 w .. of W, lane l the chunk (l % 4) ^ ((l / 8) % 4) of row l / 4.  Rows past M
// read the last one.
template <int NP>
struct Loader;

template <>
struct Loader<1> {
  glb_bytes x0, w0;            // the tile's first row at the next stage's k
  uint32_t ox0, ox1, ow;       // this lane's byte offsets
  int64_t wq;                  // 64 rows of W
  int wave;

  __device__ __forceinline__ Loader(const Operands& o, int m0, int n0, int kb, int wave_) : wave(wave_) {
    const int lane = threadIdx.x & 63;
    const int row = 8 * wave + (lane >> 3), kc = 8 * ((lane & 7) ^ ((lane >> 3) & 7));
    x0 = (glb_bytes)(o.x + (int64_t)m0 * o.ldx + kb);
    w0 = (glb_bytes)(o.w + (int64_t)n0 * o.ldw + kb);
    ox0 = (uint32_t)((int64_t)min(row, o.M - 1 - m0) * o.ldx + kc) * 2u;
    ox1 = (uint32_t)((int64_t)min(row + 64, o.M - 1 - m0) * o.ldx + kc) * 2u;
    ow = (uint32_t)((int64_t)row * o.ldw + kc) * 2u;
    wq = (int64_t)64 * o.ldw * 2;
  }
  __device__ __forceinline__ void issue(unsigned char* buf) {
    unsigned char* dx = buf + wave * 1024;
    unsigned char* dw = buf + 2 * kSubX + wave * 1024;
    to_lds(x0, ox0, dx);
    to_lds(x0, ox1, dx + 8192);
    to_lds(w0, ow, dw);
    to_lds(w0 + wq, ow, dw + 8192);
    to_lds(w0 + 2 * wq, ow, dw + 2 * 8192);
    to_lds(w0 + 3 * wq, ow, dw + 3 * 8192);
    x0 += 128; w0 += 128;
  }
};

template <>
struct Loader<3> {
  glb_bytes x0, x1, w0, w1;        // the tile's first row at the next stage's k (hi and lo parts)
  uint32_t ox, ow;                 // this lane's byte offset
  int64_t w_half;                  // 128 rows of W
  int wave;

  __device__ __forceinline__ Loader(const Operands& o, int m0, int n0, int kb, int wave_) : wave(wave_) {
    const int lane = threadIdx.x & 63;
    const int row = 16 * wave + (lane >> 2), kc = 8 * ((lane & 3) ^ ((lane >> 3) & 3));
    x0 = (glb_bytes)(o.x + (int64_t)m0 * o.ldx + kb);
    w0 = (glb_bytes)(o.w + (int64_t)n0 * o.ldw + kb);
    x1 = (glb_bytes)(o.x_lo + (int64_t)m0 * o.ldx + kb);
    w1 = (glb_bytes)(o.w_lo + (int64_t)n0 * o.ldw + kb);
    ox = (uint32_t)((int64_t)min(row, o.M - 1 - m0) * o.ldx + kc) * 2u;
    ow = (uint32_t)((int64_t)row * o.ldw + kc) * 2u;
    w_half = (int64_t)128 * o.ldw * 2;
  }

  // the next stage into buf
  __device__ __forceinline__ void issue(unsigned char* buf) {
    unsigned char* dx = buf + wave * 1024;
    unsigned char* dw = buf + 2 * kSubX + wave * 1024;
    to_lds(x0, ox, dx);
    to_lds(x1, ox, dx + kSubX);
    to_lds(w0, ow, dw);
    to_lds(w0 + w_half, ow, dw + 8 * 1024);
    to_lds(w1, ow, dw + kSubW);
    to_lds(w1 + w_half, ow, dw + kSubW + 8 * 1024);
    x0 += 64; x1 += 64; w0 += 64; w1 += 64;
  }
};

__device__ __forceinline__ bf16x8 frag(const unsigned char* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}

// The MFMAs of one staged step; fx / fw: this lane's offset in the X / W part of a stage.
template <int NP>
__device__ __forceinline__ void mma(const unsigned char* buf, int fx, int fw, f32x4 (&acc)[NP][4][4]) {
  if constexpr (NP == 3) {
    const unsigned char* px = buf + fx;
    const unsigned char* pw = buf + 2 * kSubX + fw;
    bf16x8 xh[4], xl[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      xh[i] = frag(px + i * 1024);
      xl[i] = frag(px + kSubX + i * 1024);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bf16x8 wh = frag(pw + j * 1024), wl = frag(pw + kSubW + j * 1024);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[0][j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wh, xh[i], acc[0][j][i], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[1][j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wl, xh[i], acc[1][j][i], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[2][j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wh, xl[i], acc[2][j][i], 0, 0, 0);
    }
  } else {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8 x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = frag(buf + ((fx ^ (s * 64)) + i * 2048));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bf16x8 w = frag(buf + 2 * kSubX + ((fw ^ (s * 64)) + j * 2048));
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[0][j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x[i], acc[0][j][i], 0, 0, 0);
      }
    }
  }
}

// Epilogue contract: store4(z, m, n0, v): columns n0 .. n0 + 3 (n0 a multiple of 4) of row m < M, slice z
// (product p's slice s at z = p * slices + s; kSum: the three products' sum, in their order, at slice z).  N is a
// multiple of kBN.
template <int NP, class EPI>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_nt(Operands o, EPI epi,
                                                                                               int k_split) {
  __shared__ __align__(16) unsigned char s0[kStageBytes];
  __shared__ __align__(16) unsigned char s1[kStageBytes];
  __shared__ __align__(16) unsigned char s2[kStageBytes];
  const gemm::TileId tile = gemm::xcd_tile();
  const int m0 = tile.tm * kBM, n0 = tile.tn * kBN;
  const int kb = tile.tz * k_split, len = min(o.K, kb + k_split) - kb;
  constexpr int kStep = NP == 3 ? 32 : 64;
  const int nst = len / kStep;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Loader<NP> ld(o, m0, n0, kb, wave);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int wm = wave >> 2, wn = wave & 3;
  // this lane's fragment offset: row lr, k chunk lg of the first 32 k (the second: chunk lg + 4, bit 6)
  const int off = NP == 3 ? lr * 64 + ((lg ^ ((lr >> 1) & 3)) << 4) : lr * 128 + ((lg ^ (lr & 7)) << 4);
  const int fx = off + wm * (NP == 3 ? 4096 : 8192), fw = off + wn * (NP == 3 ? 4096 : 8192);
  f32x4 acc[NP][4][4];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[p][j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  // Stage t has arrived when at most the six reads of stage t + 1 are outstanding; behind the barrier
  // every wave has it, and has read stage t - 1, whose place stage t + 2 takes.
  auto arrive = [&](bool newest) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (newest) __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
    else __builtin_amdgcn_s_waitcnt(0x0076);          // vmcnt(6) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  ld.issue(s0);
  if (nst > 1) ld.issue(s1);
  int t = 0;
  if constexpr (NP == 1) {   // whole rounds without tests (with three products that took too many registers)
    for (; t + 5 <= nst; t += 3) {
      arrive(false);
      ld.issue(s2);
      mma<NP>(s0, fx, fw, acc);
      arrive(false);
      ld.issue(s0);
      mma<NP>(s1, fx, fw, acc);
      arrive(false);
      ld.issue(s1);
      mma<NP>(s2, fx, fw, acc);
    }
  }
  auto step = [&](unsigned char* cur, unsigned char* next, int t) {
    arrive(t + 1 >= nst);
    if (t + 2 < nst) ld.issue(next);
    mma<NP>(cur, fx, fw, acc);
  };
  for (; t < nst; t += 3) {
    step(s0, s2, t);
    if (t + 1 < nst) step(s1, s0, t + 1);
    if (t + 2 < nst) step(s2, s1, t + 2);
  }
  const int slices = gridDim.z;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + wm * 64 + i * 16 + lr;
    if (m >= o.M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + wn * 64 + j * 16 + 4 * lg;
      if constexpr (EPI::kSum) {
        epi.store4(tile.tz, m, n, acc[0][j][i] + acc[1][j][i] + acc[2][j][i]);
      } else {
#pragma unroll
        for (int p = 0; p < NP; ++p) epi.store4(p * slices + tile.tz, m, n, acc[p][j][i]);
      }
    }
  }
}

// K in slices of k_split (a multiple of 64); N a multiple of kBN.
template <int NP, class EPI>
hipError_t run(const Operands& o, const EPI& epi, int k_split, hipStream_t st) {
  const uintptr_t at = (uintptr_t)o.x | (uintptr_t)o.w | (NP == 3 ? (uintptr_t)o.x_lo | (uintptr_t)o.w_lo : 0);
  if (o.M < 1 || o.K < 64 || o.N < kBN || o.N % kBN || ((o.K | o.ldx | o.ldw | k_split) & 63) || k_split < 64 || (at & 15))
    return hipErrorInvalidValue;
  const dim3 grid((o.M + kBM - 1) / kBM, o.N / kBN, (o.K + k_split - 1) / k_split);
  if (grid.y > 65535 || grid.z > 65535) return hipErrorInvalidValue;
  k_gemm_nt<NP, EPI><<<grid, kThreads, 0, st>>>(o, epi, k_split);
  return hipGetLastError();
}

// Split-K partial sums: slice z of a [slices][M][ld] FP32 buffer.
struct EpiPartial {
  static constexpr bool kSum = false;
  float* part; int64_t ld, slice;
  __device__ __forceinline__ void store4(int z, int m, int n0, const f32x4& v) const {
    *reinterpret_cast<f32x4*>(part + (int64_t)z * slice + (int64_t)m * ld + n0) = v;
  }
};

struct EpiSum : EpiPartial {
  static constexpr bool kSum = true;
};

// out = bf16(relu(v + bias))
struct EpiBiasRelu {
  static constexpr bool kSum = false;
  uint16_t* out; const float* bias; int64_t ld;
  __device__ __forceinline__ void store4(int, int m, int n0, const f32x4& v) const {
    uint16_t h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = gemm::f2bf(fmaxf(v[e] + bias[n0 + e], 0.0f));
    *reinterpret_cast<uint2*>(out + (int64_t)m * ld + n0) =
        make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
  }
};

// ---------------------------------------------------------------- conv-feature gradient
//
// out[m][n] = bf16(mask(m, n) ? sum_k dz[m][k] wt[n][k] : 0), k < 256, n < 8192: FC1's input gradient at the
// conv features through conv2's ReLU, the mask as one bit per feature (bit n % 8 of byte n / 8 of row m).
//
// What bounds it is memory: the output (16 KB a row), beside which the 128 x 128 tiles this takes the
// place of read the BF16 activations for the mask (16 KB more) and both operands of every tile again.
// Here a workgroup keeps the fragments of 64 WN features' weights in registers (a wave's 64 features: 128
// registers a lane) and walks over row tiles of 128 (64 KB, two in LDS, the next one's reads in flight), and
// the mask costs 1 KB a row.  Workgroups eight apart (one XCD) share their row tiles.  The weights' rows
// are dealt to the MFMA fragments so that a lane holds eight consecutive features of a row: one 16-byte
// store.  9000 rows: 120 -> 60 us, 16384 rows: 221 -> 97 us.
constexpr int kDxK = 256, kDxTile = kBM * kDxK * 2;   // bytes of a row tile

__device__ __forceinline__ uint32_t mask2(uint32_t bits, float lo, float hi) {
  return ((bits & 1u) ? (uint32_t)gemm::f2bf(lo) : 0u) | ((bits & 2u) ? (uint32_t)gemm::f2bf(hi) << 16 : 0u);
}

template <int WN>
__global__ __launch_bounds__(128 * WN) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_feature_grad(
    const uint16_t* __restrict__ dz, const uint16_t* __restrict__ wt, const uint8_t* __restrict__ mask,
    uint16_t* __restrict__ out, int M, int N, int groups) {
  __shared__ __align__(16) unsigned char s0[kDxTile];
  __shared__ __align__(16) unsigned char s1[kDxTile];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int wm = wave / WN, wn = wave % WN;
  const int group = blockIdx.x % groups, nw = (blockIdx.x / groups * WN + wn) * 64;   // the wave's first feature
  const int tiles = (M + kBM - 1) / kBM;
  // row tile t into buf: a wave's read covers two rows of 512 bytes; chunk c of row r lies at c ^ (r % 8)
  const int r0 = 2 * wave + (lane >> 5);
  const uint32_t chunk = (uint32_t)((lane & 31) ^ (r0 & 7)) * 16u;
  auto issue = [&](unsigned char* buf, int t) {
    const glb_bytes base = (glb_bytes)(dz + (int64_t)t * kBM * kDxK);
    const int last = M - 1 - t * kBM;   // rows past M read the last one
#pragma unroll
    for (int i = 0; i < 32 / WN; ++i)
      to_lds(base, (uint32_t)min(r0 + 4 * WN * i, last) * (kDxK * 2) + (chunk ^ ((4 * WN * i) & 7) * 16u),
             buf + (2 * WN * i + wave) * 1024);
  };
  bf16x8 w[4][8];
  const int wrow = (lr >> 2) * 8 + (lr & 3);   // + (j / 2) * 32 + (j % 2) * 4: the feature of fragment j's row lr
  issue(s0, group);
  if (WN <= 2) {
    // the weights' rows into s1 in the row tiles' layout, and from there to the registers
    const glb_bytes base = (glb_bytes)(wt + (int64_t)(nw - wn * 64) * kDxK);
#pragma unroll
    for (int i = 0; i < 16; ++i)
      to_lds(base, (uint32_t)(r0 + 4 * WN * i) * (kDxK * 2) + (chunk ^ ((4 * WN * i) & 7) * 16u),
             s1 + (2 * WN * i + wave) * 1024);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        const int n = wn * 64 + (j >> 1) * 32 + (j & 1) * 4 + wrow;
        w[j][ks] = frag(s1 + n * (kDxK * 2) + (((4 * ks + lg) ^ (n & 7)) << 4));
      }
    __syncthreads();
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int ks = 0; ks < 8; ++ks)
        w[j][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(
            wt + (int64_t)(nw + (j >> 1) * 32 + (j & 1) * 4 + wrow) * kDxK + 32 * ks + 8 * lg));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);   // the first tile (no stores follow it)
  }
  const int f0 = (wm * 64 + lr) * (kDxK * 2) + ((lg ^ (lr & 7)) << 4);
  auto tile = [&](unsigned char* cur, unsigned char* next, int t) {
    const int m0 = t * kBM + wm * 64 + lr;
    // the tile has arrived when at most the eight stores of the tile before are outstanding
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0078);   // vmcnt(8) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    uint2 mk[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      mk[i] = *reinterpret_cast<const uint2*>(mask + (int64_t)min(m0 + 16 * i, M - 1) * (N / 8) + nw / 8);
    if (t + groups < tiles) issue(next, t + groups);
    f32x4 acc[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      bf16x8 x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = frag(cur + ((f0 ^ ((ks & 1) * 64)) + (ks >> 1) * 128 + i * 16 * kDxK * 2));
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j][ks], x[i], acc[j][i], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + 16 * i;
      if (m >= M) continue;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint32_t b = (q ? mk[i].y : mk[i].x) >> (8 * lg);
        const f32x4 lo = acc[2 * q][i], hi = acc[2 * q + 1][i];
        *reinterpret_cast<uint4*>(out + (int64_t)m * N + nw + q * 32 + lg * 8) =
            make_uint4(mask2(b, lo[0], lo[1]), mask2(b >> 2, lo[2], lo[3]), mask2(b >> 4, hi[0], hi[1]),
                       mask2(b >> 6, hi[2], hi[3]));
      }
    }
  };
  for (int t = group; t < tiles; t += 2 * groups) {
    tile(s0, s1, t);
    if (t + groups < tiles) tile(s1, s0, t + groups);
  }
}

// N a multiple of 256; 16-byte aligned operands.
inline hipError_t feature_grad(const uint16_t* dz, const uint16_t* wt, const uint8_t* mask, uint16_t* out, int M, int N,
                               hipStream_t st) {
  if (M < 1 || N < kBN || N % kBN) return hipErrorInvalidValue;
  // Workgroups of 64, 128 or 256 features: few row tiles leave the chip idle with the wide ones, many reread
  // their rows in every slice.  64 / 128 / 256 features took 5.8 / 6.5 / 13 us at 96 rows, 7.0 / 7.6 / 14 at
  // 200, 12 / 9.1 / 15 at 400, 20 / 15.4 / 16.6 at 800, 125 / 77 / 59 at 9000; a whole minibatch 128.9 / 129.3 at 200
  // rows and 135.7 / 133.3 at 257 (64 / 128 features), 161.8 / 162.5 at 800 and 169.4 / 168.2 at 1025 (128 / 256).
  constexpr int kNarrowTiles = 2, kMidTiles = 7;
  const int tiles = (M + kBM - 1) / kBM, groups = std::min(8, tiles);
  if (tiles <= kNarrowTiles)
    k_feature_grad<1><<<(unsigned)(N / 64 * groups), 128, 0, st>>>(dz, wt, mask, out, M, N, groups);
  else if (tiles <= kMidTiles)
    k_feature_grad<2><<<(unsigned)(N / 128 * groups), 256, 0, st>>>(dz, wt, mask, out, M, N, groups);
  else
    k_feature_grad<4><<<(unsigned)(N / kBN * groups), kThreads, 0, st>>>(dz, wt, mask, out, M, N, groups);
  return hipGetLastError();
}

}  // namespace gemm_nt
}  // namespace aslam
