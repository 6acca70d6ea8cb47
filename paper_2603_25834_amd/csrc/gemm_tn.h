// gemm_tn.h -- weight gradients: BF16 GEMM contracted over the rows of both operands, for gfx950
// (library-internal).
//
// C[n][k] = sum_m D[m][n] X[m][k] (FP32 accumulation), D the output gradients [M][N], X the inputs [M][K]; the rows
// m may be split over z, slice z into part[z][N][K].  N a multiple of 256, both leading dimensions multiples
// of 8, 16-byte aligned operands.
//
// What bounds the 128 x 128 tile this takes the place of: it goes through registers and transposes there, one
// 4-byte LDS store per two values.  Here a stage is 32 rows of both operands, straight to LDS (16 bytes a lane), four
// stages in LDS, the reads three stages ahead, one barrier a stage.  T = 256: a workgroup of eight waves owns
// 256 x 256 of C (128 x 64 a wave), one per CU, so that N = 256 reads X, the large operand, once.  T = 128: four
// waves of 64 x 64, two workgroups per CU, for few rows or small matrices.  FC1's weight (N = 256, K = 8564), GEMM
// alone: 140 -> 57 us at M = 9000, 227 -> 92 at 16384 (42 % of the matrix cores' time; what bounds it is the way from
// HBM, 281 MB of X and 61 MB of partial sums), 62 -> 26 at 3000, 16 -> 10 at 96.
//
// The fragments want eight rows of one column a lane: ds_read_b64_tr_b16 gives four (of a group's 16 lanes, lane
// 4 r + c reads columns 4 c .. of row r, lane i receives column i of the four rows).  The rows of a stage are
// dealt to the MFMA's k index as 16 t + 4 g + r (lane group g, read t), the same for both operands; the 32-byte
// column blocks of row r lie permuted by r % 8, so that 32 lanes' eight rows cover all banks.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "gemm_bf16.h"
#include "gemm_nt.h"

namespace aslam {
namespace gemm_tn {

using gemm::bf16x8;
using gemm::f32x4;
using gemm_nt::glb_bytes;
using gemm_nt::to_lds;

constexpr int kRows = 32;   // of a stage

struct Operands {
  const uint16_t* d; int64_t ldd; int N;   // [M][N]
  const uint16_t* x; int64_t ldx; int K;   // [M][K]
  int M;
};

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4_t lds_short4;

template <int kRowBytes>
__device__ __forceinline__ bf16x8 frag_tr(const unsigned char* p) {
  struct Pair { short4_t lo, hi; } v;
  v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)p);
  v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(p + 16 * kRowBytes));
  return __builtin_bit_cast(bf16x8, v);
}

// T x T tiles, T / 32 waves
template <int T>
__global__ __launch_bounds__(2 * T) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_tn(
    Operands o, float* __restrict__ part, int m_split) {
  constexpr int kRowBytes = 2 * T, kOpBytes = kRows * kRowBytes, kStage = 2 * kOpBytes;   // D's rows, then X's
  constexpr int kLaneRow = kRowBytes / 16;   // lanes that read a row
  constexpr int FN = T / 32, WK = T / 64;    // a wave's 16-row fragments of n (and four of k); waves along k
  __shared__ __align__(16) unsigned char s0[kStage];
  __shared__ __align__(16) unsigned char s1[kStage];
  __shared__ __align__(16) unsigned char s2[kStage];
  __shared__ __align__(16) unsigned char s3[kStage];
  const gemm::TileId tile = gemm::xcd_tile();
  const int n0 = tile.tm * T, k0 = tile.tn * T;
  const int mb = tile.tz * m_split, rows = min(o.M, mb + m_split) - mb;
  const int nst = (rows + kRows - 1) / kRows;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  // this lane's part of a stage: 16 bytes of rows row and row + 16 (a wave's read covers 1 KB of rows); the
  // 16-byte chunk c of row r lies at c ^ 2 (r % 8).  Columns past X's pitch read its last ones.
  const int row = 64 / kLaneRow * wave + lane / kLaneRow, chunk = (lane % kLaneRow) ^ (2 * (row & 7));
  const uint32_t cd = (uint32_t)chunk * 16u, cx = (uint32_t)min(8 * chunk, (int)o.ldx - 8 - k0) * 2u;
  const uint32_t pd = (uint32_t)o.ldd * 2u, px = (uint32_t)o.ldx * 2u;
  glb_bytes gd = (glb_bytes)(o.d + (int64_t)mb * o.ldd + n0), gx = (glb_bytes)(o.x + (int64_t)mb * o.ldx + k0);
  int left = rows;   // rows from the next stage on; rows past the last read it
  auto issue = [&](unsigned char* buf) {
    const uint32_t r0 = (uint32_t)min(row, left - 1), r1 = (uint32_t)min(row + 16, left - 1);
    unsigned char* dst = buf + wave * 1024;
    to_lds(gd, r0 * pd + cd, dst);
    to_lds(gd, r1 * pd + cd, dst + 16 * kRowBytes);
    to_lds(gx, r0 * px + cx, dst + kOpBytes);
    to_lds(gx, r1 * px + cx, dst + kOpBytes + 16 * kRowBytes);
    gd += (int64_t)kRows * pd; gx += (int64_t)kRows * px;
    left -= kRows;
  };
  f32x4 acc[FN][4];   // [16 n][16 k]
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // this lane's 8 bytes of a fragment: row 4 lg + lr / 4, columns 4 (lr % 4) of 16; the column block b of 32 bytes
  // at b ^ (row % 8)
  const int fr = 4 * lg + (lr >> 2);
  const int f0 = fr * kRowBytes + 8 * (lr & 3), fs = (fr & 7) * 32;
  const int wn = wave / WK, wk = wave % WK;
  auto mma = [&](const unsigned char* buf) {
    bf16x8 x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = frag_tr<kRowBytes>(buf + kOpBytes + f0 + ((wk * 128 + j * 32) ^ fs));
#pragma unroll
    for (int i = 0; i < FN; ++i) {
      const bf16x8 d = frag_tr<kRowBytes>(buf + f0 + ((wn * FN * 32 + i * 32) ^ fs));
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[j], d, acc[i][j], 0, 0, 0);
    }
  };
  // Stage t has arrived when at most the four reads of each of the next two stages are outstanding; behind the
  // barrier every wave has it, and has read stage t - 1, whose place stage t + 3 takes.
  auto step = [&](unsigned char* cur, unsigned char* free_buf, int t) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (t + 2 < nst) __builtin_amdgcn_s_waitcnt(0x0078);        // vmcnt(8) lgkmcnt(0)
    else if (t + 1 < nst) __builtin_amdgcn_s_waitcnt(0x0074);   // vmcnt(4)
    else __builtin_amdgcn_s_waitcnt(0x0070);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (t + 3 < nst) issue(free_buf);
    const int valid = rows - t * kRows;
    if (valid < kRows) {   // the last stage's missing rows are zeros in both operands
      for (int v = valid * (kRowBytes / 16) + threadIdx.x; v < kOpBytes / 16; v += 2 * T) {
        reinterpret_cast<uint4*>(cur)[v] = make_uint4(0u, 0u, 0u, 0u);
        reinterpret_cast<uint4*>(cur + kOpBytes)[v] = make_uint4(0u, 0u, 0u, 0u);
      }
      __syncthreads();
    }
    mma(cur);
  };
  issue(s0);
  if (nst > 1) issue(s1);
  if (nst > 2) issue(s2);
  for (int t = 0; t < nst; t += 4) {
    step(s0, s3, t);
    if (t + 1 < nst) step(s1, s0, t + 1);
    if (t + 2 < nst) step(s2, s1, t + 2);
    if (t + 3 < nst) step(s3, s2, t + 3);
  }
  // a lane holds columns 4 lg .. 4 lg + 3 of 16 for row lr of 16
  float* const out = part + (int64_t)tile.tz * o.N * o.K;
  const bool vec = (o.K & 3) == 0 && (reinterpret_cast<uintptr_t>(part) & 15) == 0;
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + (wn * FN + i) * 16 + lr, k = k0 + wk * 64 + j * 16 + 4 * lg;
      float* q = out + (int64_t)n * o.K + k;
      if (vec) {
        if (k < o.K) *reinterpret_cast<f32x4*>(q) = acc[i][j];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (k + e < o.K) q[e] = acc[i][j][e];
      }
    }
}

inline int tiles(int N, int K, int T) { return N / T * ((K + T - 1) / T); }

// Rows of a slice: S slices of whole stages.
inline int slice_rows(int M, int S) { return ((M + S - 1) / S + kRows - 1) / kRows * kRows; }

// S slices or fewer; slices() of them are written.
inline int slices(int M, int S) { return (M + slice_rows(M, S) - 1) / slice_rows(M, S); }

inline hipError_t run(const Operands& o, float* part, int T, int S, hipStream_t st) {
  if (o.M < 1 || o.K < 1 || o.N < 256 || o.N % 256 || o.ldd % 8 || o.ldx % 8 || o.ldx < o.K || S < 1)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)(o.N / T), (unsigned)((o.K + T - 1) / T), (unsigned)slices(o.M, S));
  if (T == 256) k_gemm_tn<256><<<grid, 512, 0, st>>>(o, part, slice_rows(o.M, S));
  else k_gemm_tn<128><<<grid, 256, 0, st>>>(o, part, slice_rows(o.M, S));
  return hipGetLastError();
}

}  // namespace gemm_tn
}  // namespace aslam
