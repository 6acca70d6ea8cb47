// gru_kernels.h -- the recurrent actor-critic's GRU layer on gfx950 (library-internal).
//
// A single-layer GRU of 256 units (arXiv 2603.25834, Sec. III-F, "Recurrent Layer") sits between
// FC1 and the heads.  Gate rows of the weights are ordered reset / update / new:
//   r = sigmoid(W_ir x + b_ir + W_hr h + b_hr),  z = sigmoid(W_iz x + b_iz + W_hz h + b_hz),
//   n = tanh(W_in x + b_in + r (W_hn h + b_hn)),  h' = (1 - z) n + z h,
// with the state zeroed before a step that starts an episode.  The products run on MFMA with BF16
// operands (FC1 output, weights, the state fed to W_hh) and FP32 accumulation; the gate math and
// the state itself are FP32.
//
// A rollout step (k_gru_fwd) runs as a grid of 16-row tiles x kGruSlices workgroups: each workgroup
// (4 waves) stages its rows' FC1 output and entering state, and owns 64 of the 256 units (16 per wave)
// of every gate, so each lane ends up holding r, z and both halves of n's pre-activation for the same
// (row, unit) pairs and forms h' in registers; a workgroup reads a quarter of the weights, and a step
// of a few hundred rows spreads over many CUs.
//
// A sequence minibatch (k_gru_seq_fwd, k_gru_seq_bwd) runs all its steps in one launch per direction:
// rows (robots) are independent, so a workgroup owns 16 of them for the whole sequence and keeps W_hh
// on its CU (registers and LDS hold its 384 KB together), instead of one launch per step that reads the
// weights again.
#pragma once

#include "policy_kernels.h"

namespace aslam {
namespace pol {

constexpr int kGruRows = 16;
constexpr int kGruLdX = kHid + 8;    // BF16 rows in LDS, padded
constexpr int kGruLdF = kHid + 4;    // FP32 rows in LDS, padded
constexpr int kGruLdG = kGates + 8;  // BF16 gate-gradient rows in LDS, padded

constexpr int kGruSlices = 4;

struct GruFwdArgs {
  const float* prm;
  Offsets o;
  int rows;              // rows of this step
  const uint16_t* h1;    // the BF16 FC1 output
  const uint16_t* wih;   // BF16 [768][256]
  const uint16_t* whh;   // BF16 [768][256]
  const float* hp;       // entering state
  const uint8_t* first;  // episode start flags; NULL = none
  float* h_out;          // new state
};

__device__ __forceinline__ float sigmoidf_(float x) { return 1.0f / (1.0f + expf(-x)); }

// One GRU step over the rows of a rollout.
// h_out must not alias hp (other workgroups of the tile still read the entering state).
// The lane's weight fragments (unit u, gate g, k-step s) of a [768][256] BF16 matrix, all loads
// issued together: the step is latency-bound, so its 24 fragments cost one memory round trip.
__device__ __forceinline__ void gru_weight_frags(const uint16_t* w, int64_t u, int lg, gemm::bf16x8 (&f)[3][8]) {
#pragma unroll
  for (int g = 0; g < 3; ++g)
#pragma unroll
    for (int s = 0; s < 8; ++s)
      f[g][s] = __builtin_bit_cast(gemm::bf16x8,
                                   *reinterpret_cast<const uint4*>(w + (u + g * kHid) * kHid + 32 * s + 8 * lg));
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_gru_fwd(GruFwdArgs a) {
  __shared__ __align__(16) uint16_t s_x[kGruRows * kGruLdX];
  __shared__ __align__(16) uint16_t s_hb[kGruRows * kGruLdX];
  __shared__ __align__(16) float s_hp[kGruRows * kGruLdF];
  const int row0 = blockIdx.x * kGruRows;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const Offsets& o = a.o;
  const int64_t u = 64 * blockIdx.y + 16 * wave + lr;
  gemm::bf16x8 wi[3][8], wh[3][8];
  gru_weight_frags(a.wih, u, lg, wi);
  gru_weight_frags(a.whh, u, lg, wh);
#pragma unroll
  for (int g = threadIdx.x; g < kGruRows * (kHid / 8); g += 256) {
    const int r = g / (kHid / 8), n0 = (g % (kHid / 8)) * 8;
    const int i = row0 + r;
    uint4 vx = make_uint4(0u, 0u, 0u, 0u);
    float hv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (i < a.rows) {
      vx = *reinterpret_cast<const uint4*>(a.h1 + (int64_t)i * kHid + n0);
      const bool reset = a.first && a.first[i];
      if (!reset) {
        const float* q = a.hp + (int64_t)i * kHid + n0;
        const float4 lo = *reinterpret_cast<const float4*>(q), hi = *reinterpret_cast<const float4*>(q + 4);
        hv[0] = lo.x; hv[1] = lo.y; hv[2] = lo.z; hv[3] = lo.w;
        hv[4] = hi.x; hv[5] = hi.y; hv[6] = hi.z; hv[7] = hi.w;
      }
    }
    *reinterpret_cast<uint4*>(s_x + r * kGruLdX + n0) = vx;
    uint16_t hb[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      s_hp[r * kGruLdF + n0 + j] = hv[j];
      hb[j] = f2bf(hv[j]);
    }
    *reinterpret_cast<uint4*>(s_hb + r * kGruLdX + n0) = pack8(hb);
  }
  __syncthreads();
  // r and z accumulate the input and the state part in one accumulator (input first); n keeps them apart
  gemm::f32x4 ar = {0.f, 0.f, 0.f, 0.f}, az = ar, an = ar, ahn = ar;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const auto ax =
        __builtin_bit_cast(gemm::bf16x8, *reinterpret_cast<const uint4*>(s_x + lr * kGruLdX + 32 * s + 8 * lg));
    ar = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ax, wi[0][s], ar, 0, 0, 0);
    az = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ax, wi[1][s], az, 0, 0, 0);
    an = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ax, wi[2][s], an, 0, 0, 0);
  }
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const auto ah =
        __builtin_bit_cast(gemm::bf16x8, *reinterpret_cast<const uint4*>(s_hb + lr * kGruLdX + 32 * s + 8 * lg));
    ar = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, wh[0][s], ar, 0, 0, 0);
    az = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, wh[1][s], az, 0, 0, 0);
    ahn = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, wh[2][s], ahn, 0, 0, 0);
  }
  // gates and the new state: lane holds unit u of rows 4 lg + e
  const float* bi = a.prm + o.gbi;
  const float* bh = a.prm + o.gbh;
  const float bir = bi[u], biz = bi[u + kHid], bin = bi[u + 2 * kHid];
  const float bhr = bh[u], bhz = bh[u + kHid], bhn = bh[u + 2 * kHid];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = 4 * lg + e, i = row0 + r;
    if (i >= a.rows) continue;
    const float rg = sigmoidf_((ar[e] + bir) + bhr);
    const float zg = sigmoidf_((az[e] + biz) + bhz);
    const float ghn = ahn[e] + bhn;
    const float ng = tanhf((an[e] + bin) + rg * ghn);
    const float hpv = s_hp[r * kGruLdF + u];
    a.h_out[(int64_t)i * kHid + u] = (1.0f - zg) * ng + zg * hpv;
  }
}

// Rollout heads on the new state (no ReLU) and the Gaussian sample, one wave per row (lane l holds
// units 4 l .. 4 l + 3); also copies the state to h_out (which may alias the step's entering state,
// read completely by the step kernel before this one runs).
__global__ __launch_bounds__(256) void k_gru_heads(const float* prm, Offsets o, const float* h, int rows,
                                                   float* h_out, float* mu, float* value, ActDraws eps,
                                                   float* act, float* logp) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + wave;
  if (row >= rows) return;
  const float4 hh = *reinterpret_cast<const float4*>(h + row * kHid + lane * 4);
  if (h_out != h) *reinterpret_cast<float4*>(h_out + row * kHid + lane * 4) = hh;
  const float hv[4] = {hh.x, hh.y, hh.z, hh.w};
  float s0 = 0, s1 = 0, sv = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    s0 += prm[o.muw + lane * 4 + e] * hv[e];
    s1 += prm[o.muw + kHid + lane * 4 + e] * hv[e];
    sv += prm[o.vw + lane * 4 + e] * hv[e];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_xor(s0, off, 64);
    s1 += __shfl_xor(s1, off, 64);
    sv += __shfl_xor(sv, off, 64);
  }
  // the row's two normals on lanes 0 and 1 at once (a library draw is a long dependent chain)
  const float ed = lane < 2 ? eps(row, lane) : 0.0f;
  const float e1 = __shfl(ed, 1, 64);
  if (lane == 0) {
    const float m0 = s0 + prm[o.mub], m1 = s1 + prm[o.mub + 1];
    if (mu) {
      mu[2 * row] = m0;
      mu[2 * row + 1] = m1;
    }
    value[row] = sv + prm[o.vb];
    const float ls0 = prm[o.lstd], ls1 = prm[o.lstd + 1];
    const float e0 = ed;
    act[2 * row] = m0 + expf(ls0) * e0;
    act[2 * row + 1] = m1 + expf(ls1) * e1;
    logp[row] = -0.5f * (e0 * e0 + e1 * e1) - (ls0 + ls1) - 1.8378770664093453f;
  }
}

// ---------------------------------------------------------------- sequence minibatches
//
// One workgroup of eight waves runs 4 E robots through all T steps; wave w owns units 32 w .. 32 w + 31
// (two 16-column tiles), so a lane keeps the (robot, unit) pairs (E lg + e, 32 w + 16 j + lr), e < E,
// for the whole sequence (row 4 lg + e of the 16-row MFMA tile; the rows e >= E stay empty) and the state
// (or its gradient) never leaves its registers except as the BF16 rows that the next step's product
// reads from LDS.  E is 4, 2 or 1 (gru_seq_rows): a step's length is mostly the gate math of its rows, so while there
// are CUs left a tile is filled with fewer robots rather than with empty CUs.  W_hh stays on the CU: most fragments in
// registers, the rest in LDS in fragment order (16 bytes per lane, conflict-free).  What bounds it: a step is a serial
// chain (product, gate math, exchange) whose launch per step, which this replaces, read the 384 KB of weights and the
// rows back from L2 every time.
// T = 24, 375 robots: forward 256 us in 24 launches -> 58 us (+ 15 us for the input products as one
// GEMM), backward 304 -> 71 us; with 16 robots a workgroup (E = 4) they took 156 and 170 us.
struct GruSeqArgs {
  const float* prm;
  Offsets o;
  int nb, T, N;            // robots of the minibatch, steps, robots of the rollout
  const int32_t* robots;   // [nb] rollout robot of each row
  const float* h0;         // [N][256] state entering step 0
  const uint8_t* first;    // [T][N] episode starts
  const float* gi;         // [T nb][768] FP32 input products W_ih x, no bias (forward)
  const uint16_t* whh;     // BF16 W_hh [768][256] (forward), its transpose [256][768] (backward)
  float* hst;              // [T nb][256] new state of each step
  float *g_r, *g_z, *g_n, *g_ghn;   // [T nb][256] gate values
  uint16_t* hp_bf;         // [T nb][256] BF16 state entering each step
  const float* dh_head;    // [T nb][256] the heads' state gradient (backward)
  uint16_t *dgi, *dgh;     // [T nb][768] gate pre-activation gradients, input and state side
  float* part;             // [gridDim.x][1536] their column sums: dgi's, then dgh's
};

constexpr int kGruSeqThreads = 512;

// Robots per lane group (E above) for nb robots: the least that still gives each CU one workgroup.
inline int gru_seq_rows(int nb) { return nb <= 4 * 256 ? 1 : nb <= 8 * 256 ? 2 : 4; }

constexpr int kGruBwdRegSteps = 17;   // k-steps of W_hh^T (of 24) held in registers by the backward
constexpr int kGruSeqFwdLds = 8 * 2 * 8 * 64 * 16 + 2 * kGruRows * kGruLdX * 2;
constexpr int kGruSeqBwdLds = 8 * 2 * (kGates / 32 - kGruBwdRegSteps) * 64 * 16 + kGruRows * kGruLdG * 2 +
                              kGruRows * kGruLdX * 2;

__device__ __forceinline__ gemm::bf16x8 lds_frag(const uint16_t* p) {
  return __builtin_bit_cast(gemm::bf16x8, *reinterpret_cast<const uint4*>(p));
}

// Forward of the whole sequence.  The accumulators of r and z start from the input products and go on
// over the state's k-steps in order, as one chain over both operands; n keeps its halves apart.
template <int E>
__global__ __launch_bounds__(kGruSeqThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gru_seq_fwd(
    GruSeqArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint4* const s_w = reinterpret_cast<uint4*>(smem);                                 // n-gate fragments
  uint16_t* const s_h = reinterpret_cast<uint16_t*>(smem + 8 * 2 * 8 * 64 * 16);     // [2][16][264]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int row0 = blockIdx.x * 4 * E;
  const int u0 = 32 * wave + lr;
  gemm::bf16x8 wr[2][8], wz[2][8];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const uint16_t* w = a.whh + (int64_t)(u0 + 16 * j) * kHid + 32 * s + 8 * lg;
      wr[j][s] = lds_frag(w);
      wz[j][s] = lds_frag(w + (int64_t)kHid * kHid);
      s_w[((wave * 2 + j) * 8 + s) * 64 + lane] = *reinterpret_cast<const uint4*>(w + (int64_t)2 * kHid * kHid);
    }
  const float* bi = a.prm + a.o.gbi;
  const float* bh = a.prm + a.o.gbh;
  float bir[2], biz[2], bin[2], bhr[2], bhz[2], bhn[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int u = u0 + 16 * j;
    bir[j] = bi[u]; biz[j] = bi[u + kHid]; bin[j] = bi[u + 2 * kHid];
    bhr[j] = bh[u]; bhz[j] = bh[u + kHid]; bhn[j] = bh[u + 2 * kHid];
  }
  // rows past the minibatch read its last row and write nothing
  int row[E], rob[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    row[e] = min(row0 + E * lg + e, a.nb - 1);
    rob[e] = a.robots[row[e]];
  }
  float hp[2][E];
  gemm::f32x4 gr[2], gz[2], gn[2];   // the input products of the next step
#pragma unroll
  for (int j = 0; j < 2; ++j) gr[j] = gz[j] = gn[j] = gemm::f32x4{0.f, 0.f, 0.f, 0.f};
  if (E < 4) {   // the tile's empty rows
    uint4* z = reinterpret_cast<uint4*>(s_h);
    for (int i = threadIdx.x; i < 2 * kGruRows * kGruLdX / 8; i += kGruSeqThreads) z[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
  }
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const bool reset = a.first[rob[e]];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int u = u0 + 16 * j;
      const float h = a.h0[(int64_t)rob[e] * kHid + u];
      hp[j][e] = reset ? 0.0f : h;
      s_h[(4 * lg + e) * kGruLdX + u] = f2bf(hp[j][e]);
      const float* g = a.gi + (int64_t)row[e] * kGates + u;
      gr[j][e] = g[0];
      gz[j][e] = g[kHid];
      gn[j][e] = g[2 * kHid];
    }
  }
  for (int t = 0; t < a.T; ++t) {
    __syncthreads();
    const uint16_t* sh = s_h + (t & 1) * kGruRows * kGruLdX;
    uint16_t* sn = s_h + ((t + 1) & 1) * kGruRows * kGruLdX;
    gemm::f32x4 ar[2], az[2], an[2], ahn[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      ar[j] = gr[j];
      az[j] = gz[j];
      an[j] = gn[j];
      ahn[j] = gemm::f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int tn = min(t + 1, a.T - 1);   // the next step's inputs (the last step's again at the end)
    bool reset[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      reset[e] = a.first[(int64_t)tn * a.N + rob[e]];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float* g = a.gi + ((int64_t)tn * a.nb + row[e]) * kGates + u0 + 16 * j;
        gr[j][e] = g[0];
        gz[j][e] = g[kHid];
        gn[j][e] = g[2 * kHid];
      }
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const gemm::bf16x8 ah = lds_frag(sh + lr * kGruLdX + 32 * s + 8 * lg);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const gemm::bf16x8 wn = __builtin_bit_cast(gemm::bf16x8, s_w[((wave * 2 + j) * 8 + s) * 64 + lane]);
        ar[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, wr[j][s], ar[j], 0, 0, 0);
        az[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, wz[j][s], az[j], 0, 0, 0);
        ahn[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, wn, ahn[j], 0, 0, 0);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int u = u0 + 16 * j;
        const float rg = sigmoidf_((ar[j][e] + bir[j]) + bhr[j]);
        const float zg = sigmoidf_((az[j][e] + biz[j]) + bhz[j]);
        const float ghn = ahn[j][e] + bhn[j];
        const float ng = tanhf((an[j][e] + bin[j]) + rg * ghn);
        const float h = (1.0f - zg) * ng + zg * hp[j][e];
        if (row0 + E * lg + e < a.nb) {
          const int64_t q = ((int64_t)t * a.nb + row[e]) * kHid + u;
          a.hst[q] = h;
          a.g_r[q] = rg;
          a.g_z[q] = zg;
          a.g_n[q] = ng;
          a.g_ghn[q] = ghn;
          a.hp_bf[q] = f2bf(hp[j][e]);
        }
        hp[j][e] = reset[e] ? 0.0f : h;
        sn[(4 * lg + e) * kGruLdX + u] = f2bf(hp[j][e]);
      }
  }
}

// Backpropagation through time of the whole sequence, step T - 1 first:
//   dh = dh_head + dh_next (the gradient reaching h_t from the heads and from step t + 1),
//   gate pre-activation gradients dgi = [dr', dz', dn'], dgh = [dr', dz', dn' r] (BF16, the operands
//   of the weight-gradient and input-gradient GEMMs), and the gradient reaching h_{t-1}:
//   dh_next = z dh + dgh W_hh, zero where step t starts an episode.
// The BF16 rows go through LDS (the product's operand, and 16-byte stores to memory); each lane sums
// its gradients' columns over the steps for the bias gradients.
template <int E>
__global__ __launch_bounds__(kGruSeqThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gru_seq_bwd(
    GruSeqArgs a) {
  constexpr int KS = kGates / 32, KR = kGruBwdRegSteps, KL = KS - KR;
  extern __shared__ __align__(16) unsigned char smem[];
  uint4* const s_w = reinterpret_cast<uint4*>(smem);                                   // the last KL k-steps
  uint16_t* const s_g = reinterpret_cast<uint16_t*>(smem + 8 * 2 * KL * 64 * 16);      // [16][776]: dgh
  uint16_t* const s_n = s_g + kGruRows * kGruLdG;                                      // [16][264]: dn'
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
  const int row0 = blockIdx.x * 4 * E;
  const int u0 = 32 * wave + lr;
  gemm::bf16x8 wf[2][KR];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint16_t* w = a.whh + (int64_t)(u0 + 16 * j) * kGates + 8 * lg;
#pragma unroll
    for (int s = 0; s < KR; ++s) wf[j][s] = lds_frag(w + 32 * s);
#pragma unroll
    for (int s = 0; s < KL; ++s)
      s_w[((wave * 2 + j) * KL + s) * 64 + lane] = *reinterpret_cast<const uint4*>(w + 32 * (KR + s));
  }
  int row[E], rob[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    row[e] = min(row0 + E * lg + e, a.nb - 1);
    rob[e] = a.robots[row[e]];
  }
  float dhn[2][E], cs[2][4];   // dh_next; column sums of dr', dz', dn', dn' r over the lane's rows
#pragma unroll
  for (int j = 0; j < 2; ++j) {
#pragma unroll
    for (int e = 0; e < E; ++e) dhn[j][e] = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) cs[j][k] = 0.0f;
  }
  // a step's inputs, loaded one step ahead
  float x_dh[2][E], x_r[2][E], x_z[2][E], x_n[2][E], x_g[2][E], x_h[2][E];
  bool x_first[E];
  auto load = [&](int t) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      x_first[e] = a.first[(int64_t)t * a.N + rob[e]];
      const int64_t q = ((int64_t)t * a.nb + row[e]) * kHid + u0;
      const float* hp = t > 0 ? a.hst + q - (int64_t)a.nb * kHid : a.h0 + (int64_t)rob[e] * kHid + u0;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        x_dh[j][e] = a.dh_head[q + 16 * j];
        x_r[j][e] = a.g_r[q + 16 * j];
        x_z[j][e] = a.g_z[q + 16 * j];
        x_n[j][e] = a.g_n[q + 16 * j];
        x_g[j][e] = a.g_ghn[q + 16 * j];
        x_h[j][e] = hp[16 * j];
      }
    }
  };
  load(a.T - 1);
  if (E < 4) {   // the tile's empty rows
    uint4* z = reinterpret_cast<uint4*>(s_g);
    for (int i = threadIdx.x; i < kGruRows * kGruLdG / 8; i += kGruSeqThreads) z[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
  }
  for (int t = a.T - 1; t >= 0; --t) {
    float dd[2][E];
    bool reset[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      reset[e] = x_first[e];
      const bool valid = row0 + E * lg + e < a.nb;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int u = u0 + 16 * j;
        const float rg = x_r[j][e], zg = x_z[j][e], ng = x_n[j][e];
        const float hp = reset[e] ? 0.0f : x_h[j][e];
        const float dh = x_dh[j][e] + dhn[j][e];
        dd[j][e] = dh * zg;
        const float dn_pre = (dh * (1.0f - zg)) * (1.0f - ng * ng);
        const uint16_t dz = f2bf((dh * (hp - ng)) * (zg * (1.0f - zg)));
        const uint16_t dr = f2bf((dn_pre * x_g[j][e]) * (rg * (1.0f - rg)));
        const uint16_t dn = f2bf(dn_pre), dnr = f2bf(dn_pre * rg);
        uint16_t* g = s_g + (4 * lg + e) * kGruLdG + u;
        g[0] = dr;
        g[kHid] = dz;
        g[2 * kHid] = dnr;
        s_n[(4 * lg + e) * kGruLdX + u] = dn;
        if (valid) {
          cs[j][0] += bf2f(dr);
          cs[j][1] += bf2f(dz);
          cs[j][2] += bf2f(dn);
          cs[j][3] += bf2f(dnr);
        }
      }
    }
    __syncthreads();
    load(max(t - 1, 0));
    // the rows to memory: 96 vectors of dgh and 96 of dgi (its n part from s_n) per row
#pragma unroll
    for (int k = 0; k < (4 * E * (kGates / 8) + kGruSeqThreads - 1) / kGruSeqThreads; ++k) {
      const int v = threadIdx.x + k * kGruSeqThreads;
      const int r = v / (kGates / 8), c = (v - r * (kGates / 8)) * 8;
      if (r < 4 * E && row0 + r < a.nb) {
        const int m = 4 * (r / E) + r % E;   // the robot's row of the tile
        const int64_t q = ((int64_t)t * a.nb + row0 + r) * kGates + c;
        const uint4 h = *reinterpret_cast<const uint4*>(s_g + m * kGruLdG + c);
        *reinterpret_cast<uint4*>(a.dgh + q) = h;
        *reinterpret_cast<uint4*>(a.dgi + q) =
            c < 2 * kHid ? h : *reinterpret_cast<const uint4*>(s_n + m * kGruLdX + c - 2 * kHid);
      }
    }
    gemm::f32x4 acc[2] = {gemm::f32x4{0.f, 0.f, 0.f, 0.f}, gemm::f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const gemm::bf16x8 ag = lds_frag(s_g + lr * kGruLdG + 32 * s + 8 * lg);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const gemm::bf16x8 w = s < KR ? wf[j][s < KR ? s : 0]
                                      : __builtin_bit_cast(gemm::bf16x8, s_w[((wave * 2 + j) * KL + s - KR) * 64 + lane]);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ag, w, acc[j], 0, 0, 0);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < E; ++e) dhn[j][e] = reset[e] ? 0.0f : dd[j][e] + acc[j][e];
    __syncthreads();
  }
  // column sums over the tile's rows (lanes lr of the four row groups), one partial per workgroup
  float* part = a.part + (int64_t)blockIdx.x * 2 * kGates;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float v = cs[j][k];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (lg == 0) {
        const int u = u0 + 16 * j;
        if (k < 2) part[k * kHid + u] = part[kGates + k * kHid + u] = v;
        else if (k == 2) part[2 * kHid + u] = v;
        else part[kGates + 2 * kHid + u] = v;
      }
    }
}

// Minibatch rows of a sequence minibatch: sample s = t * nb + i is rollout row t * N + robots[i].
__global__ void k_seq_rows(const int32_t* robots, int nb, int T, int N, int32_t* rows) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= T * nb) return;
  const int t = s / nb, i = s - t * nb;
  rows[s] = t * N + robots[i];
}

}  // namespace pol
}  // namespace aslam
