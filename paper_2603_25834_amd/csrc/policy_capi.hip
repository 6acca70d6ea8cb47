// policy_capi.hip -- C-ABI of the PPO actor-critic (declared in include/aslam.h).
//
// The handle owns the minibatch workspaces (activations recomputed per
// minibatch, gradient partial sums), allocated once at create time for
// `max_batch` samples; forward and backward allocate nothing.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <mutex>
#include <string>
#include <vector>

#include "aslam.h"
#include "policy_kernels.h"
#include "conv_fused.h"
#include "gemm_nt.h"
#include "gemm_tn.h"
#include "gru_kernels.h"

using namespace aslam;
using namespace aslam::pol;

// Error messages of the policy calls are reported through aslam_last_error.
namespace aslam {
void set_last_error(const std::string& msg);
}  // namespace aslam

namespace {
int pfail(int code, const std::string& m) {
  aslam::set_last_error(m);
  return code;
}
}  // namespace

// Row length of FC1's operands: whole cache lines of BF16.
constexpr int32_t fc1_pitch(int32_t k1) { return (k1 + 63) / 64 * 64; }

struct aslam_policy {
  aslam_policy_config cfg{};
  Offsets off{};
  int64_t max_b = 0;
  uint16_t *x = nullptr;   // FC1 input [B][k1p]: conv features (8192) | scan | state | zero pad, BF16
  uint16_t *h1 = nullptr, *dz2 = nullptr, *dz1 = nullptr, *dz2c = nullptr;
  uint16_t* amask = nullptr;   // conv2's ReLU mask, one bit per feature: [B][32][16] words
  float *z2 = nullptr, *part = nullptr, *hpart = nullptr;
  uint16_t *w1b = nullptr, *w1t = nullptr, *w2b = nullptr, *w2t = nullptr;   // BF16 weight copies
  uint4* cfrag = nullptr;   // the encoder's weight fragments (k_conv_frags, k_conv_bwd_frags)
  int32_t k1p = 0;   // FC1 input width padded with zeros (fc1_pitch)
  // split-precision forward (config precision 1): the lo parts of the FC1 input rows, of h1 and of the
  // FC weights (the encoder's lo fragments sit in cfrag from kConvLoFrag on)
  bool prec = false;
  uint16_t *x_lo = nullptr, *h1_lo = nullptr, *w1b_lo = nullptr, *w2b_lo = nullptr;
  int64_t part_floats = 0;
  bool prepared = false;   // w1b / w2b hold the weights of some params (the caller tracks which)
  // recurrent handle: the GRU's weight copies and the sequence minibatch's buffers
  bool rec = false;
  uint16_t *wihb = nullptr, *whhb = nullptr, *wiht = nullptr, *whht = nullptr;
  float *hst = nullptr, *g_r = nullptr, *g_z = nullptr, *g_n = nullptr, *g_ghn = nullptr;
  float* dh_head = nullptr;
  uint16_t *hp_bf = nullptr, *dg = nullptr;   // dg: the gate gradients dgi and dgh; before them, the FP32 input products
  int32_t* rows = nullptr;
};

namespace {

constexpr int kConvGrid = 1024;    // encoder forward: the resident workgroups (four per CU), each looping over samples
constexpr int kConvGridPrec = 512; // the split-precision encoder forward holds twice the LDS: two per CU
constexpr int kConvFragsAll = kConvLoFrag + kConvFrags;   // forward, backward phase and lo fragments
constexpr int kConvBwdGrid = 512;  // encoder backward: two workgroups per CU (LDS)
constexpr int64_t kFc1Splits = 12, kFc2Splits = 64;
constexpr int kFc1MinBlocks = 512;   // FC1: resident 128 x 128 workgroups (two per CU) that its K splits fill
constexpr int kFc1WideBlocks = 160;  // workgroups from which FC1 takes the 128 x 256 tiles

// Number of K slices gemm::run launches for `splits` requested splits (chunks rounded up to BK).
int slices_used(int64_t K, int64_t splits, int BK) {
  int64_t chunk = (K + splits - 1) / splits;
  chunk = (chunk + BK - 1) / BK * BK;
  return (int)((K + chunk - 1) / chunk);
}

// Slices of the rows for a weight gradient in tiles of T x T: the workgroups that are resident (two per CU of
// the small tile, one of the large) take their stages' time, and the slices' partial sums cost as much as a stage
// per 30 small tiles or 17 large ones (FC1's weight, GEMM and reduction, us: 9000 rows 74 (7 large slices) / 76 (6) /
// 92 (4); 3000 rows 45 (1 small slice + 10) / 42 (2) / 37 (3) / 45 (4); 96 rows 19 (1) / 23 (3)).
int weight_slices(int64_t rows, int T, int tiles, int64_t max_slices) {
  const int slots = T == 256 ? 256 : 512, tiles_per_stage = T == 256 ? 17 : 30;
  int best = 1;
  int64_t best_cost = -1;
  for (int s = 1; s <= max_slices; ++s) {
    const int64_t rounds = ((int64_t)tiles * s + slots - 1) / slots;
    const int64_t cost = tiles_per_stage * rounds * (gemm_tn::slice_rows(rows, s) / gemm_tn::kRows) + (int64_t)tiles * s;
    if (best_cost < 0 || cost < best_cost) { best = s; best_cost = cost; }
  }
  return best;
}

// k of an FC1 slice for the split forward with rt tiles of 128 rows: the workgroups (one per CU) take their rounds'
// time, 64 k by 64 k, and 80 tiles of partial sums cost as much as such a step.  A length that only fills the CUs on
// average leaves a few workgroups for a round of their own: the actor's call took 95 us with 448 k (260 workgroups)
// at 1664 rows and 76 with 512 (221), 382 and 306 with 2176 and 2880 at 8320, 541 and 410 with 3264 and 1728 (two full
// rounds) at 12288.  The partial sums stay within part_need's 3 x 32768 rows, or are one slice.
int split_fc1_chunk(int k1p, int rt) {
  constexpr int kSlots = 256, kTilesPerStep = 80, kMinChunk = 128, kMaxTiles = 3 * kFc1MinBlocks * 64 / 128;
  int best = k1p, best_cost = INT_MAX;
  for (int s = 1; s == 1 || (s * rt <= kMaxTiles && s * kMinChunk <= k1p + kMinChunk); ++s) {
    const int chunk = std::max(kMinChunk, ((k1p + s - 1) / s + 63) / 64 * 64);
    const int tiles = rt * ((k1p + chunk - 1) / chunk);
    const int cost = kTilesPerStep * ((tiles + kSlots - 1) / kSlots) * (chunk / 64) + tiles;
    if (cost < best_cost) { best = chunk; best_cost = cost; }
  }
  return std::min(best, k1p);
}

// Gradient at `off`, [n][k] += sum_m d[m][n] x[m][k], its partial sums in `part` for `red`.  256 x 256 tiles read FC1's
// large operand once, but leave the chip idle where there are few of them or few rows (GEMM and reduction, us, small /
// large tiles: FC1's weight 19 / 28 at 96 rows, 27 / 29 at 750, 37 / 43 at 3000, 81 / 74 at 9000; FC2's at 9000 rows
// 16 / 22, one of the GRU's 21 / 24).
hipError_t weight_grad(const gemm_tn::Operands& g, int64_t max_slices, float* part, int64_t off, Reducer& red,
                       hipStream_t st) {
  constexpr int kLargeTiles = 32, kLargeRows = 6144;
  const int T = gemm_tn::tiles(g.N, g.K, 256) >= kLargeTiles && g.M >= kLargeRows ? 256 : 128;
  const int S = weight_slices(g.M, T, gemm_tn::tiles(g.N, g.K, T), max_slices);
  red.add(part, gemm_tn::slices(g.M, S), (int64_t)g.N * g.K, off);
  return gemm_tn::run(g, part, T, S, st);
}

// Where a backward pass leaves the partial sums of its weight and bias gradients, side by side, as they are reduced in
// one launch at its end: FC1's weight, FC2's or the GRU's W_ih, W_hh, the GRU's biases, FC1's bias, the encoder's.  At
// 360 rays 132 MB a handle (217 with the GRU), also of one that only runs forward; one region for all in turn took
// 105, and a launch for each.
struct PartRegions {
  int64_t w1, w2, whh, gb, b1, conv, total;
};

PartRegions part_regions(const aslam_policy* p) {
  PartRegions r{};
  r.w2 = kFc1Splits * 256 * p->off.k1;
  r.whh = r.w2 + kFc2Splits * (p->rec ? kGates : kHid) * kHid;
  r.gb = r.whh + (p->rec ? (int64_t)kFc2Splits * kGates * kHid : 0);
  r.b1 = r.gb + (p->rec ? std::max<int64_t>(256, (p->max_b + 15) / 16) * 2 * kGates : 0);
  r.conv = r.b1 + (int64_t)kBiasBlocks * 256;
  r.total = r.conv + (int64_t)kConvBwdGrid * kConvPart;
  return r;
}

int64_t part_need(const aslam_policy* p) {
  int64_t need = part_regions(p).total;
  need = std::max<int64_t>(need, (int64_t)kFc1MinBlocks * 64 * kHid);   // FC1 forward split-K: S * B <= 512 * 64
  if (p->prec)   // the three products of a split FC1, over z (S * B <= 512 * 64 each, or one slice of more rows)
    need = std::max<int64_t>(need, 3 * std::max<int64_t>((int64_t)kFc1MinBlocks * 64, p->max_b) * kHid);
  return need;
}

#define PCHK(e)                                                      \
  do {                                                               \
    hipError_t e_ = (e);                                             \
    if (e_ != hipSuccess) return pfail(ASL_EHIP, hipGetErrorString(e_)); \
  } while (0)

// The MLP policy's weight preparation in one launch, the jobs taken by workgroup ranges in this order:
// kPrepFrags form the encoder's fragments, an element a thread (the forward's, with PREC their lo parts, with
// `transposed` the backward's phase fragments: gathers, so they start first; as one last workgroup's loop they
// were the launch's tail: 15.5 us, now 9), kPrepW1 convert W1 (and its lo part), kPrepW2 convert W2, then with
// `transposed` the 32 x 32 tiles of W1's conv-feature columns and of W2 transposed.  Each job does what its own
// kernel (k_convert_bf16, k_transpose_bf16, k_conv_frags, k_conv_bwd_frags) does, value for value; one launch
// instead of up to seven per parameter update.
constexpr int kPrepFrags = (64 * (2 * kConvFrags + kConvPhaseFrags) + 255) / 256;
constexpr int kPrepW1 = 1024, kPrepW2 = 256;
constexpr int kPrepT1 = (kFeat / 32) * (kHid / 32), kPrepT2 = (kHid / 32) * (kHid / 32);

__global__ __launch_bounds__(256) void k_prep_mlp(const float* __restrict__ prm, Offsets o, int k1p,
                                                  uint16_t* w1b, uint16_t* w1b_lo, uint16_t* w2b, uint16_t* w2b_lo,
                                                  uint16_t* w1t, uint16_t* w2t, uint4* cfrag, int transposed) {
  __shared__ float tile[32][33];
  int b = blockIdx.x;
  if (b < kPrepFrags) {
    int t = b * 256 + threadIdx.x;
    if (t < 64 * kConvFrags) {
      conv_frag_elem<false>(prm, o, cfrag, t);
    } else if ((t -= 64 * kConvFrags) < 64 * kConvFrags) {
      if (w1b_lo) conv_frag_elem<true>(prm, o, cfrag + 64 * kConvLoFrag, t);
    } else if ((t -= 64 * kConvFrags) < 64 * kConvPhaseFrags) {
      if (transposed) conv_bwd_frag_elem(prm, o, cfrag, t);
    }
    return;
  }
  b -= kPrepFrags;
  if (b < kPrepW1) {
    convert_bf16_part(prm + o.f1w, o.k1, kHid, o.k1, w1b, k1p, w1b_lo, b, kPrepW1);
    return;
  }
  b -= kPrepW1;
  if (b < kPrepW2) {
    convert_bf16_part(prm + o.f2w, kHid, kHid, kHid, w2b, kHid, w2b_lo, b, kPrepW2);
    return;
  }
  b -= kPrepW2;
  if (transposed) {
    if (b < kPrepT1) {
      transpose_bf16_tile(prm + o.f1w, o.k1, kHid, kFeat, w1t, kHid, tile, b % (kFeat / 32), b / (kFeat / 32));
      return;
    }
    b -= kPrepT1;
    transpose_bf16_tile(prm + o.f2w, kHid, kHid, kHid, w2t, kHid, tile, b % (kHid / 32), b / (kHid / 32));
  }
}

// BF16 copies of W1 (rows padded to k1p) and W2 and the encoder's weight fragments that the forward
// reads; with `transposed` also what only the backward reads (the transposes for the input gradients,
// the encoder backward's phase fragments).
int convert_weights(aslam_policy* P, const float* prm, hipStream_t st, bool transposed) {
  const Offsets& o = P->off;
  if (P->rec) {
    k_convert_bf16<<<1024, 256, 0, st>>>(prm + o.f1w, o.k1, kHid, o.k1, P->w1b, P->k1p, P->prec ? P->w1b_lo : nullptr);
    PCHK(hipGetLastError());
    k_convert_bf16<<<768, 256, 0, st>>>(prm + o.gih, kHid, kGates, kHid, P->wihb, kHid);
    PCHK(hipGetLastError());
    k_convert_bf16<<<768, 256, 0, st>>>(prm + o.ghh, kHid, kGates, kHid, P->whhb, kHid);
    PCHK(hipGetLastError());
    k_conv_frags<<<1, 64 * kConvFrags, 0, st>>>(prm, o, P->cfrag);
    PCHK(hipGetLastError());
    if (transposed) {
      k_conv_bwd_frags<<<1, 64 * kConvPhaseFrags, 0, st>>>(prm, o, P->cfrag);
      PCHK(hipGetLastError());
      k_transpose_bf16<<<dim3(kFeat / 32, kHid / 32), 256, 0, st>>>(prm + o.f1w, o.k1, kHid, kFeat, P->w1t, kHid);
      PCHK(hipGetLastError());
      k_transpose_bf16<<<dim3(kHid / 32, kGates / 32), 256, 0, st>>>(prm + o.gih, kHid, kGates, kHid, P->wiht, kGates);
      PCHK(hipGetLastError());
      k_transpose_bf16<<<dim3(kHid / 32, kGates / 32), 256, 0, st>>>(prm + o.ghh, kHid, kGates, kHid, P->whht, kGates);
      PCHK(hipGetLastError());
    }
    P->prepared = true;
    return ASL_OK;
  }
  const int blocks = kPrepFrags + kPrepW1 + kPrepW2 + (transposed ? kPrepT1 + kPrepT2 : 0);
  k_prep_mlp<<<blocks, 256, 0, st>>>(prm, o, P->k1p, P->w1b, P->prec ? P->w1b_lo : nullptr, P->w2b,
                                     P->prec ? P->w2b_lo : nullptr, P->w1t, P->w2t, P->cfrag, transposed ? 1 : 0);
  PCHK(hipGetLastError());
  P->prepared = true;
  return ASL_OK;
}

// Encoder (conv features and the scan / state tail into the FC1 input x) and FC1.  Small batches
// split K so that the launch fills the chip: then *S_used split-K slices are left in P->part;
// otherwise FC1 writes h1 = bf16(relu(. + b1)) and *S_used = 0.
int encode_fc1(aslam_policy* P, const float* prm, const int16_t* crop, const float* scan, const float* state,
               const int32_t* rows, int B, hipStream_t st, int* S_used, bool training = false) {
  (P->prec ? (training ? k_conv_fwd<true, true> : k_conv_fwd<true, false>)
           : (training ? k_conv_fwd<false, true> : k_conv_fwd<false, false>))<<<
      std::min(B, P->prec ? kConvGridPrec : kConvGrid), kConvFwdThreads, 0, st>>>(
      prm, P->off, P->cfrag, crop, scan, state, P->cfg.n_scan, rows, P->x, P->x_lo, P->k1p, B, P->amask);
  PCHK(hipGetLastError());
  // FC1: [B x k1] x [k1 x 256] (both operands zero-padded from k1 to k1p)
  const int K1 = (int)((P->off.k1 + 7) / 8 * 8);
  // as many K splits as keep the grid within one round of kFc1MinBlocks resident workgroups; with the three
  // split-precision products of a training pass and few row tiles a third of that: the products fill the round
  // themselves, and more slices would only add partial-sum traffic (at 750 rows, 32 splits of 3 products wrote and
  // re-read 74 MB of partial sums per call)
  const int tiles = ((B + 127) / 128) * (kHid / 128);
  int S = std::max(1, std::min(32, kFc1MinBlocks / tiles));
  if (P->prec && tiles < 32) S = std::max(1, std::min(32, kFc1MinBlocks / (3 * tiles)));
  const int64_t slice = (int64_t)B * kHid;
  if (P->prec && !training) {
    // Forward only: the three products summed by the workgroup, so that a slice is a third of the partial sums (128 x
    // 128 tiles with each product in slices of its own, GEMM and reduction: 14 us at 16 rows, 34 at 750, 75 at 2000,
    // 228 at 8000; this: 12, 28, 43, 137).  The training pass keeps its slices: its ReLU signs, and so its gradients,
    // follow their rounding.
    const int k_split = split_fc1_chunk(P->k1p, (B + 127) / 128);
    PCHK(gemm_nt::run<3>(gemm_nt::Operands{P->x, P->x_lo, P->w1b, P->w1b_lo, P->k1p, P->k1p, B, kHid, P->k1p},
                         gemm_nt::EpiSum{{P->part, kHid, slice}}, k_split, st));
    *S_used = (int)((P->k1p + k_split - 1) / k_split);
    return ASL_OK;
  }
  const int nz = slices_used(K1, S, 64);
  // The wide kernel (128 x 256 tiles, one workgroup per CU) from where its tiles and slices come near a round of the
  // CUs; below that the 128 x 128 tiles, with each split-precision product in slices of its own.  Engine / wide, us: a
  // BF16 forward 39.8 / 39.9 at 400 rows (128 workgroups), 41.9 / 40.1 at 513 (160), 57.2 / 53.3 at 2000; a split
  // minibatch, whose six slices leave the wide tiles few, 192 / 206 at 750 rows (36 workgroups), 239 / 265 at 1600
  // (78), 280 / 268 at 2000 (256).
  if (S == 1 || (B + 127) / 128 * nz >= kFc1WideBlocks) {
    const gemm_nt::Operands fc1{P->x, P->x_lo, P->w1b, P->w1b_lo, P->k1p, P->k1p, B, kHid, P->k1p};
    const int k_split = ((K1 + S - 1) / S + 63) / 64 * 64;
    const gemm_nt::EpiPartial part{P->part, kHid, slice};
    if (P->prec) PCHK(gemm_nt::run<3>(fc1, part, k_split, st));
    else if (S == 1) PCHK(gemm_nt::run<1>(fc1, gemm_nt::EpiBiasRelu{P->h1, prm + P->off.f1b, kHid}, k_split, st));
    else PCHK(gemm_nt::run<1>(fc1, part, k_split, st));
    *S_used = P->prec ? 3 * nz : S == 1 ? 0 : nz;
    return ASL_OK;
  }
  const LdBF16K xa{P->x, P->k1p, B, K1};
  const LdBF16K wa{P->w1b, P->k1p, kHid, K1};
  if (P->prec) {
    // x_hi W_hi, x_hi W_lo and x_lo W_hi, each split S ways, into consecutive groups of slices (one
    // launch, the products over z: product 1 reads W's lo part, product 2 x's)
    PCHK((gemm::run<128, 128, 64, 2, 2>(gemm::HiLo<LdBF16K>{xa, LdBF16K{P->x_lo, P->k1p, B, K1}, 4u},
                                         gemm::HiLo<LdBF16K>{wa, LdBF16K{P->w1b_lo, P->k1p, kHid, K1}, 2u},
                                         EpiPartial{P->part, kHid, slice}, B, kHid, K1, S, st, 3)));
    *S_used = 3 * nz;
  } else {
    *S_used = nz;
    PCHK((gemm::run<128, 128, 64, 2, 2>(xa, wa, EpiPartial{P->part, kHid, slice}, B, kHid, K1, S, st)));
  }
  return ASL_OK;
}

// The backward's forward: every weight copy, the encoder, FC1 to h1 and the FC2 pre-activation z2 (FP32).
int forward_core(aslam_policy* P, const float* prm, const int16_t* crop, const float* scan, const float* state,
                 const int32_t* rows, int B, hipStream_t st) {
  const Offsets& o = P->off;
  int rc = convert_weights(P, prm, st, true);
  if (rc) return rc;
  int S = 0;
  rc = encode_fc1(P, prm, crop, scan, state, rows, B, st, &S, true);
  if (rc) return rc;
  if (S > 0) {
    PCHK(launch_reduce_relu(P->part, S, B, prm + o.f1b, P->h1, P->prec ? P->h1_lo : nullptr, st));
  }
  const LdBF16K ha{P->h1, kHid, B, kHid}, wb{P->w2b, kHid, kHid, kHid};
  if (P->prec) {
    // z2 = h1_hi W2_hi + h1_hi W2_lo + h1_lo W2_hi + b2, the three products in one accumulator
    PCHK((gemm::run<128, 128, 64, 2, 2>(gemm::HiLo<LdBF16K>{ha, LdBF16K{P->h1_lo, kHid, B, kHid}, 4u},
                                       gemm::HiLo<LdBF16K>{wb, LdBF16K{P->w2b_lo, kHid, kHid, kHid}, 2u},
                                       EpiBiasF32{P->z2, prm + o.f2b, kHid}, B, kHid, kHid, 1, st, 3, true)));
    return ASL_OK;
  }
  PCHK((gemm::run<128, 128, 64, 2, 2>(ha, wb, EpiBiasF32{P->z2, prm + o.f2b, kHid}, B, kHid, kHid, 1, st)));
  return ASL_OK;
}

// Forward-only pass: encoder, FC1, then the fused tail (FC2, heads and, with eps, the sample).
int act_core(aslam_policy* P, const float* prm, bool prepared, const int16_t* crop, const float* scan,
             const float* state, int B, bool sample, ActDraws eps, float* mu, float* value, float* act,
             float* logp, hipStream_t st) {
  if (!prepared) {
    int rc = convert_weights(P, prm, st, false);
    if (rc) return rc;
  }
  int S = 0;
  int rc = encode_fc1(P, prm, crop, scan, state, nullptr, B, st, &S);
  if (rc) return rc;
  if (S > 8) {
    // many split-K slices: their sum is spread over the chip first (the tail kernel has B / 16 workgroups)
    const int64_t groups = (int64_t)B * (kHid / 8);
    k_reduce_bias_relu_bf16_q<<<(unsigned)((groups + 63) / 64), 256, 0, st>>>(P->part, S, B, kHid, prm + P->off.f1b,
                                                                              P->h1, kHid, P->prec ? P->h1_lo : nullptr);
    PCHK(hipGetLastError());
    S = 0;
  }
  const int tail_blocks = (B + kTailRows - 1) / kTailRows;
  const bool many = B >= kTailManyRows;
  (P->prec ? (many ? k_fwd_tail<true, 4> : k_fwd_tail<true, 16>)
           : (many ? k_fwd_tail<false, 4> : k_fwd_tail<false, 16>))<<<tail_blocks, many ? 256 : 1024, 0, st>>>(
      prm, P->off, P->part, S, P->h1, P->prec ? P->h1_lo : nullptr, P->w2b, P->prec ? P->w2b_lo : nullptr, B, mu, value,
      sample, eps, act, logp);
  PCHK(hipGetLastError());
  return ASL_OK;
}

int backward_fc1_encoder(aslam_policy* P, const float* params, const int16_t* crop, const int32_t* rows, int B,
                         Reducer& red, float* grads, hipStream_t st);

}  // namespace

extern "C" {

int64_t aslam_policy_num_params(int32_t n_scan) {
  if (n_scan < 0) return -1;
  return offsets(n_scan).total;
}

int aslam_policy_create(const aslam_policy_config* cfg, aslam_policy** out) {
  if (!cfg || !out) return pfail(ASL_EINVAL, "config or out is NULL");
  *out = nullptr;
  if (cfg->n_scan < 1 || cfg->n_scan > 4096) return pfail(ASL_EINVAL, "n_scan must be in [1, 4096]");
  if (cfg->max_batch < 1 || cfg->max_batch > (1 << 20)) return pfail(ASL_EINVAL, "max_batch must be in [1, 2^20]");
  if (cfg->recurrent != 0 && cfg->recurrent != 1) return pfail(ASL_EINVAL, "recurrent must be 0 or 1");
  if (cfg->precision != 0 && cfg->precision != 1) return pfail(ASL_EINVAL, "precision must be 0 or 1");
  if (cfg->precision == 1 && cfg->recurrent == 1)
    return pfail(ASL_ENOTIMPL, "the split-precision forward is built for the feed-forward policy only");
  aslam_policy* p = new (std::nothrow) aslam_policy();
  if (!p) return pfail(ASL_ENOMEM, "host allocation failed");
  p->cfg = *cfg;
  p->rec = cfg->recurrent == 1;
  p->prec = cfg->precision == 1;
  p->off = offsets(cfg->n_scan, p->rec);
  p->max_b = cfg->max_batch;
  const int64_t Bm = p->max_b;
  p->part_floats = part_need(p);
  p->k1p = fc1_pitch(p->off.k1);
  struct A { void** ptr; size_t bytes; } al[] = {
      {(void**)&p->x, 2 * (size_t)Bm * p->k1p},  {(void**)&p->h1, 2 * (size_t)Bm * kHid},
      {(void**)&p->dz2, 2 * (size_t)Bm * kHid},  {(void**)&p->dz1, 2 * (size_t)Bm * kHid},
      {(void**)&p->dz2c, 2 * (size_t)Bm * kFeat}, {(void**)&p->amask, (size_t)Bm * kFeat / 8},
      {(void**)&p->z2, 4 * (size_t)Bm * kHid},
      {(void**)&p->part, 4 * (size_t)p->part_floats},
      {(void**)&p->hpart, 4 * (size_t)((Bm + kHeadRows - 1) / kHeadRows) * kHeadPart},
      {(void**)&p->w1b, 2 * (size_t)kHid * p->k1p}, {(void**)&p->w1t, 2 * (size_t)kFeat * kHid},
      {(void**)&p->w2b, 2 * (size_t)kHid * kHid},                        {(void**)&p->w2t, 2 * (size_t)kHid * kHid},
      {(void**)&p->cfrag, sizeof(uint4) * 64 * kConvFragsAll},
  };
  for (auto& a : al) {
    if (hipMalloc(a.ptr, a.bytes) != hipSuccess) {
      aslam_policy_destroy(p);
      return pfail(ASL_ENOMEM, "hipMalloc of policy workspace failed");
    }
  }
  if (p->prec) {
    struct A pl[] = {
        {(void**)&p->x_lo, 2 * (size_t)Bm * p->k1p}, {(void**)&p->h1_lo, 2 * (size_t)Bm * kHid},
        {(void**)&p->w1b_lo, 2 * (size_t)kHid * p->k1p}, {(void**)&p->w2b_lo, 2 * (size_t)kHid * kHid},
    };
    for (auto& a : pl) {
      if (hipMalloc(a.ptr, a.bytes) != hipSuccess) {
        aslam_policy_destroy(p);
        return pfail(ASL_ENOMEM, "hipMalloc of policy workspace failed");
      }
    }
  }
  if (p->rec) {
    const size_t f = 4 * (size_t)Bm * kHid, h = 2 * (size_t)Bm * kHid, g = 2 * (size_t)Bm * kGates;
    const size_t w = 2 * (size_t)kGates * kHid;
    struct A rl[] = {
        {(void**)&p->wihb, w}, {(void**)&p->whhb, w}, {(void**)&p->wiht, w}, {(void**)&p->whht, w},
        {(void**)&p->hst, f}, {(void**)&p->g_r, f}, {(void**)&p->g_z, f}, {(void**)&p->g_n, f},
        {(void**)&p->g_ghn, f}, {(void**)&p->dh_head, f},
        {(void**)&p->hp_bf, h}, {(void**)&p->dg, 2 * g},
        {(void**)&p->rows, 4 * (size_t)Bm},
    };
    for (auto& a : rl) {
      if (hipMalloc(a.ptr, a.bytes) != hipSuccess) {
        aslam_policy_destroy(p);
        return pfail(ASL_ENOMEM, "hipMalloc of policy workspace failed");
      }
    }
    hipError_t e = hipSuccess;
    for (const void* f : {reinterpret_cast<const void*>(&k_gru_seq_fwd<1>), reinterpret_cast<const void*>(&k_gru_seq_fwd<2>),
                          reinterpret_cast<const void*>(&k_gru_seq_fwd<4>)})
      if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kGruSeqFwdLds);
    for (const void* f : {reinterpret_cast<const void*>(&k_gru_seq_bwd<1>), reinterpret_cast<const void*>(&k_gru_seq_bwd<2>),
                          reinterpret_cast<const void*>(&k_gru_seq_bwd<4>)})
      if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kGruSeqBwdLds);
    if (e != hipSuccess) {
      aslam_policy_destroy(p);
      return pfail(ASL_EHIP, hipGetErrorString(e));
    }
  }
  *out = p;
  return ASL_OK;
}

int64_t aslam_policy_param_count(const aslam_policy_config* cfg) {
  if (!cfg || cfg->n_scan < 0 || (cfg->recurrent != 0 && cfg->recurrent != 1)) return -1;
  return offsets(cfg->n_scan, cfg->recurrent == 1).total;
}

int aslam_policy_destroy(aslam_policy* p) {
  if (!p) return pfail(ASL_EINVAL, "policy is NULL");
  void* ptrs[] = {p->x, p->h1, p->dz2, p->dz1, p->dz2c, p->amask, p->z2, p->part, p->hpart,
                  p->w1b, p->w1t, p->w2b, p->w2t, p->cfrag,
                  p->wihb, p->whhb, p->wiht, p->whht, p->hst, p->g_r, p->g_z, p->g_n, p->g_ghn,
                  p->dh_head, p->hp_bf, p->dg, p->rows, p->x_lo, p->h1_lo, p->w1b_lo,
                  p->w2b_lo};
  for (void* q : ptrs)
    if (q) (void)hipFree(q);
  delete p;
  return ASL_OK;
}

int aslam_policy_forward(aslam_policy* P, const float* params, const int16_t* crop, const float* scan,
                         const float* state, int32_t batch, float* mu, float* value, aslam_stream_t stream) {
  if (!P || !params || !crop || !scan || !state || !mu || !value) return pfail(ASL_EINVAL, "null argument");
  if (batch < 1 || batch > P->max_b) return pfail(ASL_EINVAL, "batch must be in [1, max_batch]");
  if (P->rec) return pfail(ASL_EINVAL, "recurrent policy: use aslam_policy_act_rnn");
  return act_core(P, params, false, crop, scan, state, batch, false, ActDraws{nullptr, 0, 0}, mu, value, nullptr,
                  nullptr, (hipStream_t)stream);
}

}  // extern "C"

// ------------------------------------------------------------------ forward without allocation
//
// aslam_policy_forward_noalloc keeps what the forward stages between its kernels (the BF16 weight
// copies, the encoder's weight fragments, the FC1 input rows, FC1's split-K partial sums and the
// hidden rows) in one file-scope device array instead of a handle's allocations.  Its layout is fixed
// for the largest scan and batch it accepts.  Host code never passes the array's name to a kernel:
// the device address is looked up once per device with hipGetSymbolAddress and kept.
namespace {
constexpr int64_t kNoAllocMaxScan = 720;
constexpr int64_t kNoAllocMaxBatch = 256;
constexpr int64_t kNoAllocK1p = fc1_pitch(kFeat + kNoAllocMaxScan + 12);
constexpr int64_t align256(int64_t v) { return (v + 255) / 256 * 256; }
constexpr int64_t kNaW1b = 0;
constexpr int64_t kNaW2b = kNaW1b + align256(2 * kHid * kNoAllocK1p);
constexpr int64_t kNaFrag = kNaW2b + align256(2 * kHid * kHid);
constexpr int64_t kNaX = kNaFrag + align256(16 * 64 * (kConvFrags + kConvPhaseFrags));
constexpr int64_t kNaH1 = kNaX + align256(2 * kNoAllocMaxBatch * kNoAllocK1p);
constexpr int64_t kNaPart = kNaH1 + align256(2 * kNoAllocMaxBatch * kHid);
constexpr int64_t kNaBytes = kNaPart + align256(4 * 32 * kNoAllocMaxBatch * kHid);   // at most 32 K slices
}  // namespace

static __device__ __align__(256) unsigned char scratch[kNaBytes];

namespace {
std::mutex g_scratch_mu;
std::vector<unsigned char*> g_scratch_ptr;   // per device: the array's device address, looked up once

int scratch_for_current_device(unsigned char** out) {
  int dev = 0;
  PCHK(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if ((int)g_scratch_ptr.size() <= dev) g_scratch_ptr.resize(dev + 1, nullptr);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    PCHK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return pfail(ASL_EHIP, "hipGetSymbolAddress returned no address for the forward's scratch");
    g_scratch_ptr[dev] = static_cast<unsigned char*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return ASL_OK;
}

}  // namespace

extern "C" {

int64_t aslam_policy_noalloc_limits(int32_t* max_scan, int32_t* max_batch) {
  if (max_scan) *max_scan = (int32_t)kNoAllocMaxScan;
  if (max_batch) *max_batch = (int32_t)kNoAllocMaxBatch;
  return kNaBytes;
}

int aslam_policy_forward_noalloc(const float* params, int32_t n_scan, const int16_t* crop, const float* scan,
                                 const float* state, int32_t batch, float* mu, float* value, aslam_stream_t stream) {
  if (!params || !crop || !scan || !state || !mu || !value) return pfail(ASL_EINVAL, "null argument");
  if (n_scan < 1 || n_scan > kNoAllocMaxScan)
    return pfail(ASL_EINVAL, "forward_noalloc: n_scan must be in [1, " + std::to_string(kNoAllocMaxScan) + "]");
  if (batch < 1 || batch > kNoAllocMaxBatch)
    return pfail(ASL_EINVAL, "forward_noalloc: batch must be in [1, " + std::to_string(kNoAllocMaxBatch) +
                                 "] (the scratch array is sized for that)");
  unsigned char* base = nullptr;
  int rc = scratch_for_current_device(&base);
  if (rc) return rc;
  // a handle on the stack whose workspaces are views of the scratch array: the same kernels as
  // aslam_policy_forward, in the same order, with the same split of FC1's K
  aslam_policy P{};
  P.cfg.n_scan = n_scan;
  P.cfg.max_batch = batch;
  P.off = offsets(n_scan);
  P.max_b = batch;
  P.k1p = fc1_pitch(P.off.k1);
  P.w1b = reinterpret_cast<uint16_t*>(base + kNaW1b);
  P.w2b = reinterpret_cast<uint16_t*>(base + kNaW2b);
  P.cfrag = reinterpret_cast<uint4*>(base + kNaFrag);
  P.x = reinterpret_cast<uint16_t*>(base + kNaX);
  P.h1 = reinterpret_cast<uint16_t*>(base + kNaH1);
  P.part = reinterpret_cast<float*>(base + kNaPart);
  return act_core(&P, params, false, crop, scan, state, batch, false, ActDraws{nullptr, 0, 0}, mu, value, nullptr,
                  nullptr, (hipStream_t)stream);
}

int aslam_policy_prepare(aslam_policy* P, const float* params, aslam_stream_t stream) {
  if (!P || !params) return pfail(ASL_EINVAL, "null argument");
  return convert_weights(P, params, (hipStream_t)stream, false);
}

int aslam_policy_act(aslam_policy* P, const float* params, int32_t prepared, const int16_t* crop, const float* scan,
                     const float* state, int32_t batch, const float* eps, uint64_t seed, uint64_t counter, float* mu,
                     float* value, float* act, float* logp, aslam_stream_t stream) {
  if (!P || !params || !crop || !scan || !state || !value || !act || !logp)
    return pfail(ASL_EINVAL, "null argument");
  if (batch < 1 || batch > P->max_b) return pfail(ASL_EINVAL, "batch must be in [1, max_batch]");
  if (P->rec) return pfail(ASL_EINVAL, "recurrent policy: use aslam_policy_act_rnn");
  if (prepared && !P->prepared) return pfail(ASL_ESTATE, "act with prepared = 1 before any prepare");
  return act_core(P, params, prepared != 0, crop, scan, state, batch, true, ActDraws{eps, seed, counter}, mu, value,
                  act, logp, (hipStream_t)stream);
}

int aslam_policy_backward(aslam_policy* P, const float* params, const int16_t* crop, const float* scan,
                          const float* state, int32_t batch, const float* act, const float* old_logp,
                          const float* adv, const float* ret, float* grads, float* loss, aslam_stream_t stream) {
  return aslam_policy_backward_rows(P, params, crop, scan, state, nullptr, batch, act, old_logp, adv, ret, grads,
                                    loss, stream);
}

int aslam_policy_backward_rows(aslam_policy* P, const float* params, const int16_t* crop, const float* scan,
                               const float* state, const int32_t* rows, int32_t batch, const float* act,
                               const float* old_logp, const float* adv, const float* ret, float* grads, float* loss,
                               aslam_stream_t stream) {
  if (!P || !params || !crop || !scan || !state || !act || !old_logp || !adv || !ret || !grads || !loss)
    return pfail(ASL_EINVAL, "null argument");
  if (batch < 1 || batch > P->max_b) return pfail(ASL_EINVAL, "batch must be in [1, max_batch]");
  if (P->rec) return pfail(ASL_EINVAL, "recurrent policy: use aslam_policy_backward_seq");
  hipStream_t st = (hipStream_t)stream;
  const Offsets& o = P->off;
  const int B = batch;
  int rc = forward_core(P, params, crop, scan, state, rows, B, st);
  if (rc) return rc;
  // heads + loss -> dz2, head / fc2-bias / log-std partial sums
  const int nb = (B + kHeadRows - 1) / kHeadRows;
  LossCoef lc{P->cfg.clip_eps, P->cfg.c_value, P->cfg.c_entropy, 1.0f / (float)B};
  k_heads<true><<<nb, kHeadThreads, 0, st>>>(params, o, P->z2, B, nullptr, nullptr, act, old_logp, adv, ret, rows, lc, P->dz2,
                                    P->hpart);
  PCHK(hipGetLastError());
  PCHK(launch_reduce_heads(P->hpart, nb, params, o, grads, loss, P->cfg.c_value, P->cfg.c_entropy, st));
  // FC2 weight: dW2[out][in] = sum_b dz2[b][out] h1[b][in]
  const PartRegions pr = part_regions(P);
  Reducer red;
  PCHK(weight_grad(gemm_tn::Operands{P->dz2, kHid, kHid, P->h1, kHid, kHid, B}, kFc2Splits, P->part + pr.w2, o.f2w, red,
                   st));
  // dh1 -> dz1 = (dz2 W2) * [h1 > 0]
  PCHK((gemm::run<128, 128, 64, 2, 2>(LdBF16K{P->dz2, kHid, B, kHid}, LdBF16K{P->w2t, kHid, kHid, kHid},
                                     EpiReluGradBF16{P->dz1, P->h1, kHid, kHid}, B, kHid, kHid, 1, st)));
  return backward_fc1_encoder(P, params, crop, rows, B, red, grads, st);
}

}  // extern "C"

namespace {

// Everything below the FC1 output gradient dz1 (BF16, already masked by FC1's ReLU): the FC1 bias and
// weight gradients, the conv-feature gradient and the encoder backward.
int backward_fc1_encoder(aslam_policy* P, const float* params, const int16_t* crop, const int32_t* rows, int B,
                         Reducer& red, float* grads, hipStream_t st) {
  const Offsets& o = P->off;
  const PartRegions pr = part_regions(P);
  // FC1 bias
  k_bias_rows<<<kBiasBlocks, 256, 0, st>>>(P->dz1, B, kHid, P->part + pr.b1);
  PCHK(hipGetLastError());
  red.add(P->part + pr.b1, kBiasBlocks, kHid, o.f1b);
  // FC1 weight: dW1[out][k] = sum_b dz1[b][out] X[b][k]
  PCHK(weight_grad(gemm_tn::Operands{P->dz1, kHid, kHid, P->x, P->k1p, o.k1, B}, kFc1Splits, P->part + pr.w1, o.f1w, red,
                   st));
  // dA2 -> dz2c = (dz1 W1[:, :8192]) * [a2 > 0]
  PCHK(gemm_nt::feature_grad(P->dz1, P->w1t, reinterpret_cast<const uint8_t*>(P->amask), P->dz2c, B, kFeat, st));
  // encoder: conv2 / conv1 weight and bias gradients in one pass over the minibatch
  {
    const int grid = std::min(B, kConvBwdGrid);
    if (P->prec)
      k_conv_bwd<true><<<grid, kBwdThreads, 0, st>>>(params, o, P->cfrag, crop, rows, P->dz2c, B, P->part + pr.conv);
    else
      k_conv_bwd<false><<<grid, kBwdThreads, 0, st>>>(params, o, P->cfrag, crop, rows, P->dz2c, B, P->part + pr.conv);
    PCHK(hipGetLastError());
    const ReduceSegs sg{{kConvPartW2, kConvPartW1, kC1, kC2}, {1, 2, 0, 0}, {o.c2w, o.c1w, o.c1b, o.c2b}};
    red.add(P->part + pr.conv, grid, kConvPart, sg);
  }
  PCHK(red.launch(grads, st));
  return ASL_OK;
}

}  // namespace

extern "C" {

int aslam_policy_sample(aslam_policy* P, const float* params, const float* mu, const float* eps, uint64_t seed,
                        uint64_t counter, int32_t batch, float* act, float* logp, aslam_stream_t stream) {
  if (!P || !params || !mu || !act || !logp) return pfail(ASL_EINVAL, "null argument");
  if (batch < 1) return pfail(ASL_EINVAL, "batch must be >= 1");
  k_sample<<<(batch + 255) / 256, 256, 0, (hipStream_t)stream>>>(params, P->off, mu, ActDraws{eps, seed, counter},
                                                                  batch, act, logp);
  PCHK(hipGetLastError());
  return ASL_OK;
}

int64_t aslam_permutation_work_bytes(int32_t n) {
  if (n <= 0) return 0;
  return (int64_t)4 << (2 * rng::perm_half_bits(n));
}

int aslam_permutation(int32_t n, uint64_t seed, uint64_t counter, int32_t* out, void* work, int64_t work_bytes,
                      aslam_stream_t stream) {
  if (n < 0) return pfail(ASL_EINVAL, "n must be >= 0");
  if (n == 0) return ASL_OK;
  if (!out) return pfail(ASL_EINVAL, "null argument");
  const int h = rng::perm_half_bits(n);
  hipStream_t st = (hipStream_t)stream;
  if (!work) {
    k_permutation<<<(n + 255) / 256, 256, 0, st>>>(n, h, seed, counter, out);
  } else {
    const int64_t dom = (int64_t)1 << (2 * h);
    if (work_bytes < 4 * dom) return pfail(ASL_EINVAL, "work_bytes below aslam_permutation_work_bytes(n)");
    if ((uintptr_t)work & 3) return pfail(ASL_EINVAL, "work must be 4-byte aligned");
    uint32_t* tab = static_cast<uint32_t*>(work);
    k_feistel_table<<<(unsigned)((dom + 255) / 256), 256, 0, st>>>(h, seed, counter, tab);
    PCHK(hipGetLastError());
    k_permutation_walk<<<(n + 255) / 256, 256, 0, st>>>(n, tab, out);
  }
  PCHK(hipGetLastError());
  return ASL_OK;
}

int aslam_gather_rows(const void* src, int64_t row_bytes, const int32_t* idx, int32_t n, void* dst,
                      aslam_stream_t stream) {
  if (!src || !idx || !dst) return pfail(ASL_EINVAL, "null argument");
  if (n < 0 || row_bytes < 4 || (row_bytes & 3)) return pfail(ASL_EINVAL, "row_bytes must be a positive multiple of 4");
  if (((uintptr_t)src & 3) || ((uintptr_t)dst & 3)) return pfail(ASL_EINVAL, "src and dst must be 4-byte aligned");
  if (n == 0) return ASL_OK;
  const int vec = ((row_bytes & 15) == 0 && ((uintptr_t)src & 15) == 0 && ((uintptr_t)dst & 15) == 0) ? 1 : 0;
  const int64_t items = vec ? (int64_t)n * (row_bytes >> 4) : (int64_t)n * (row_bytes >> 2);
  const int blocks = (int)std::min<int64_t>(8192, (items + 255) / 256);
  k_gather_rows<<<blocks, 256, 0, (hipStream_t)stream>>>(static_cast<const uint32_t*>(src), row_bytes >> 2, idx, n,
                                                         static_cast<uint32_t*>(dst), vec);
  PCHK(hipGetLastError());
  return ASL_OK;
}

int aslam_gae(const float* rewards, const float* values, const uint8_t* dones, const float* last_value, int32_t T,
              int32_t N, float gamma, float lam, float* adv, float* ret, aslam_stream_t stream) {
  if (!rewards || !values || !dones || !last_value || !adv || !ret) return pfail(ASL_EINVAL, "null argument");
  if (T < 1 || N < 1) return pfail(ASL_EINVAL, "T and N must be >= 1");
  k_gae<<<(N + 255) / 256, 256, 0, (hipStream_t)stream>>>(rewards, values, dones, last_value, T, N, gamma, lam,
                                                           adv, ret);
  PCHK(hipGetLastError());
  return ASL_OK;
}

int aslam_adam(float* params, const float* grads, float* m, float* v, int64_t n, int32_t step, float lr,
               float beta1, float beta2, float eps, aslam_stream_t stream) {
  if (!params || !grads || !m || !v) return pfail(ASL_EINVAL, "null argument");
  if (n < 1 || step < 1) return pfail(ASL_EINVAL, "n and step must be >= 1");
  const float bc1 = (float)(1.0 - std::pow((double)beta1, (double)step));
  const float bc2 = (float)(1.0 - std::pow((double)beta2, (double)step));
  const int blocks = (int)std::min<int64_t>(4096, (n + 255) / 256);
  k_adam<<<blocks, 256, 0, (hipStream_t)stream>>>(params, grads, m, v, n, lr, beta1, beta2, eps, bc1, bc2);
  PCHK(hipGetLastError());
  return ASL_OK;
}

int aslam_policy_act_rnn(aslam_policy* P, const float* params, int32_t prepared, const int16_t* crop,
                         const float* scan, const float* state, int32_t batch, const float* h_in, const uint8_t* first,
                         const float* eps, uint64_t seed, uint64_t counter, float* mu, float* value, float* act,
                         float* logp, float* h_out, aslam_stream_t stream) {
  if (!P || !params || !crop || !scan || !state || !h_in || !value || !act || !logp || !h_out)
    return pfail(ASL_EINVAL, "null argument");
  if (!P->rec) return pfail(ASL_EINVAL, "feed-forward policy: use aslam_policy_act");
  if (batch < 1 || batch > P->max_b) return pfail(ASL_EINVAL, "batch must be in [1, max_batch]");
  if (prepared && !P->prepared) return pfail(ASL_ESTATE, "act_rnn with prepared = 1 before any prepare");
  hipStream_t st = (hipStream_t)stream;
  if (!prepared) {
    int rc = convert_weights(P, params, st, false);
    if (rc) return rc;
  }
  int S = 0;
  int rc = encode_fc1(P, params, crop, scan, state, nullptr, batch, st, &S);
  if (rc) return rc;
  if (S > 0) {   // the split-K slices summed over the whole chip first (h1 = bf16(relu(. + b1)))
    const int64_t groups = (int64_t)batch * (kHid / 8);
    if (S > 8)
      k_reduce_bias_relu_bf16_q<<<(unsigned)((groups + 63) / 64), 256, 0, st>>>(P->part, S, batch, kHid,
                                                                                params + P->off.f1b, P->h1, kHid);
    else
      k_reduce_bias_relu_bf16<<<(int)std::min<int64_t>(4096, (groups + 255) / 256), 256, 0, st>>>(
          P->part, S, batch, kHid, params + P->off.f1b, P->h1, kHid);
    PCHK(hipGetLastError());
  }
  // the step writes the new state to a workspace (h_out may alias h_in); the heads copy it out
  GruFwdArgs a{};
  a.prm = params; a.o = P->off; a.rows = batch;
  a.h1 = P->h1;
  a.wih = P->wihb; a.whh = P->whhb;
  a.hp = h_in; a.first = first;
  a.h_out = P->hst;
  k_gru_fwd<<<dim3((batch + kGruRows - 1) / kGruRows, kGruSlices), 256, 0, st>>>(a);
  PCHK(hipGetLastError());
  k_gru_heads<<<(batch + 3) / 4, 256, 0, st>>>(params, P->off, P->hst, batch, h_out, mu, value,
                                                ActDraws{eps, seed, counter}, act, logp);
  PCHK(hipGetLastError());
  return ASL_OK;
}

int aslam_policy_backward_seq(aslam_policy* P, const float* params, const int16_t* crop, const float* scan,
                              const float* state, int32_t T, int32_t N, const int32_t* robots, int32_t nb,
                              const float* h0, const uint8_t* first, const float* act, const float* old_logp,
                              const float* adv, const float* ret, float* grads, float* loss, aslam_stream_t stream) {
  if (!P || !params || !crop || !scan || !state || !robots || !h0 || !first || !act || !old_logp || !adv || !ret ||
      !grads || !loss)
    return pfail(ASL_EINVAL, "null argument");
  if (!P->rec) return pfail(ASL_EINVAL, "feed-forward policy: use aslam_policy_backward");
  if (T < 1 || N < 1 || nb < 1 || nb > N) return pfail(ASL_EINVAL, "need T >= 1 and 1 <= nb <= N");
  if ((int64_t)T * nb > P->max_b) return pfail(ASL_EINVAL, "T * nb exceeds max_batch");
  hipStream_t st = (hipStream_t)stream;
  const Offsets& o = P->off;
  const int B = T * nb;
  k_seq_rows<<<(B + 255) / 256, 256, 0, st>>>(robots, nb, T, N, P->rows);
  PCHK(hipGetLastError());
  int rc = convert_weights(P, params, st, true);
  if (rc) return rc;
  int S = 0;
  rc = encode_fc1(P, params, crop, scan, state, P->rows, B, st, &S, true);
  if (rc) return rc;
  if (S > 0) {
    PCHK(launch_reduce_relu(P->part, S, B, params + o.f1b, P->h1, nullptr, st));
  }
  // the GRU over the T steps: the input products of every sample at once, then the recurrence, keeping
  // what the backward reads
  GruSeqArgs a{};
  a.prm = params; a.o = o;
  a.nb = nb; a.T = T; a.N = N;
  a.robots = robots; a.h0 = h0; a.first = first;
  a.gi = reinterpret_cast<const float*>(P->dg); a.whh = P->whhb;
  a.hst = P->hst; a.g_r = P->g_r; a.g_z = P->g_z; a.g_n = P->g_n; a.g_ghn = P->g_ghn; a.hp_bf = P->hp_bf;
  const int rpl = gru_seq_rows(nb);
  const unsigned tiles = (unsigned)((nb + 4 * rpl - 1) / (4 * rpl));
  PCHK((gemm::run<128, 128, 64, 2, 2>(LdBF16K{P->h1, kHid, B, kHid}, LdBF16K{P->wihb, kHid, kGates, kHid},
                                     EpiPartial{reinterpret_cast<float*>(P->dg), kGates, 0}, B, kGates, kHid, 1, st)));
  (rpl == 1 ? k_gru_seq_fwd<1>
            : rpl == 2 ? k_gru_seq_fwd<2> : k_gru_seq_fwd<4>)<<<tiles, kGruSeqThreads, kGruSeqFwdLds, st>>>(a);
  PCHK(hipGetLastError());
  // heads + loss on every sample -> dh (FP32), head / log-std partial sums
  const int nh = (B + kHeadRows - 1) / kHeadRows;
  LossCoef lc{P->cfg.clip_eps, P->cfg.c_value, P->cfg.c_entropy, 1.0f / (float)B};
  k_heads<true, true><<<nh, kHeadThreads, 0, st>>>(params, o, P->hst, B, nullptr, nullptr, act, old_logp, adv, ret, P->rows,
                                          lc, nullptr, P->hpart, P->dh_head);
  PCHK(hipGetLastError());
  PCHK(launch_reduce_heads(P->hpart, nh, params, o, grads, loss, P->cfg.c_value, P->cfg.c_entropy, st));
  // backpropagation through time, and the GRU biases' column sums
  const PartRegions pr = part_regions(P);
  Reducer red;
  uint16_t* const dgi = P->dg;
  uint16_t* const dgh = P->dg + (int64_t)B * kGates;
  a.whh = P->whht; a.dh_head = P->dh_head; a.dgi = dgi; a.dgh = dgh; a.part = P->part + pr.gb;
  (rpl == 1 ? k_gru_seq_bwd<1>
            : rpl == 2 ? k_gru_seq_bwd<2> : k_gru_seq_bwd<4>)<<<tiles, kGruSeqThreads, kGruSeqBwdLds, st>>>(a);
  PCHK(hipGetLastError());
  red.add(P->part + pr.gb, (int)tiles, 2 * kGates,
          ReduceSegs{{kGates, kGates, 0, 0}, {0, 0, 0, 0}, {o.gbi, o.gbh, 0, 0}});
  // GRU weights: dW_ih = sum_s dgi[s] h1[s]^T, dW_hh = sum_s dgh[s] hp[s]^T
  PCHK(weight_grad(gemm_tn::Operands{dgi, kGates, kGates, P->h1, kHid, kHid, B}, kFc2Splits, P->part + pr.w2, o.gih, red,
                   st));
  PCHK(weight_grad(gemm_tn::Operands{dgh, kGates, kGates, P->hp_bf, kHid, kHid, B}, kFc2Splits, P->part + pr.whh, o.ghh,
                   red, st));
  // FC1 output gradient: dz1 = (dgi W_ih) * [h1 > 0]
  PCHK((gemm::run<128, 128, 64, 2, 2>(LdBF16K{dgi, kGates, B, kGates}, LdBF16K{P->wiht, kGates, kHid, kGates},
                                     EpiReluGradBF16{P->dz1, P->h1, kHid, kHid}, B, kHid, kGates, 1, st)));
  return backward_fc1_encoder(P, params, crop, P->rows, B, red, grads, st);
}

}  // extern "C"
