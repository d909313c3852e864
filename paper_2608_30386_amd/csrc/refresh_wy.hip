// Chunkwise WY-form refresh kernel on bf16 MFMA (gfx950), dk = dv = 128.
//
// Same recurrence as the per-column kernel (Sec. 3.1, Eq. 1 on S' = S^T):
//     S~ = Diag(exp(g_t)) S'_{t-1},   S'_t = S~ + beta_t k_t (v_t - S~^T k_t)^T.
// Unrolled over a chunk of C = 32 tokens with G_t = sum_{r<=t} g_r (per channel):
//     A_ts = beta_t sum_c k_tc k_sc exp(G_tc - G_sc)      (s < t)
//     T    = (I + A)^{-1},   T' = T Diag(beta)
//     U    = T' (V - K_G S')          K_G = k * exp(G)         (per-token deltas)
//     S'  <- Diag(exp(G_C)) S' + K_H^T U   K_H = k * exp(G_C - G)
// which is the per-token rule exactly, up to rounding.
//
// Work split: one 576-thread block per (request, head), one block per CU, its nine waves in
// three roles that work on three different chunks at a time:
//   state waves 0..3    own columns [32w, 32w + 32) of S' (128 x 32 fp32 = four 32x32 MFMA
//                       accumulator tiles, in VGPRs for the whole replay) and run the three
//                       chained contractions K_G S', T'(V - .), K_H^T U of chunk c;
//   factor waves 4..7   form chunk c + 2's decays, K_G, K_H and A from the gates and keys,
//                       32 channels each (A as one partial sum per wave);
//   solver wave 8       sums A of chunk c + 1, inverts I + A and leaves -T'.
// One barrier per chunk closes a step of this pipeline.  A block whose four waves run all of
// this in turn pays for the sum of the phases (11.5k cycles a chunk alone on its CU, 15.1k
// with a second block beside it); here a chunk costs the longest role, about 5.6k cycles.
//
// What bounds it: instruction issue.  A SIMD issues one VALU instruction in 4 cycles (8 for an
// exponential), a 32x32x16 MFMA holds the others back for about 10 of its 32, and a state
// wave's ~390 and a factor wave's ~345 VALU instructions a chunk (64 and 48 fewer when the
// decay is not applied, see below) fill 4.5k cycles of their SIMD; SIMD 0 also carries the
// solver (5.4k).  Hence the 32x32x16 tiles instead of 16x16x32,
// the split without dot products (wy_ops.h), and every operand staged in the order its reader
// loads it, 16 bytes per lane.  Waves of the same SIMD are served oldest first unless their
// priorities differ: the solver, which everything waits for, goes first, then the state waves.
//
// Measured (us; before: one 256-thread block per head, two per CU): fused Load of 16 requests x
// 32 heads, W = 1024: 225 -> 205; the plain refresh, W = 2048: 432 -> 387; of 5 requests, W = 777:
// 127 -> 67; fused Load of 1 request, W = 128: 30.2 -> 19.3.  With all 256 CUs busy the clock falls from
// 2.45 to 2.1 GHz, which is why the batches gain less.  One block per CU has nothing beside it
// during its first loads and last stores: the plain refresh of 32 requests x 32 heads, W = 16, takes
// 50 where two blocks per CU took 48.
//
// Precision.  The products run on bf16 MFMA with fp32 accumulation.  An fp32 operand x is
// split into x_hi = bf16(x) and x_lo = bf16(x - x_hi); a product is formed as a_lo b_hi +
// a_hi b_lo + a_hi b_hi, which keeps ~16 mantissa bits per term.  This is what lets an fp32
// state survive thousands of tokens within 2e-3 while running at the bf16 matrix-core rate.
// The diagonal blocks of T are fp32 throughout, block (1, 0) is formed by split products.
//
// Register-resident chaining.  The contraction index of an MFMA can be any bijection shared by
// A and B, so accumulators are fed straight back as B operands: lane l of a 32x32x16 product
// holds rows (i % 4) + 8 (i / 4) + 4 (l / 32), i < 16, of column l % 32, and registers 8s ..
// 8s + 7 are step s of the next contraction, whose A operand is stored in that order.  S',
// K_G S', V - K_G S' and U never leave registers.
//
// Decay factors.  exp(G_t - G_s) <= 1 for s <= t, but a factorised form needs
// exp(G_t - G_ref) exp(G_ref - G_s).  Fast path: when none of a factor wave's 32 channels passes
// 2^96 in the chunk, what the state lags behind included (see below; a test per wave, and
// realistic gates decay far less), the reference is where G starts: A = Diag(beta) strictly-lower(K_G Q^T) with K_G = k 2^G (which
// X needs anyway) and Q = k 2^{-G} <= 2^96 |k|, and K_H = Q 2^{G_C}: two exponentials per
// (token, channel).  Strong-decay path otherwise, for that wave's channels only: each 16x16
// tile of A takes a reference token of its own (8, 15 or 24), whose factors are bounded by
// exp(8 |g|max), and K_H its own exponentials.
//
// The state decays lazily, by groups of 32 channels: a group's running sums G start from the
// exponent its state still lags behind, K_H is then Q itself, and 2^G is multiplied into the
// group's rows (and into K_H) only after the chunk in which some |G| exceeds kLazy, a chunk on
// the strong-decay path, or the last one.  Channels that decay by 2^-30 a chunk, the fastest of
// a group at the serving shape, have it applied every second chunk (211.6 -> 205.7 us for the
// 16-request Load, 392.4 -> 383.8 for W = 2048, when it came in).
//
// Per-token log-gates are floored at -10 (a decay of 4.5e-5 per token instead of anything
// smaller), which keeps every factor below e^80 in fp32 and changes the state by at most 4.5e-5
// of its magnitude per floored token.
//
// Fused with the restore (FUSED = true), the initial state of a head is read from the
// packed checkpoint instead of the active state (kept rows from their packed position,
// omitted rows +0.0), and every row of the layer is written: kept rows copied bit for bit
// from the checkpoint by the state waves while the first chunk is being factored, omitted rows
// from the replay at the end.  A head with no omitted row is a plain copy.  The arithmetic is
// the unfused kernel's, so the result equals restore followed by refresh bit for bit.
//
// Inputs are read through raw buffer resources sized to one head's window, so tokens
// past the window load as zeros: k = v = 0, g = 0, beta = 0, an identity step.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "ckpt_layout.h"
#include "refresh_kernels.h"
#include "wy_ops.h"
#include "wy_roles.h"

namespace {

using namespace dasc_wy;

constexpr int C = 32;       // tokens per chunk
constexpr int D = kDim;     // dk = dv
constexpr float kGateFloor = -10.f;
// Fast path bound: |G| at the end of the chunk, the exponent carried into it included, at most
// kFastRange, so that k 2^G and k 2^{-G} stay normal fp32 (and their bf16 low parts too) for
// every token.
constexpr float kFastRange = 96.f;
// |log2| by which the state of a group of 32 channels may lag behind its decay: K_H is then Q as
// it is, at most 2^kLazy |k|, and the state's values stay below 2^kLazy times their own.
constexpr float kLazy = 40.f;
constexpr float kLog2e = 1.4426950408889634f;

constexpr int kStateWaves = 4;    // waves 0..3, 32 value columns each
constexpr int kFactorWaves = 4;   // waves 4..7
constexpr int kWaves = kStateWaves + kFactorWaves + 1;   // wave 8 solves
constexpr int kThreads = 64 * kWaves;

// LDS map (bytes).
constexpr int KG_BYTES = 8 * 2 * 1024;           // [step of 16 channels][hi/lo][lane][8 bf16]
constexpr int KH_HALF = 32 * 16 + 16;            // 32 channels x 8 bf16, padded
constexpr int KH_BYTES = 4 * 2 * 2 * 2 * KH_HALF;   // [32 channels][hi/lo][step][lane / 32][KH_HALF]
constexpr int AP_BYTES = 3 * 4 * 1024;           // [tile][factor wave][lane][4 f32]
constexpr int OFF_KG = 0;                        // 3 buffers
constexpr int OFF_KH = OFF_KG + 3 * KG_BYTES;    // 2 buffers
constexpr int OFF_AP = OFF_KH + 2 * KH_BYTES;    // 2 buffers
constexpr int OFF_TP = OFF_AP + 2 * AP_BYTES;    // 2 buffers
constexpr int OFF_GAM = OFF_TP + 2 * TP32_BYTES;   // f32 [3][D] 2^{G_C}
constexpr int OFF_FLAG = OFF_GAM + 3 * D * 4;    // int [3][4] is 2^{..} to be applied, by group of 32 channels
constexpr int OFF_TR = OFF_FLAG + 3 * 16;      // the solver's A, then T
constexpr int OFF_BETA = OFF_TR + 2 * T_BYTES;   // f32 [64] the solver's betas (twice)
constexpr int OFF_ROWS = OFF_BETA + 64 * 4;      // int64 [D] fused: checkpoint row table
constexpr int OFF_OMIT = OFF_ROWS + D * 8;       // u8 [D] row omitted (replayed)
constexpr int OFF_ANY = OFF_OMIT + D;            // int64 [2] fused: some_row of each half
constexpr int LDS_BYTES = OFF_ANY + 16;
static_assert(LDS_BYTES <= 160 * 1024, "one block per CU");

// Packed checkpoint of the fused variant (unused when FUSED is false).
using dasc::CkptView;

// Lane L of the row of 16 to every lane of the row (row_newbcast).
template <int L>
__device__ inline float row_bcast(float v) { return dpp_row<0x150 + L>(v); }

template <bool PER_CHANNEL, bool FUSED>
__global__ __launch_bounds__(kThreads) void refresh_wy_kernel(
    int head0, int H, int Hqk, int layer, int L, const int32_t* __restrict__ inv_row,
    float* __restrict__ states, int64_t n_pool, const int32_t* __restrict__ slot,
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, const float* __restrict__ g,
    const float* __restrict__ beta, int W, int init_zero, CkptView ck) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[LDS_BYTES];
  unsigned char* const sOmit = smem + OFF_OMIT;

  const int nh = head0 + int(blockIdx.x);
  const int n = nh / H;
  const int h = nh - n * H;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, r = lane & 15;

  // the head's row map and slots, loaded together
  const int64_t head_row = (int64_t(layer) * H + h) * D;
  const int32_t inv = tid < D ? inv_row[head_row + tid] : 0;
  const int64_t sl = slot[n];
  const int64_t cslot = FUSED ? ck.slot[n] : 0;

  const int hk = h / (H / Hqk);
  const uint16_t* kp = k + (int64_t(n) * Hqk + hk) * W * D;
  const uint16_t* vp = v + (int64_t(n) * H + h) * W * D;
  const float* gp = PER_CHANNEL ? g + (int64_t(n) * H + h) * W * D : g + (int64_t(n) * H + h) * W;
  const float* bp = beta + (int64_t(n) * H + h) * W;
  const int n_chunks = (W + C - 1) / C;
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};

  const bool factor_wave = w >= kStateWaves && w < kStateWaves + kFactorWaves;
  // Fused: where dense row c of this head sits in the checkpoint, as a float offset
  // (dasc::kOmitted for an omitted row, dasc::kNoRow for an index outside the packed rows,
  // which restores as +0.0).
  int64_t* sOff = reinterpret_cast<int64_t*>(smem + OFF_ROWS);
  int64_t* sAny = reinterpret_cast<int64_t*>(smem + OFF_ANY);
  if (tid < D) {
    sOmit[tid] = inv < 0;
    if (FUSED) {
      const int64_t o = dasc::ckpt_row_offset(inv, ck, cslot, D);
      sOff[tid] = o;
      sAny[w] = some_row(o);
    }
  }
  const bool any_omitted = __syncthreads_or(inv < 0);
  if (!FUSED && !any_omitted) return;
  if (sl < 0 || sl >= n_pool) return;
  if (FUSED && (cslot < 0 || cslot >= ck.n_slots)) return;
  float* S_head = states + (sl * L * H * D + head_row) * D;
  if (FUSED && !any_omitted) {   // nothing to replay: a plain copy of the head
    copy_head(S_head, ck.ckpt, sOff, tid, kThreads);
    return;
  }

  if (factor_wave) {
    // ---- factor waves ---------------------------------------------------------------------
    const int kk = w - kStateWaves;
    const int c4 = 32 * kk + 16 * (q >> 1) + 4 * (q & 1);   // channels c4 + i and c4 + 8 + i
    const __amdgpu_buffer_rsrc_t rk = rsrc(kp, W * D * 2);
    const __amdgpu_buffer_rsrc_t rg = rsrc(gp, PER_CHANNEL ? W * D * 4 : W * 4);
    f32x4 graw[2][2];
    uint2 kraw[2][2];
    auto fetch = [&](int c0) {
#pragma unroll
      for (int mu = 0; mu < 2; ++mu)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
          kraw[mu][hf] = __builtin_bit_cast(
              uint2, __builtin_amdgcn_raw_buffer_load_b64(rk, ((16 * mu + r) * D + c4 + 8 * hf) * 2,
                                                          c0 * D * 2, 0));
#pragma unroll
      for (int mu = 0; mu < 2; ++mu)
        if (PER_CHANNEL) {
#pragma unroll
          for (int hf = 0; hf < 2; ++hf)
            graw[mu][hf] = ldf4(rg, ((16 * mu + r) * D + c4 + 8 * hf) * 4, c0 * D * 4);
        } else {
          const float x = ldf(rg, (16 * mu + r) * 4, c0 * 4);
          graw[mu][0] = graw[mu][1] = f32x4{x, x, x, x};
        }
    };
    fetch(0);
    uint32_t khh[8], khl[8];
    auto store_kh = [&](int c) {
      unsigned char* b = smem + OFF_KH + (c & 1) * KH_BYTES + kk * (2 * 2 * 2 * KH_HALF) +
                         (r >> 2) * KH_HALF + (c4 & 31) * 16 + (r & 3) * 4;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        unsigned char* o = b + ((e & 3) + 2 * (e & 4)) * 16;
        *reinterpret_cast<uint32_t*>(o) = khh[e];
        *reinterpret_cast<uint32_t*>(o + 4 * KH_HALF) = khl[e];
      }
    };
    // log2 of what the state still has to be multiplied by, per channel, held in lane r = 0 of
    // each row of 16 (0 in the others), where the chunk's running sums start
    float carry[8] = {};
    const uint32_t first = r == 0 ? ~0u : 0u;
    auto stage = [&](int c, int kg_buf) {
      float G[2][8], kf[2][8];
#pragma unroll
      for (int mu = 0; mu < 2; ++mu)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          // (med3 with +inf is the floor in one instruction; fmaxf would first quiet a NaN)
          G[mu][e] = __builtin_amdgcn_fmed3f(graw[mu][e >> 2][e & 3], kGateFloor, __builtin_inff()) * kLog2e;
          const uint32_t kw = (e & 2) ? kraw[mu][e >> 2].y : kraw[mu][e >> 2].x;
          kf[mu][e] = __uint_as_float((e & 1) ? (kw & 0xFFFF0000u) : (kw << 16));
        }
      fetch((c + 1) * C);
      // running sums over the chunk's tokens, from the carried exponent on
#pragma unroll
      for (int e = 0; e < 8; ++e) G[0][e] += carry[e];
#pragma unroll
      for (int mu = 0; mu < 2; ++mu) {
#pragma unroll
        for (int e = 0; e < 8; ++e) G[mu][e] += dpp_row<0x111>(G[mu][e]);
#pragma unroll
        for (int e = 0; e < 8; ++e) G[mu][e] += dpp_row<0x112>(G[mu][e]);
#pragma unroll
        for (int e = 0; e < 8; ++e) G[mu][e] += dpp_row<0x114>(G[mu][e]);
#pragma unroll
        for (int e = 0; e < 8; ++e) G[mu][e] += dpp_row<0x118>(G[mu][e]);
      }
      float gmax = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        G[1][e] += row_bcast<15>(G[0][e]);
        gmax = fmaxf(gmax, fabsf(G[1][e]));
      }
      const bool fast = __all(gmax <= kFastRange);
      const bool apply = !__all(gmax <= kLazy) || c == n_chunks - 1;   // 2^G goes into the state
      const uint32_t keep = apply ? 0u : first;
#pragma unroll
      for (int e = 0; e < 8; ++e)   // row_ror:1: lane 0 takes the chunk's total from lane 15
        carry[e] = __uint_as_float(__float_as_uint(dpp_row<0x121>(G[1][e])) & keep);
      if (lane == 0) reinterpret_cast<int*>(smem + OFF_FLAG)[4 * kg_buf + kk] = apply;
      f32x4* const ap = reinterpret_cast<f32x4*>(smem + OFF_AP + (c & 1) * AP_BYTES + kk * 1024) + lane;
      bf16x8 ah[2], al[2];
      float eg[2][8];
#pragma unroll
      for (int mu = 0; mu < 2; ++mu) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          eg[mu][e] = ex2(G[mu][e]);
          x[e] = kf[mu][e] * eg[mu][e];
        }
        split8(x, ah[mu], al[mu]);
        bf16x8* o = reinterpret_cast<bf16x8*>(smem + OFF_KG + kg_buf * KG_BYTES + (2 * kk + (q >> 1)) * 2048) + 16 * mu + r + 32 * (q & 1);
        o[0] = ah[mu];
        o[64] = al[mu];
      }
      if (r == 15) {
        float* o = reinterpret_cast<float*>(smem + OFF_GAM) + kg_buf * D + c4;
        *reinterpret_cast<f32x4*>(o) = f32x4{eg[1][0], eg[1][1], eg[1][2], eg[1][3]};
        *reinterpret_cast<f32x4*>(o + 8) = f32x4{eg[1][4], eg[1][5], eg[1][6], eg[1][7]};
      }
      if (fast) {
        bf16x8 bh[2], bl[2];
        float qf[2][8];
#pragma unroll
        for (int mu = 0; mu < 2; ++mu) {
#pragma unroll
          for (int e = 0; e < 8; ++e) qf[mu][e] = kf[mu][e] * ex2(-G[mu][e]);
          split8(qf[mu], bh[mu], bl[mu]);
        }
        ap[0] = mma3(ah[0], al[0], bh[0], bl[0], zero4);
        ap[256] = mma3(ah[1], al[1], bh[0], bl[0], zero4);
        ap[512] = mma3(ah[1], al[1], bh[1], bl[1], zero4);
        if (apply) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float gam = row_bcast<15>(eg[1][e]);
            split2(qf[0][e] * gam, qf[1][e] * gam, khh[e], khl[e]);
          }
        } else {   // K_H is Q: its words of two channels dealt out to words of two tokens
          const uint4 h0 = __builtin_bit_cast(uint4, bh[0]), h1 = __builtin_bit_cast(uint4, bh[1]);
          const uint4 l0 = __builtin_bit_cast(uint4, bl[0]), l1 = __builtin_bit_cast(uint4, bl[1]);
          const uint32_t hw[2][4] = {{h0.x, h0.y, h0.z, h0.w}, {h1.x, h1.y, h1.z, h1.w}};
          const uint32_t lw[2][4] = {{l0.x, l0.y, l0.z, l0.w}, {l1.x, l1.y, l1.z, l1.w}};
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
            khh[e] = __builtin_amdgcn_perm(hw[1][e >> 1], hw[0][e >> 1], sel);
            khl[e] = __builtin_amdgcn_perm(lw[1][e >> 1], lw[0][e >> 1], sel);
          }
        }
      } else {
#pragma unroll
        for (int tile = 0; tile < 3; ++tile) {
          const int ti = tile == 0 ? 0 : 1, si = tile == 2 ? 1 : 0;
          float fa[8], fb[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float gf = tile == 0 ? row_bcast<8>(G[0][e])
                           : tile == 1 ? row_bcast<15>(G[0][e]) : row_bcast<8>(G[1][e]);
            fa[e] = kf[ti][e] * ex2(G[ti][e] - gf);
            fb[e] = kf[si][e] * ex2(gf - G[si][e]);
          }
          bf16x8 xh, xl, yh, yl;
          split8(fa, xh, xl);
          split8(fb, yh, yl);
          ap[256 * tile] = mma3(xh, xl, yh, yl, zero4);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float gc = row_bcast<15>(G[1][e]);
          split2(kf[0][e] * ex2(gc - G[0][e]), kf[1][e] * ex2(gc - G[1][e]), khh[e], khl[e]);
        }
      }
    };
    int kg_buf = 0;
    for (int p = -2; p < n_chunks; ++p) {
      if (p >= -1 && p + 1 < n_chunks) store_kh(p + 1);
      if (p + 2 < n_chunks) stage(p + 2, kg_buf);
      kg_buf = kg_buf == 2 ? 0 : kg_buf + 1;
      __syncthreads();
    }
    return;
  }

  if (w == kWaves - 1) {
    __builtin_amdgcn_s_setprio(3);
    // ---- solver wave ------------------------------------------------------------------------
    const __amdgpu_buffer_rsrc_t rb = rsrc(bp, W * 4);
    float* const sB = reinterpret_cast<float*>(smem + OFF_BETA);
    for (int b = 0; b < 2; ++b) clear_tp(smem + OFF_TP + b * TP32_BYTES, lane);
    float braw = ldf(rb, (lane & (C - 1)) * 4, 0);
    float* const tr = reinterpret_cast<float*>(smem + OFF_TR);
    for (int p = -2; p < n_chunks; ++p) {
      const int c = p + 1;
      if (c >= 0 && c < n_chunks) {
        sB[lane] = braw;
        braw = ldf(rb, (lane & (C - 1)) * 4, (c + 1) * C * 4);
        const f32x4* ap = reinterpret_cast<const f32x4*>(smem + OFF_AP + (c & 1) * AP_BYTES) + lane;
        f32x4 acc[3];
#pragma unroll
        for (int tile = 0; tile < 3; ++tile)
          acc[tile] = (ap[256 * tile] + ap[256 * tile + 64]) + (ap[256 * tile + 128] + ap[256 * tile + 192]);
        wave_lds_sync();
        const f32x4 b0 = *reinterpret_cast<const f32x4*>(sB + 4 * q);
        const f32x4 b1 = *reinterpret_cast<const f32x4*>(sB + 16 + 4 * q);
        const f32x4 a10 = acc[1] * b1;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          tr[(4 * q + i) * ST + r] = acc[0][i] * b0[i];
          tr[(16 + 4 * q + i) * ST + r] = acc[2][i] * b1[i];
        }
        wave_lds_sync();
        solve_chunk<false>(tr, a10, sB, b0, tr + 32 * ST, smem + OFF_TP + (c & 1) * TP32_BYTES, q, r);
      }
      __syncthreads();
    }
    return;
  }

  __builtin_amdgcn_s_setprio(1);
  // ---- state waves ----------------------------------------------------------------------------
  const __amdgpu_buffer_rsrc_t rv = rsrc(vp, W * D * 2);
  const int hi = lane >> 5, col = 32 * w + (lane & 31);
  // this lane's value column at tokens (i % 4) + 8 (i / 4) + 4 hi
  uint32_t vreg[16];
  auto fetch_v = [&](int c0) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      vreg[i] = uint16_t(__builtin_amdgcn_raw_buffer_load_b16(
          rv, (((i & 3) + 8 * (i >> 2) + 4 * hi) * D + col) * 2, c0 * D * 2, 0));
  };
  fetch_v(0);
  // S'[c][col] for c = 32 mt + (i % 4) + 8 (i / 4) + 4 hi
  f32x16 S[4] = {};
  const int64_t any = FUSED ? std::max(sAny[0], sAny[1]) : 0;
  if (!init_zero) load_state<FUSED>(S, S_head, ck.ckpt, sOff, any, col, hi);
  __syncthreads();
  // (kept rows are written while the first chunk is being solved)
  if (FUSED) copy_kept_rows<64 * kStateWaves>(S_head, ck.ckpt, sOff, any, tid);
  __syncthreads();

  struct Frag { bf16x8 h, l; };
  auto load_kg = [&](int buf, int j) {
    const bf16x8* p = reinterpret_cast<const bf16x8*>(smem + OFF_KG + buf * KG_BYTES + j * 2048) + lane;
    return Frag{p[0], p[64]};
  };
  auto split_s = [&](int j) {   // S' rows 16 j + ... in the order of K_G's step j
    Frag f;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = S[j >> 1][8 * (j & 1) + e];
    split8(x, f.h, f.l);
    return f;
  };

  Frag gf = load_kg(0, 0), sf = split_s(0);
  int kg_buf = 0;
  for (int c = 0; c < n_chunks; ++c) {
    const bf16x8* tp = reinterpret_cast<const bf16x8*>(smem + OFF_TP + (c & 1) * TP32_BYTES) + lane;
    const float* gamp = reinterpret_cast<const float*>(smem + OFF_GAM) + kg_buf * D + 4 * hi;
    const unsigned char* kh = smem + OFF_KH + (c & 1) * KH_BYTES + hi * KH_HALF + (lane & 31) * 16;
    auto load_kh = [&](int mt, int s) {
      const unsigned char* p = kh + mt * (2 * 2 * 2 * KH_HALF) + s * (2 * KH_HALF);
      return Frag{*reinterpret_cast<const bf16x8*>(p), *reinterpret_cast<const bf16x8*>(p + 4 * KH_HALF)};
    };
    const int4 fl = *reinterpret_cast<const int4*>(smem + OFF_FLAG + 16 * kg_buf);
    const int flag[4] = {__builtin_amdgcn_readfirstlane(fl.x), __builtin_amdgcn_readfirstlane(fl.y),
                         __builtin_amdgcn_readfirstlane(fl.z), __builtin_amdgcn_readfirstlane(fl.w)};
    // ---- X = K_G S' on this wave's columns (rows t, contraction over channels) ------------
    f32x16 X = {};
    Frag tf[2], hf[2];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      Frag gn, sn;
      if (j < 7) {
        gn = load_kg(kg_buf, j + 1);
        sn = split_s(j + 1);
      } else {
#pragma unroll
        for (int s = 0; s < 2; ++s) tf[s] = Frag{tp[128 * s], tp[128 * s + 64]};
      }
      X = mmb3(gf.h, gf.l, sf.h, sf.l, X);
      __builtin_amdgcn_sched_barrier(0);
      gf = gn;
      sf = sn;
    }

    // ---- U = (-T')(X - V): the difference stays in registers as the B operand ------
    f32x16 U = {};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = X[8 * s + e] - __uint_as_float(vreg[8 * s + e] << 16);
      Frag y;
      split8(x, y.h, y.l);
      U = mmb3(tf[s].h, tf[s].l, y.h, y.l, U);
    }
    fetch_v((c + 1) * C);   // the next chunk's values (zeros past the window)
#pragma unroll
    for (int s = 0; s < 2; ++s) hf[s] = load_kh(0, s);

    // ---- S' <- Diag(exp(G_C)) S' + K_H^T U ----------------------------------------------
    Frag uf[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = U[4 * s + (e >> 1) + 8 * (e & 1)];   // tokens t, 16 + t in turn
      split8(x, uf[s].h, uf[s].l);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int kg_next = kg_buf == 2 ? 0 : kg_buf + 1;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      Frag hn[2];
      if (mt < 3) {
#pragma unroll
        for (int s = 0; s < 2; ++s) hn[s] = load_kh(mt + 1, s);
      } else {
        gf = load_kg(kg_next, 0);
      }
      if (flag[mt]) {
#pragma unroll
        for (int gr = 0; gr < 4; ++gr) {
          const f32x4 gam = *reinterpret_cast<const f32x4*>(gamp + 32 * mt + 8 * gr);
#pragma unroll
          for (int i = 0; i < 4; ++i) S[mt][4 * gr + i] *= gam[i];
        }
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) S[mt] = mmb3(hf[s].h, hf[s].l, uf[s].h, uf[s].l, S[mt]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 2; ++s) hf[s] = hn[s];
    }
    kg_buf = kg_next;
    sf = split_s(0);
    __syncthreads();
  }

  store_state(S, S_head, sOmit, col, hi);
}

}  // namespace

namespace dasc {

bool refresh_wy_supported(int dk, int dv) { return dk == D && dv == D; }

template <bool PER_CHANNEL, bool FUSED>
static void launch(int n_req, int H, int Hqk, int layer, int L, const int32_t* inv_row, float* states,
                   int64_t n_pool, const int32_t* slot, const uint16_t* k, const uint16_t* v,
                   const float* g, const float* beta, int W, int init_zero, const CkptView& ck,
                   hipStream_t st) {
  const unsigned heads = unsigned(n_req) * unsigned(H);
  for (unsigned h0 = 0; h0 < heads; h0 += kWyHeadsPerLaunch) {
    const dim3 grid(std::min(heads - h0, kWyHeadsPerLaunch)), block(kThreads);
    hipLaunchKernelGGL((refresh_wy_kernel<PER_CHANNEL, FUSED>), grid, block, 0, st, int(h0), H, Hqk, layer,
                       L, inv_row, states, n_pool, slot, k, v, g, beta, W, init_zero, ck);
  }
}

void launch_refresh_wy(bool per_channel, int n_req, int H, int Hqk, int layer, int L,
                       const int32_t* inv_row, float* states, int64_t n_pool, const int32_t* slot,
                       const uint16_t* k, const uint16_t* v, const float* g, const float* beta,
                       int W, int init_zero, hipStream_t st) {
  const auto f = per_channel ? launch<true, false> : launch<false, false>;
  f(n_req, H, Hqk, layer, L, inv_row, states, n_pool, slot, k, v, g, beta, W, init_zero,
    CkptView{nullptr, 1, 1, 0, nullptr}, st);
}

void launch_restore_refresh_wy(int n_req, int H, int Hqk, int layer, int L, const float* ckpt,
                               int64_t n_ckpt_slots, const int32_t* ck_slot,
                               int64_t slice_rows, int64_t n_rows, const int32_t* inv_row,
                               float* states, int64_t n_pool, const int32_t* slot,
                               const uint16_t* k, const uint16_t* v, const float* g,
                               const float* beta, int W, int init_zero, hipStream_t st) {
  launch<true, true>(n_req, H, Hqk, layer, L, inv_row, states, n_pool, slot, k, v, g, beta, W, init_zero,
                     CkptView{ckpt, n_ckpt_slots, slice_rows, n_rows, ck_slot}, st);
}

}  // namespace dasc
