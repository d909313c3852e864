// Chunkwise WY-form refresh for GDN heads (one scalar gate per token), dk = dv = 128,
// on bf16 MFMA (gfx950).
//
// Same recurrence and chunk algebra as the channel-wise kernel (Sec. 3.1, Eq. 1 on
// S' = S^T, chunks of C = 32 tokens, G_t = sum_{r<=t} g_r in log2 units), but with a
// scalar decay per token every decay factor leaves the contractions:
//     A_ts = beta_t (K K^T)_ts 2^{G_t - G_s}           (s < t)
//     T'   = (I + A)^{-1} Diag(beta)
//     X    = K_G S' = Diag(2^{G_t}) (K S')
//     S'  <- 2^{G_C} S' + K^T (Diag(2^{G_C - G_t}) U),  U = T'(V - X)
// Keys are bf16, so K is an exact MFMA operand: K K^T takes one bf16 pass (the products
// are exact in fp32) and K S', K^T U take two (state and update split into bf16 hi + lo)
// instead of three.
//
// The state decays lazily: it is held as S' = 2^c S^ with one exponent c per head, X is scaled
// by 2^{c + G_t} and U by 2^{-(c + G_t)}, and only when |c| would exceed kLazy, and after the last
// chunk, is 2^c multiplied into the state (U then takes 2^{G_C - G_t}, at most 1, as above).
// Gates that decay by 2^-4 a chunk cost a lane's 32 multiplications every fifth chunk.
//
// Work split, as in the channel-wise kernel: eight state waves of 16 value columns each on
// chunk c, one factor wave that forms A and lays out the keys of chunk c + 2, one solver wave
// that turns chunk c + 1's A into -T'; one barrier per chunk.  Two layouts: a block per head
// with all eight state waves, or two blocks per head with four each (and a factor and a solver
// wave of their own), chosen by kSplitHeads below.  ORDER: the refreshed heads first (kOrderHeads).
//
// What bounds it: a SIMD's waves for one chunk.  Two state waves alone on their SIMD take 2.9k
// cycles; with the solver wave beside them (the factor and solver waves go first) 3.5k, and the
// barrier makes it 3.8k.  With two blocks per head a SIMD has one state wave and at most one
// other: about 3k.  State waves of 32 columns on 32x32x16 tiles, four per head, issue less but
// take 4k a chunk (one wave's own chain).
//
// Measured (us; before: a factor launch for all chunks, then a recurrence launch of two blocks
// per head reading -T' back from memory): fused Load of one layer, 8 requests x 20 heads of 32,
// W = 1024: 80.5 -> 59.9; refresh of 3 requests, W = 517: 42.4 -> 28.0; 1 request of 4 heads,
// W = 2048: 106 -> 84.  Where more heads are refreshed than there are CUs the second round is
// nearly empty, and a long window loses up to 9% against the two launches, whose half-head blocks
// shared CUs (W = 1024: 13 requests 105 -> 114, 14 107 -> 114, 16 111 -> 115; W = 256: 16 44.5 -> 41; 24
// requests, W = 1024: 185 -> 171).
//
// Precision.  T = (I + A)^{-1} is formed in fp32 throughout, block (1, 0) on fp32 MFMA, and U's rows
// are scaled in fp32; what the products read of T is -T', split into bf16 hi + lo.  Scaling the
// rows of T' before they are split instead saves a state wave eight multiplications a chunk (2% of
// the 8-request refresh) and loses the entries that bf16 holds exactly, such as a diagonal of
// betas of 0.5: 4.3e-6 of the state's norm instead of 3.7e-6 with independent keys.
//
// Register chaining, operand splitting and order, and the buffer-resource loads (tokens past
// the window read as zeros: identity steps) are as in the channel-wise kernel; per-token
// log-gates are floored at -10 in the same way.

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
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLazy = 16.f;   // |log2| a state may lag behind: its values stay below 2^16 |S'|


// LDS map (bytes).
constexpr int K_BYTES = 4 * 2 * 1024;            // [step of 32 channels][row tile][lane][8 bf16]
constexpr int KT_ROW = 16 * 16 + 16;             // 16 channels x 8 bf16, padded
constexpr int KT_BYTES = 8 * 4 * KT_ROW;         // [16 channels][lane / 16][KT_ROW]
constexpr int A_BYTES = T_BYTES + 1024;          // diagonal blocks, then block (1, 0) by lane
constexpr int OFF_K = 0;                         // 3 buffers
constexpr int OFF_KT = OFF_K + 3 * K_BYTES;      // 3 buffers
constexpr int OFF_A = OFF_KT + 3 * KT_BYTES;     // 2 buffers
constexpr int OFF_TP = OFF_A + 2 * A_BYTES;      // 2 buffers
constexpr int OFF_EG = OFF_TP + 2 * TP16_BYTES;    // f32 [3][C] 2^{c + G_t}
constexpr int OFF_GAM = OFF_EG + 3 * C * 4;      // f32 [4]    what the state is multiplied by
constexpr int OFF_EU = OFF_GAM + 4 * 4;          // f32 [3][C] the scale of U's rows
constexpr int OFF_B = OFF_EU + 3 * C * 4;        // f32 [2][C] beta
constexpr int OFF_G = OFF_B + 2 * C * 4;         // f32 [C]    G_t (factor wave)
constexpr int OFF_T = OFF_G + C * 4;             // solver scratch
constexpr int OFF_ROWS = OFF_T + T_BYTES;        // int64 [D] fused: checkpoint row table
constexpr int OFF_OMIT = OFF_ROWS + D * 8;       // u8 [D] row omitted (replayed)
constexpr int OFF_ANY = OFF_OMIT + D;            // int64 [2] fused: some_row of each half
constexpr int LDS_BYTES = OFF_ANY + 16;
static_assert(OFF_ROWS % 16 == 0 && OFF_T % 16 == 0, "alignment");
static_assert(LDS_BYTES <= 81920, "two blocks of six waves per CU");

template <int CTRL, int ROW_MASK>
__device__ inline float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                                               ROW_MASK, 0xF, true));
}

// Inclusive prefix sum over lanes 0..31: shifts by 1, 2, 4, 8 within each row of 16
// lanes, then row 1 adds the last lane of row 0 (row_bcast:15).  No LDS round trips.
__device__ inline float scan32(float x) {
  x += dpp<0x111, 0xF>(x);   // row_shr:1
  x += dpp<0x112, 0xF>(x);   // row_shr:2
  x += dpp<0x114, 0xF>(x);   // row_shr:4
  x += dpp<0x118, 0xF>(x);   // row_shr:8
  x += dpp<0x142, 0xA>(x);   // row_bcast:15 into rows 1 and 3
  return x;
}

// Blocks are dealt to the eight XCDs in turn (block b starts on XCD b mod 8).  Renumber
// them so that each XCD takes a contiguous range of (request, head) items: the blocks that
// read one key head then sit on the same XCD and share its L2.  A bijection whenever the
// grid is a multiple of 8.
__device__ inline int xcd_major(int b, int n_blocks) {
  if (n_blocks & 7) return b;
  return (b & 7) * (n_blocks >> 3) + (b >> 3);
}

// The r-th set bit of a mask that every lane holds.
__device__ inline int nth_set(uint64_t mask, int lane, int r) {
  const int below = __builtin_amdgcn_mbcnt_hi(uint32_t(mask >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(mask), 0));
  return __builtin_ctzll(__ballot(((mask >> lane) & 1) && below == r));
}

// The (request, head) item of block b when the refreshed heads go first, in an XCD-major order of
// their own, and the heads that the refresh leaves alone last.  inv: the layer's row map; a head's
// first row stands for it here, which decides an order and nothing else.  For H <= 64.
__device__ inline int refreshed_first(int b, int n_blocks, int H, const int32_t* inv, int lane) {
  const uint64_t mask = __ballot(lane < H && inv[(lane < H ? lane : 0) * D] < 0);
  const int cnt = __builtin_popcountll(mask), n_ref = n_blocks / H * cnt;
  if (b < n_ref) {
    const int x = b & 7, i = x * (n_ref >> 3) + min(x, n_ref & 7) + (b >> 3);
    return i / cnt * H + nth_set(mask, lane, i % cnt);
  }
  const int i = b - n_ref, kept = H - cnt;
  return i / kept * H + nth_set(~mask & (~uint64_t(0) >> (64 - H)), lane, i % kept);
}

// Up to kSplitHeads heads a launch takes two blocks per head: all of them run at once on the 256 CUs,
// each with the shorter chunk.  Beyond it they may share CUs or wait for one: us, split and whole,
// requests of 32 heads, 20 of them refreshed, W = 1024: 4 requests 49.9 and 59.0, 5 49.9 and 58.5, 6
// 90.6 and 59.5, 8 91.4 and 59.9.  (The line counts heads, since the host does not see which are
// refreshed; at 5 requests with as many kept it gives 9 us away.)
constexpr unsigned kSplitHeads = 128;
// From 257 heads, more than there are CUs, up to kOrderHeads a launch takes the refreshed heads first.
// In list order the heads that exit at once leave CUs idle while refreshed ones queue for another
// shader engine's, and the call takes two rounds even where the refreshed heads alone would fit
// the chip: us, list order -> refreshed first, same heads, W = 1024: 9 requests 60 -> 62, 10 60 or
// 110 -> 62 (by the heads kept), 11 110 -> 62, 12 111 -> 62; W = 16: 12 17.1 -> 12.2.
// Where they do not fit, finding the order only delays each block (13 to 16 requests: by 1% at W =
// 1024, 4% at W = 256, 6% at W = 16), so the line stands at 1.5 heads per CU, which fits whenever a
// third of the heads is kept.
constexpr unsigned kOrderHeads = 384;

// FUSED: the initial state comes from the packed checkpoint (kept rows from their packed
// position, written back to the pool at once; omitted rows +0.0) and every row of the
// layer is written, as the channel-wise kernel's fused variant does.
template <bool FUSED, int NS, bool ORDER>
__global__ __launch_bounds__(64 * (NS + 2)) void refresh_wy_gdn_kernel(
    int head0, int H, int Hqk, int layer, int L, const int32_t* __restrict__ inv_row,
    float* __restrict__ states, int64_t n_pool, const int32_t* __restrict__ slot,
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, const float* __restrict__ g,
    const float* __restrict__ beta, int W, int init_zero, dasc::CkptView ck) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[LDS_BYTES];
  constexpr int kThreads = 64 * (NS + 2);
  constexpr int kParts = 8 / NS;   // blocks per head
  unsigned char* const sOmit = smem + OFF_OMIT;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int item = ORDER ? refreshed_first(blockIdx.x, gridDim.x, H, inv_row + int64_t(layer) * H * D, lane)
                         : xcd_major(blockIdx.x, gridDim.x);
  const int part = item % kParts;
  const int nh = head0 + item / kParts;
  const int n = nh / H;
  const int h = nh - n * H;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, r = lane & 15;

  // the head's row map and slots, loaded together
  const int64_t head_row = (int64_t(layer) * H + h) * D;
  const int32_t inv = tid < D ? inv_row[head_row + tid] : 0;
  const int64_t sl = slot[n];
  const int64_t cslot = FUSED ? ck.slot[n] : 0;

  // Fused: the head's checkpoint row table (float offsets, or dasc::kOmitted / dasc::kNoRow)
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
    copy_head(S_head, ck.ckpt, sOff, part * kThreads + tid, kParts * kThreads);
    return;
  }

  const int hk = h / (H / Hqk);
  const int n_chunks = (W + C - 1) / C;

  if (w == NS) {
    __builtin_amdgcn_s_setprio(2);
    // ---- factor wave ------------------------------------------------------------------------
    // Lane (q, r) holds tokens r and 16 + r at channels 32 kk + 4q + i and 32 kk + 16 + 4q + i.
    const __amdgpu_buffer_rsrc_t rk = rsrc(k + (int64_t(n) * Hqk + hk) * W * D, W * D * 2);
    const __amdgpu_buffer_rsrc_t rg = rsrc(g + (int64_t(n) * H + h) * W, W * 4);
    const __amdgpu_buffer_rsrc_t rb = rsrc(beta + (int64_t(n) * H + h) * W, W * 4);
    uint2 kraw[4][2][2];
    float graw, braw;
    auto fetch = [&](int c0) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int mu = 0; mu < 2; ++mu)
#pragma unroll
          for (int hf = 0; hf < 2; ++hf)
            kraw[kk][mu][hf] = __builtin_bit_cast(
                uint2, __builtin_amdgcn_raw_buffer_load_b64(
                           rk, ((16 * mu + r) * D + 32 * kk + 4 * q + 16 * hf) * 2, c0 * D * 2, 0));
      graw = ldf(rg, (lane & (C - 1)) * 4, c0 * 4);
      braw = ldf(rb, (lane & (C - 1)) * 4, c0 * 4);
    };
    float* const sG = reinterpret_cast<float*>(smem + OFF_G);
    float carry = 0.f;   // c: log2 of what the state still has to be multiplied by
    auto stage = [&](int c, int buf) {
      f32x4 acc[3] = {};
      uint4* const kb = reinterpret_cast<uint4*>(smem + OFF_K + buf * K_BYTES) + lane;
      unsigned char* const kt = smem + OFF_KT + buf * KT_BYTES + (r >> 2) * KT_ROW + 64 * q + (r & 3) * 4;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        bf16x8 f[2];
#pragma unroll
        for (int mu = 0; mu < 2; ++mu) {
          const uint4 x = make_uint4(kraw[kk][mu][0].x, kraw[kk][mu][0].y, kraw[kk][mu][1].x, kraw[kk][mu][1].y);
          f[mu] = __builtin_bit_cast(bf16x8, x);
          kb[(2 * kk + mu) * 64] = x;
        }
        acc[0] = mma(f[0], f[0], acc[0]);
        acc[1] = mma(f[1], f[0], acc[1]);
        acc[2] = mma(f[1], f[1], acc[2]);
        // keys transposed: tokens (r, 16 + r) of a channel in one word
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint2 x0 = kraw[kk][0][e >> 2], x1 = kraw[kk][1][e >> 2];
          *reinterpret_cast<uint32_t*>(kt + (2 * kk + (e >> 2)) * (4 * KT_ROW) + (e & 3) * 16) =
              __builtin_amdgcn_perm((e & 2) ? x1.y : x1.x, (e & 2) ? x0.y : x0.x,
                                    (e & 1) ? 0x07060302u : 0x05040100u);
        }
      }
      const float g_c = graw, b_c = braw;
      fetch((c + 1) * C);   // (issued here: a chunk's time before it is used)
      const float gl = scan32(lane < C ? __builtin_amdgcn_fmed3f(g_c, kGateFloor, __builtin_inff()) * kLog2e : 0.f);
      const float total = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, gl), C - 1));
      const float end = carry + total;
      const bool apply = fabsf(end) > kLazy || c == n_chunks - 1;   // 2^end goes into the state
      const float gc = carry + gl;
      float* const sB = reinterpret_cast<float*>(smem + OFF_B) + (c & 1) * C;
      if (lane < C) {
        sG[lane] = gl;
        sB[lane] = b_c;
        (reinterpret_cast<float*>(smem + OFF_EG) + buf * C)[lane] = ex2(gc);
        (reinterpret_cast<float*>(smem + OFF_EU) + buf * C)[lane] = ex2((apply ? end : 0.f) - gc);
      }
      if (lane == 0) reinterpret_cast<float*>(smem + OFF_GAM)[buf] = apply ? ex2(end) : 1.f;
      carry = apply ? 0.f : end;
      wave_lds_sync();
      // A = Diag(beta) K K^T scaled by 2^{G_t - G_s} (the solver uses what is below the diagonal)
      const f32x4 g0 = *reinterpret_cast<const f32x4*>(sG + 4 * q), g1 = *reinterpret_cast<const f32x4*>(sG + 16 + 4 * q);
      const f32x4 b0 = *reinterpret_cast<const f32x4*>(sB + 4 * q), b1 = *reinterpret_cast<const f32x4*>(sB + 16 + 4 * q);
      const float gs0 = sG[r], gs1 = sG[16 + r];
      float* const sA = reinterpret_cast<float*>(smem + OFF_A + (c & 1) * A_BYTES);
      f32x4 a10;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sA[(4 * q + i) * ST + r] = acc[0][i] * b0[i] * ex2(g0[i] - gs0);
        sA[(16 + 4 * q + i) * ST + r] = acc[2][i] * b1[i] * ex2(g1[i] - gs1);
        a10[i] = acc[1][i] * b1[i] * ex2(g1[i] - gs0);
      }
      reinterpret_cast<f32x4*>(sA + 32 * ST)[lane] = a10;
    };
    fetch(0);
    int buf = 0;
    for (int p = -2; p < n_chunks; ++p) {
      if (p + 2 < n_chunks) stage(p + 2, buf);
      buf = buf == 2 ? 0 : buf + 1;
      __syncthreads();
    }
    return;
  }

  if (w == NS + 1) {
    __builtin_amdgcn_s_setprio(2);
    // ---- solver wave --------------------------------------------------------------------------
    for (int p = -2; p < n_chunks; ++p) {
      const int c = p + 1, par = c & 1;
      if (c >= 0 && c < n_chunks) {
        const float* sA = reinterpret_cast<const float*>(smem + OFF_A + par * A_BYTES);
        const float* sB = reinterpret_cast<const float*>(smem + OFF_B) + par * C;
        solve_chunk<true>(sA, reinterpret_cast<const f32x4*>(sA + 32 * ST)[lane], sB,
                          *reinterpret_cast<const f32x4*>(sB + 4 * q),
                          reinterpret_cast<float*>(smem + OFF_T), smem + OFF_TP + par * TP16_BYTES, q, r);
      }
      __syncthreads();
    }
    return;
  }

  // ---- state waves ------------------------------------------------------------------------------
  const __amdgpu_buffer_rsrc_t rv = rsrc(v + (int64_t(n) * H + h) * W * D, W * D * 2);
  const int col = 16 * (NS * part + w) + r;
  // this lane's value column at tokens 16 mu + 4q + i
  uint32_t vreg[8];
  auto fetch_v = [&](int c0) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      vreg[i] = uint16_t(__builtin_amdgcn_raw_buffer_load_b16(
          rv, ((16 * (i >> 2) + 4 * q + (i & 3)) * D + col) * 2, c0 * D * 2, 0));
  };
  fetch_v(0);
  f32x4 S[8] = {};
  const int64_t any = FUSED ? std::max(sAny[0], sAny[1]) : 0;
  if (!init_zero) load_state<FUSED>(S, S_head, ck.ckpt, sOff, any, col, q);
  __syncthreads();
  // (kept rows are written while the first chunk is being solved)
  if (FUSED) copy_kept_rows<64 * 8>(S_head, ck.ckpt, sOff, any, 64 * NS * part + tid);
  __syncthreads();

  struct Frag { bf16x8 h, l; };
  struct KFrag { bf16x8 k[2]; };
  auto split_s = [&](int kk) {   // S' rows of K's step kk
    Frag f;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = S[2 * kk + (e >> 2)][e & 3];
    split8(x, f.h, f.l);
    return f;
  };
  auto load_k = [&](int buf, int kk) {
    const bf16x8* p = reinterpret_cast<const bf16x8*>(smem + OFF_K + buf * K_BYTES) + 128 * kk + lane;
    return KFrag{{p[0], p[64]}};
  };

  KFrag kf = load_k(0, 0);
  Frag sf = split_s(0);
  int buf = 0;
  for (int c = 0; c < n_chunks; ++c) {
    const unsigned char* tp = smem + OFF_TP + (c & 1) * TP16_BYTES;
    const unsigned char* kt = smem + OFF_KT + buf * KT_BYTES + q * KT_ROW + r * 16;
    auto load_kt = [&](int mt) { return *reinterpret_cast<const bf16x8*>(kt + mt * (4 * KT_ROW)); };
    // ---- X = K S' on this wave's columns (rows t, contraction over channels) ---------------
    f32x4 X[2] = {};
    bf16x8 th[2], tl[2];
    f32x4 eg[2], eu[2];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      KFrag kn;
      Frag sn;
      if (kk < 3) {
        kn = load_k(buf, kk + 1);
        sn = split_s(kk + 1);
      } else {
        const uint2 h0 = reinterpret_cast<const uint2*>(tp)[lane], l0 = reinterpret_cast<const uint2*>(tp + 1536)[lane];
        th[0] = __builtin_bit_cast(bf16x8, make_uint4(h0.x, h0.y, 0, 0));
        tl[0] = __builtin_bit_cast(bf16x8, make_uint4(l0.x, l0.y, 0, 0));
        th[1] = reinterpret_cast<const bf16x8*>(tp + 512)[lane];
        tl[1] = reinterpret_cast<const bf16x8*>(tp + 1536 + 512)[lane];
#pragma unroll
        for (int mu = 0; mu < 2; ++mu) {
          eg[mu] = *reinterpret_cast<const f32x4*>(smem + OFF_EG + (buf * C + 16 * mu + 4 * q) * 4);
          eu[mu] = *reinterpret_cast<const f32x4*>(smem + OFF_EU + (buf * C + 16 * mu + 4 * q) * 4);
        }
      }
#pragma unroll
      for (int mu = 0; mu < 2; ++mu) X[mu] = mma(kf.k[mu], sf.l, X[mu]);
#pragma unroll
      for (int mu = 0; mu < 2; ++mu) X[mu] = mma(kf.k[mu], sf.h, X[mu]);
      __builtin_amdgcn_sched_barrier(0);
      kf = kn;
      sf = sn;
    }

    // ---- U = (-T')(Diag(2^{c + G}) X - V), scaled for the update -----------------------------
    f32x4 U[2] = {};
    {
      float x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        x[i] = fmaf(eg[i >> 2][i & 3], X[i >> 2][i & 3], -__uint_as_float(vreg[i] << 16));
      bf16x8 yh, yl;
      split8(x, yh, yl);
      // all four products: two more MFMAs a chunk for a tenth less error
#pragma unroll
      for (int mu = 0; mu < 2; ++mu) U[mu] = mma(tl[mu], yl, U[mu]);
#pragma unroll
      for (int mu = 0; mu < 2; ++mu) U[mu] = mma(tl[mu], yh, U[mu]);
#pragma unroll
      for (int mu = 0; mu < 2; ++mu) U[mu] = mma(th[mu], yl, U[mu]);
#pragma unroll
      for (int mu = 0; mu < 2; ++mu) U[mu] = mma(th[mu], yh, U[mu]) * eu[mu];
    }
    fetch_v((c + 1) * C);   // the next chunk's values (zeros past the window)
    bf16x8 hf[2] = {load_kt(0), load_kt(1)};
    const float gam = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(
        int, reinterpret_cast<const float*>(smem + OFF_GAM)[buf])));
    if (gam != 1.f) {
#pragma unroll
      for (int mt = 0; mt < 8; ++mt) S[mt] *= gam;
    }

    // ---- S' <- 2^c S' + K^T U -------------------------------------------------------------------
    bf16x8 uh, ul;
    {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = U[e & 1][e >> 1];   // tokens t, 16 + t in turn
      split8(x, uh, ul);
    }
    __builtin_amdgcn_sched_barrier(0);
    const int next = buf == 2 ? 0 : buf + 1;
#pragma unroll
    for (int pr = 0; pr < 4; ++pr) {
      bf16x8 hn[2];
      if (pr < 3) {
        hn[0] = load_kt(2 * pr + 2);
        hn[1] = load_kt(2 * pr + 3);
      } else {
        kf = load_k(next, 0);
      }
#pragma unroll
      for (int x = 0; x < 2; ++x) S[2 * pr + x] = mma(hf[x], ul, S[2 * pr + x]);
#pragma unroll
      for (int x = 0; x < 2; ++x) S[2 * pr + x] = mma(hf[x], uh, S[2 * pr + x]);
      __builtin_amdgcn_sched_barrier(0);
      hf[0] = hn[0];
      hf[1] = hn[1];
    }
    buf = next;
    sf = split_s(0);
    __syncthreads();
  }

  store_state(S, S_head, sOmit, col, q);
}

}  // namespace

namespace dasc {

template <bool FUSED>
static void launch(int n_req, int H, int Hqk, int layer, int L, const int32_t* inv_row, float* states,
                   int64_t n_pool, const int32_t* slot, const uint16_t* k, const uint16_t* v,
                   const float* g, const float* beta, int W, int init_zero, const CkptView& ck,
                   hipStream_t st) {
  const unsigned heads = unsigned(n_req) * unsigned(H);
  if (heads <= kSplitHeads)
    hipLaunchKernelGGL((refresh_wy_gdn_kernel<FUSED, 4, false>), dim3(2 * heads), dim3(64 * 6), 0, st, 0, H,
                       Hqk, layer, L, inv_row, states, n_pool, slot, k, v, g, beta, W, init_zero, ck);
  else if (heads > 256 && heads <= kOrderHeads && H <= 64)
    hipLaunchKernelGGL((refresh_wy_gdn_kernel<FUSED, 8, true>), dim3(heads), dim3(64 * 10), 0, st, 0, H, Hqk,
                       layer, L, inv_row, states, n_pool, slot, k, v, g, beta, W, init_zero, ck);
  else
    for (unsigned h0 = 0; h0 < heads; h0 += kWyHeadsPerLaunch)
      hipLaunchKernelGGL((refresh_wy_gdn_kernel<FUSED, 8, false>), dim3(std::min(heads - h0, kWyHeadsPerLaunch)),
                         dim3(64 * 10), 0, st, int(h0), H, Hqk, layer, L, inv_row, states, n_pool, slot,
                         k, v, g, beta, W, init_zero, ck);
}

void launch_refresh_wy_gdn(int n_req, int H, int Hqk, int layer, int L, const int32_t* inv_row,
                           float* states, int64_t n_pool, const int32_t* slot, const uint16_t* k,
                           const uint16_t* v, const float* g, const float* beta, int W,
                           int init_zero, hipStream_t st) {
  launch<false>(n_req, H, Hqk, layer, L, inv_row, states, n_pool, slot, k, v, g, beta, W, init_zero,
                CkptView{nullptr, 1, 1, 0, nullptr}, st);
}

void launch_restore_refresh_wy_gdn(int n_req, int H, int Hqk, int layer, int L, const float* ckpt,
                                   int64_t n_ckpt_slots, const int32_t* ck_slot,
                                   int64_t slice_rows, int64_t n_rows, const int32_t* inv_row,
                                   float* states, int64_t n_pool, const int32_t* slot,
                                   const uint16_t* k, const uint16_t* v, const float* g,
                                   const float* beta, int W, int init_zero, hipStream_t st) {
  launch<true>(n_req, H, Hqk, layer, L, inv_row, states, n_pool, slot, k, v, g, beta, W, init_zero,
               CkptView{ckpt, n_ckpt_slots, slice_rows, n_rows, ck_slot}, st);
}

}  // namespace dasc
