// Parts that the two chunkwise WY refresh kernels share: how the state waves of a block take up
// and put down a head's state, and how the solver wave turns a chunk's A into -T'.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "ckpt_layout.h"
#include "wy_ops.h"

namespace dasc_wy {

constexpr int kDim = 128;         // dk = dv

// One DPP read: lane l takes v from the lane CTRL selects within its row of 16 (0 where that
// lane is outside the row).
template <int CTRL>
__device__ inline float dpp_row(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                                               0xF, 0xF, true));
}

// ---- state waves ---------------------------------------------------------------------------------
// A wave holds one value column per lane of a row of lanes, as MFMA accumulators:
//   f32x16 S[4]  32x32 tiles: register i of tile mt is row 32 mt + (i % 4) + 8 (i / 4) + 4 q,
//                q = lane / 32;
//   f32x4  S[8]  16x16 tiles: register i of tile mt is row 16 mt + 4 q + i, q = lane / 16.
template <typename TILE> struct Tiles;
template <> struct Tiles<f32x16> {
  static constexpr int N = 4, REGS = 16;
  __device__ static int row(int mt, int i, int q) { return 32 * mt + (i & 3) + 8 * (i >> 2) + 4 * q; }
};
template <> struct Tiles<f32x4> {
  static constexpr int N = 8, REGS = 4;
  __device__ static int row(int mt, int i, int q) { return 16 * mt + 4 * q + i; }
};

// Fused: some row that a 64-row half of the head reads from the checkpoint, by the wave whose lanes
// hold the half's offsets (negative where it reads none).
__device__ inline int64_t some_row(int64_t o) {
  const uint64_t read = __ballot(o >= 0);
  const int l = read ? __builtin_ctzll(read) : 0;
  const uint32_t lo = __builtin_amdgcn_readlane(uint32_t(o), l);
  const uint32_t hi = __builtin_amdgcn_readlane(uint32_t(uint64_t(o) >> 32), l);
  return int64_t(uint64_t(hi) << 32 | lo);
}

// The initial state of this lane's column.  FUSED: from the packed checkpoint, off[c] being
// row c's float offset (negative: the row restores as +0.0).  Such a row loads `any`, a row that
// the head reads anyhow, and drops it, so that no load waits on a branch and none goes to memory
// for nothing; a head that reads no row (any < 0) loads nothing.  Loading the head's own pool row
// instead moved 25 MB more in the Load of 16 requests x 32 KDA heads; a branch per row moves as
// little and takes longer (us, W = 16 and 64: pool row 27.5 and 35.2, branch 27.2 and 32.8, this
// 25.7 and 32.6; 1 request, W = 16: 13.1, 13.7, 12.8).
template <bool FUSED, typename TILE>
__device__ inline void load_state(TILE (&S)[Tiles<TILE>::N], const float* S_head, const float* ckpt,
                                  const int64_t* off, int64_t any, int col, int q) {
  using T = Tiles<TILE>;
  constexpr int R = T::REGS;
  if (FUSED && any < 0) return;
#pragma unroll
  for (int mt = 0; mt < T::N; ++mt) {
    float val[R];
    bool ok[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const int c = T::row(mt, i, q);
      const float* src = S_head + int64_t(c) * kDim;
      ok[i] = true;
      if (FUSED) {
        const int64_t o = off[c];
        ok[i] = o >= 0;
        src = ckpt + (ok[i] ? o : any);
      }
      val[i] = src[col];
    }
#pragma unroll
    for (int i = 0; i < R; ++i) S[mt][i] = ok[i] ? val[i] : 0.f;
  }
}

// Fused: every row that is not replayed is final already; its checkpoint row (or +0.0) goes to
// the pool, 16 bytes per thread and access, by THREADS threads.
template <int THREADS>
__device__ inline void copy_kept_rows(float* S_head, const float* ckpt, const int64_t* off,
                                      int64_t any, int tid) {
  if (any < 0) {   // no row to read
    for (int e = tid; e < kDim * kDim / 4; e += THREADS)
      if (off[e >> 5] != dasc::kOmitted) reinterpret_cast<f32x4*>(S_head)[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    return;
  }
#pragma unroll 4
  for (int e = tid; e < kDim * kDim / 4; e += THREADS) {
    const int64_t o = off[e >> 5];
    const f32x4 val = reinterpret_cast<const f32x4*>(ckpt + (o >= 0 ? o : any))[e & 31];
    if (o != dasc::kOmitted)
      reinterpret_cast<f32x4*>(S_head)[e] = o >= 0 ? val : f32x4{0.f, 0.f, 0.f, 0.f};
  }
}

// Fused: a head with nothing to replay is a plain copy (all threads of the block).
__device__ inline void copy_head(float* S_head, const float* ckpt, const int64_t* off, int tid, int n) {
  for (int e = tid; e < kDim * kDim / 4; e += n) {
    const int c = e >> 5, v4 = e & 31;
    const int64_t o = off[c];
    const f32x4 val = o >= 0 ? reinterpret_cast<const f32x4*>(ckpt + o)[v4] : f32x4{0.f, 0.f, 0.f, 0.f};
    reinterpret_cast<f32x4*>(S_head + int64_t(c) * kDim)[v4] = val;
  }
}

// The replayed rows (omitted[c] != 0) of this lane's column.
template <typename TILE>
__device__ inline void store_state(const TILE (&S)[Tiles<TILE>::N], float* S_head,
                                   const unsigned char* omitted, int col, int q) {
  using T = Tiles<TILE>;
#pragma unroll
  for (int mt = 0; mt < T::N; ++mt)
#pragma unroll
    for (int gr = 0; gr < T::REGS / 4; ++gr) {
      const int c = T::row(mt, 4 * gr, q);   // four rows: one omitted flag per byte
      const uint32_t om = *reinterpret_cast<const uint32_t*>(omitted + c);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if ((om >> (8 * i)) & 0xFFu) S_head[int64_t(c + i) * kDim + col] = S[mt][4 * gr + i];
    }
}

// ---- solver wave ---------------------------------------------------------------------------------

// A 16x16 block in the accumulator layout (lane (q, r) holds rows 4q + i of column r), split
// hi/lo into two packed words: the 16x16x16 bf16 MFMA's operand layout for the left factor's
// transpose and for the right factor.
struct Split4 { uint2 h, l; };
__device__ inline Split4 split4(const f32x4 x) {
  Split4 s;
  split2(x[0], x[1], s.h.x, s.l.x);
  split2(x[2], x[3], s.h.y, s.l.y);
  return s;
}
// left * right, the left factor given transposed
__device__ inline f32x4 mulb(const Split4& lt, const Split4& rt) {
  f32x4 c = mma16(lt.l, rt.h, f32x4{0.f, 0.f, 0.f, 0.f});
  c = mma16(lt.h, rt.l, c);
  return mma16(lt.h, rt.h, c);
}

constexpr int ST = 20;                  // row stride (f32) of the 16x16 blocks in LDS
constexpr int T_BYTES = 32 * ST * 4;    // two diagonal blocks, one above the other

// -T' in LDS, as the left operand of U, in one of two orders:
//   for 32x32x16  [step of 16 tokens][hi/lo][lane][8 bf16]; rows 0..15 of the second step are
//                 zero (clear_tp, once per buffer)
//   for 16x16x32  [hi/lo][row tile 0: 4 bf16 (the rest is zero), row tile 1: 8 bf16, by lane]
constexpr int TP32_BYTES = 2 * 2 * 1024, TP16_BYTES = 2 * (512 + 1024);

__device__ inline void clear_tp(unsigned char* tp, int lane) {
#pragma unroll
  for (int hl = 0; hl < 2; ++hl)
    if ((lane & 16) == 0)
      *reinterpret_cast<uint4*>(tp + 2048 + 1024 * hl + lane * 16) = make_uint4(0, 0, 0, 0);
}

// -T' = -(I + A)^{-1} Diag(beta), split hi/lo for 32x32x16 products or (TP16) for 16x16x32 ones.  a: the diagonal blocks of A in LDS (row stride ST; only the entries
// below the diagonal are used); a10: block (1, 0) in the accumulator layout; b: the chunk's
// betas in LDS, b0 those of tokens 4q .. 4q + 3; tf: T_BYTES of scratch.
template <bool TP16>
__device__ inline void solve_chunk(const float* a, const f32x4 a10, const float* b, const f32x4 b0,
                                   float* tf, unsigned char* tp, int q, int r) {
  // T = (I + A)^{-1} row by row from T (I + A) = I: lane r of diagonal block blk takes row r,
  // columns descending; once T[r][s] is known it is taken out of the columns before it
  // (T[r][c] -= T[r][s] A[s][c]), which need row s of A, the same for all lanes of the block.
  // Both blocks at once on lanes 0..31 (lanes 32..63 repeat them).  120 FMAs on operands that
  // depend on nothing: the doubling product (I - B)(I + B^2)(I + B^4)(I + B^8) on split bf16
  // MFMAs takes more instructions (240 for its splits alone) and five dependent levels; the
  // KDA refresh of 5 requests, W = 777, ran 77.2 us with it and 70.7 with the substitution.
  const int blk = q & 1;
  const float* ar = a + 16 * blk * ST;
  float y[16];
#pragma unroll
  for (int t = 0; t < 16; ++t) y[t] = t == r ? 1.f : 0.f;
#pragma unroll
  for (int t = 15; t > 0; --t) {
#pragma unroll
    for (int c4 = 0; c4 < (t + 3) / 4; ++c4) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(ar + t * ST + 4 * c4);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * c4 + i < t) y[4 * c4 + i] = fmaf(-y[t], x[i], y[4 * c4 + i]);
    }
  }
  // the diagonal blocks, rows by lane: tokens 4 h2 .. + 3 and 8 + 4 h2 .. + 3 of a row sit
  // together (lanes of the two halves take one h2 each)
  const int h2 = q >> 1;
  float o[8];
  {
    const f32x4 ba = *reinterpret_cast<const f32x4*>(b + 16 * blk + 4 * h2);
    const f32x4 bb = *reinterpret_cast<const f32x4*>(b + 16 * blk + 8 + 4 * h2);
    f32x4 ya, yb;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ya[i] = h2 ? y[4 + i] : y[i];
      yb[i] = h2 ? y[12 + i] : y[8 + i];
      o[i] = -(ya[i] * ba[i]);
      o[4 + i] = -(yb[i] * bb[i]);
    }
    *reinterpret_cast<f32x4*>(tf + (16 * blk + r) * ST + 4 * h2) = ya;
    *reinterpret_cast<f32x4*>(tf + (16 * blk + r) * ST + 8 + 4 * h2) = yb;
  }
  bf16x8 oh, ol;
  split8(o, oh, ol);
  if (TP16) {   // token groups h2 and 2 + h2 of the row: lanes (h2, r) and (2 + h2, r)
    unsigned char* const od = blk ? tp + 512 + 8 + (16 * h2 + r) * 16 : tp + (16 * h2 + r) * 8;
    const int step = blk ? 32 * 16 : 32 * 8;
    const uint4 hw = __builtin_bit_cast(uint4, oh), lw = __builtin_bit_cast(uint4, ol);
    *reinterpret_cast<uint2*>(od) = make_uint2(hw.x, hw.y);
    *reinterpret_cast<uint2*>(od + step) = make_uint2(hw.z, hw.w);
    *reinterpret_cast<uint2*>(od + 1536) = make_uint2(lw.x, lw.y);
    *reinterpret_cast<uint2*>(od + 1536 + step) = make_uint2(lw.z, lw.w);
  } else {
    unsigned char* const od = tp + (2048 + 256) * blk + (r + 32 * h2) * 16;
    *reinterpret_cast<bf16x8*>(od) = oh;
    *reinterpret_cast<bf16x8*>(od + 1024) = ol;
  }
  wave_lds_sync();
  // T10 = -T11 A10 T00, formed as its transpose -T00^T (A10^T T11^T): lane (q, r) then holds
  // row r of the block at tokens 4q .. 4q + 3
  f32x4 t00;
#pragma unroll
  for (int i = 0; i < 4; ++i) t00[i] = tf[(4 * q + i) * ST + r];
  const f32x4 t11t = *reinterpret_cast<const f32x4*>(tf + (16 + r) * ST + 4 * q);
  f32x4 t10;
  if (TP16) {
    // GDN heads: both products in fp32 (16x16x4 MFMA, step i contracts the tokens 4q + i).  With
    // correlated keys and betas near 1 the entries of T00 and T11 are large and cancel in T10:
    // split bf16 products here cost 7.9e-5 of the state's norm instead of 1.7e-5 (keys of length
    // 1.35 around one direction, beta = 1), 4.56e-6 instead of 4.54e-6 with independent keys.
    // The fp32 MFMAs take up to 1% more time (8-request refresh, W = 1024: 59.0 -> 59.3 us).
    f32x4 z = {0.f, 0.f, 0.f, 0.f};
    t10 = z;
#pragma unroll
    for (int i = 0; i < 4; ++i) z = mma32(a10[i], t11t[i], z);
#pragma unroll
    for (int i = 0; i < 4; ++i) t10 = mma32(t00[i], z[i], t10);
  } else {
    const f32x4 z = mulb(split4(a10), split4(t11t));
    t10 = mulb(split4(t00), split4(z));
  }
  t10 *= b0;   // -T10 Diag(beta)
  const Split4 o10 = split4(t10);
  unsigned char* const o1 = TP16 ? tp + 512 + (16 * q + r) * 16
                                   : tp + 256 + (r + 32 * (q & 1)) * 16 + (q >> 1) * 8;
  *reinterpret_cast<uint2*>(o1) = o10.h;
  *reinterpret_cast<uint2*>(o1 + (TP16 ? 1536 : 1024)) = o10.l;
}

}  // namespace dasc_wy
