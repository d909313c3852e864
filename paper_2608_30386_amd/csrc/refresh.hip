// Bounded-suffix refresh (DASC-WR, Sec. 4.2) of the gated delta-rule state (Eq. 1).
//
// The state of one head is stored transposed, S' = S^T in R^{dk x dv}; per token
//     S~   = Diag(exp(g_t)) S'_{t-1}
//     S'_t = S~ + beta_t k_t (v_t - S~^T k_t)^T
// Column j of S' (value channel j) evolves on its own: it needs k_t, g_t, beta_t and
// the single value v_t[j].  This kernel, for every head size the MFMA kernels are not built
// for, holds a column in G = dk / 8 adjacent lanes, eight rows each, so that S~^T k_t is eight
// products per lane and log2 G lane-shift additions (DPP), and a head of 64 x 64 runs on eight
// waves.  Blocks of 256 threads take 2048 / dk columns of a (request, head), smaller ones the
// narrow heads of large calls (kNarrowHeads); the columns of a head that need more blocks repeat
// the staging of k and g.  k, exp(g), v and beta of the next tile of tokens are loaded while a
// tile is worked on, and staged into the other of two LDS buffers after it.
//
// What bounds it: the chain of one token (decay, products, lane additions, delta, update) at
// about 250 cycles while the chip has no more than a wave or two per SIMD, which is any call of
// up to a few hundred heads; vector issue (about 30 instructions per token and wave) beyond.  A
// thread per column with its dk rows in registers instead does dk dependent FMAs a token and
// leaves most SIMDs idle: 8 requests x 16 KDA heads of 64 x 64, W = 512: 619 us, now 58; at W = 256
// 16 x 32 heads 325 -> 69, 8 x 16 heads of 16 x 16 63 -> 27, 16 x 32 heads of 128 x 100 643 -> 235 to
// 260 (with the clock).  It is the faster one still for windows of one or two tokens of thousands
// of heads of 64 or 128 rows (64 x 32 of 128 x 64: 54 and 69 at W = 1, 79 and 71 at W = 4), where the
// prologue is all there is.  Two columns per lane (half the LDS reads per column) gain 5-9% from 512 heads of 64 or
// more rows on and lose 40% below.
//
// Everything is fp32, the state within fp32 rounding of the per-token rule (3.7e-7 of its norm
// after 512 tokens).  Only the omitted rows of the head (KDA) or the omitted heads (GDN) are
// written back; everything else in the active state keeps its bits.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "dasc.h"
#include "dasc_testing.h"
#include "launch_common.h"
#include "refresh_kernels.h"
#include "wy_ops.h"

namespace {

using dasc_wy::f32x2;
using dasc_wy::f32x4;

constexpr int kRows = 8;      // state rows per lane
// Heads of 16 or 32 rows whose columns need 64 or 128 lanes take blocks of that many threads from
// this many heads on, where waves without a column would keep others off the chip; the other
// calls take blocks of 256, of which fewer heads leave the chip idle and four waves stage a tile
// sooner.  us, 256 threads -> 64 or 128: 64 requests x 32 heads of 16 x 16, W = 512: 213 -> 71 (a
// thread per column: 177), of 16 x 4, W = 256: 108 -> 37 (83), of 32 x 32: 111 -> 75 (178); 512 heads
// of 16 x 16, W = 256: 33.4 -> 29.8, of 32 x 32: 34.7 -> 32.7; 256 heads of 32 x 16: 29.2 -> 29.2, 128
// heads, W = 512: 51.8 -> 53.4; 16 heads of 16 x 64: 48.5 -> 51.3.
constexpr int64_t kNarrowHeads = 512;
// Heads of one launch: the grid counts threads in 32 bits, so longer lists go in slices.
constexpr int64_t kHeadsPerLaunch = int64_t(1) << 19;
// Tokens staged per LDS tile.  32 measures 7-9% better than 16 for 16 or 32 rows (fewer
// barriers), but from 64 rows on its LDS (41 KB, 68 KB) costs resident blocks: 1-15% worse on
// 512 heads (64 x 64 70 against 70.5 us, 128 x 100 257 against 296).
constexpr int tile_tokens(int dk) { return dk <= 32 ? 32 : 16; }

template <int CTRL>
__device__ inline float dpp_add(float x) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL,
                                                                   0xF, 0xF, true));
}
// Sum over the G = 2 .. 16 adjacent lanes that hold one column, the result in each of them:
// lane l adds lane l ^ 1, l ^ 2, then its mirror in the group of 8 and in the row of 16 (whose
// quads, then halves, hold equal values by then).
template <int G>
__device__ inline float group_sum(float x) {
  x = dpp_add<0xB1>(x);                   // quad_perm [1,0,3,2]
  if (G >= 4) x = dpp_add<0x4E>(x);       // quad_perm [2,3,0,1]
  if (G >= 8) x = dpp_add<0x141>(x);      // row_half_mirror
  if (G >= 16) x = dpp_add<0x140>(x);     // row_mirror
  return x;
}

template <int DK, bool PER_CHANNEL, int NT>
__global__ __launch_bounds__(NT) void refresh_column_kernel(
    int H, int Hqk, int dv, int layer, int L, const int32_t* __restrict__ inv_row,
    float* __restrict__ states, int64_t n_pool, const int32_t* __restrict__ slot,
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, const float* __restrict__ g,
    const float* __restrict__ beta, int W, int init_zero, int head0,
    int col_blocks) {
  constexpr int kTile = tile_tokens(DK);
  constexpr int G = DK / kRows;           // lanes per column
  constexpr int CB = NT / G;              // columns per block
  constexpr int HALF = DK / 2;
  __shared__ __attribute__((aligned(16))) float k_s[2][kTile][DK];
  __shared__ __attribute__((aligned(16))) float a_s[2][kTile][PER_CHANNEL ? DK : 1];
  __shared__ __attribute__((aligned(16))) float v_s[2][kTile][CB];
  __shared__ float b_s[2][kTile];

  // the column blocks of a head are neighbours, so that they find its k and g in a cache
  // (8 requests x 16 GDN heads of 128 x 256: 83 us, 104 with the columns as the grid's second
  // dimension)
  const int nh = head0 + int(blockIdx.x) / col_blocks;
  const int cb = int(blockIdx.x) % col_blocks;
  const int n = nh / H;
  const int h = nh - n * H;
  const int tid = threadIdx.x;
  const int rg = tid % G;
  const int jb = tid / G;                 // this lane's column in the block
  const int j = cb * CB + jb;

  const int64_t head_row = (int64_t(layer) * H + h) * DK;
  // Does this head have anything to refresh?
  bool mine = false;
  for (int c = tid; c < DK; c += NT) mine |= inv_row[head_row + c] < 0;
  const int64_t s = slot[n];
  if (!__syncthreads_or(mine)) return;
  if (s < 0 || s >= n_pool) return;

  const int hk = h / (H / Hqk);
  const __amdgpu_buffer_rsrc_t rk = dasc_wy::rsrc(k + (int64_t(n) * Hqk + hk) * W * DK, W * DK * 2);
  const __amdgpu_buffer_rsrc_t rv = dasc_wy::rsrc(v + (int64_t(n) * H + h) * W * dv, W * dv * 2);
  const __amdgpu_buffer_rsrc_t rg_ = dasc_wy::rsrc(
      PER_CHANNEL ? g + (int64_t(n) * H + h) * W * DK : g + (int64_t(n) * H + h) * W,
      PER_CHANNEL ? W * DK * 4 : W * 4);
  const __amdgpu_buffer_rsrc_t rb = dasc_wy::rsrc(beta + (int64_t(n) * H + h) * W, W * 4);

  // One tile's inputs as this thread loads them, a tile ahead: words of two keys or values
  // (two gates), tokens past the window as zeros (not used).
  constexpr int KW = (kTile * DK / 2 + NT - 1) / NT, VW = (kTile * CB / 2 + NT - 1) / NT;
  uint32_t kraw[KW], vraw[VW];
  f32x2 graw[PER_CHANNEL ? KW : 1];
  float braw = 0.f, g1 = 0.f;
  auto fetch = [&](int t0) {
#pragma unroll
    for (int i = 0; i < KW; ++i) {
      const int e = tid + i * NT;         // word e: token e / (DK/2), channels 2 (e % (DK/2)), +1
      kraw[i] = __builtin_amdgcn_raw_buffer_load_b32(rk, e * 4, t0 * DK * 2, 0);
      if (PER_CHANNEL) graw[i] = dasc_wy::ldf2(rg_, e * 8, t0 * DK * 4);
    }
#pragma unroll
    for (int i = 0; i < VW; ++i) {
      const int e = tid + i * NT;
      const int t = e / (CB / 2), c = 2 * (e % (CB / 2));
      vraw[i] = __builtin_amdgcn_raw_buffer_load_b32(rv, (t * dv + cb * CB + c) * 2, t0 * dv * 2, 0);
    }
    if (tid < kTile) {
      braw = dasc_wy::ldf(rb, tid * 4, t0 * 4);
      if (!PER_CHANNEL) g1 = dasc_wy::ldf(rg_, tid * 4, t0 * 4);
    }
  };
  auto stage = [&](int b) {
#pragma unroll
    for (int i = 0; i < KW; ++i) {
      const int e = tid + i * NT;
      if (kTile * DK / 2 % NT == 0 || e < kTile * DK / 2) {
        reinterpret_cast<f32x2*>(k_s[b])[e] =
            f32x2{__uint_as_float(kraw[i] << 16), __uint_as_float(kraw[i] & 0xFFFF0000u)};
        if (PER_CHANNEL) reinterpret_cast<f32x2*>(a_s[b])[e] = f32x2{expf(graw[i][0]), expf(graw[i][1])};
      }
    }
#pragma unroll
    for (int i = 0; i < VW; ++i) {
      const int e = tid + i * NT;
      if (kTile * CB / 2 % NT == 0 || e < kTile * CB / 2)
        reinterpret_cast<f32x2*>(v_s[b])[e] =
            f32x2{__uint_as_float(vraw[i] << 16), __uint_as_float(vraw[i] & 0xFFFF0000u)};
    }
    if (tid < kTile) {
      b_s[b][tid] = braw;
      if (!PER_CHANNEL) a_s[b][tid][0] = expf(g1);
    }
  };

  // This lane's rows: 4 rg .. 4 rg + 3 and DK/2 + 4 rg .. + 3, so that the lanes of a column
  // read a token's keys as two contiguous runs
  float* S_head = states + (s * L * H * DK + head_row) * dv;
  const bool col = j < dv;
  float st[kRows];
#pragma unroll
  for (int i = 0; i < kRows; ++i) {
    const int c = (i >> 2) * HALF + 4 * rg + (i & 3);
    st[i] = (col && !init_zero) ? S_head[int64_t(c) * dv + j] : 0.f;
  }

  struct Token { f32x4 k[2], a[2]; float a1, b, v; };
  auto load = [&](int b, int tt) {
    Token x;
    x.k[0] = *reinterpret_cast<const f32x4*>(&k_s[b][tt][4 * rg]);
    x.k[1] = *reinterpret_cast<const f32x4*>(&k_s[b][tt][HALF + 4 * rg]);
    if (PER_CHANNEL) {
      x.a[0] = *reinterpret_cast<const f32x4*>(&a_s[b][tt][4 * rg]);
      x.a[1] = *reinterpret_cast<const f32x4*>(&a_s[b][tt][HALF + 4 * rg]);
    } else {
      x.a1 = a_s[b][tt][0];
    }
    x.v = v_s[b][tt][jb];
    x.b = b_s[b][tt];
    return x;
  };
  auto step = [&](const Token& x) {
    float y[2];
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      st[i] *= PER_CHANNEL ? x.a[i >> 2][i & 3] : x.a1;                // decay first
      const float kk = x.k[i >> 2][i & 3];
      y[i & 1] = i < 2 ? kk * st[i] : fmaf(kk, st[i], y[i & 1]);        // S~^T k_t
    }
    const float d = x.b * (x.v - group_sum<G>(y[0] + y[1]));
#pragma unroll
    for (int i = 0; i < kRows; ++i) st[i] = fmaf(x.k[i >> 2][i & 3], d, st[i]);   // + beta k (v - S~^T k)^T
  };

  fetch(0);
  stage(0);
  int b = 0;
  for (int t0 = 0; t0 < W; t0 += kTile, b ^= 1) {
    if (t0 + kTile < W) fetch(t0 + kTile);
    __syncthreads();   // tile b is staged, and every wave is done with the other buffer
    const int nt = min(kTile, W - t0);
    Token cur = load(b, 0);
    if (nt == kTile) {
#pragma unroll
      for (int tt = 0; tt < kTile; ++tt) {
        Token nxt = cur;
        if (tt + 1 < kTile) nxt = load(b, tt + 1);
        step(cur);
        cur = nxt;
      }
    } else {
      for (int tt = 0; tt < nt; ++tt) {
        const Token nxt = load(b, min(tt + 1, kTile - 1));
        step(cur);
        cur = nxt;
      }
    }
    if (t0 + kTile < W) stage(b ^ 1);
  }

  if (!col) return;
#pragma unroll
  for (int i = 0; i < kRows; ++i) {
    const int c = (i >> 2) * HALF + 4 * rg + (i & 3);
    if (inv_row[head_row + c] < 0) S_head[int64_t(c) * dv + j] = st[i];
  }
}

template <int DK, int NT>
void launch_column_nt(bool per_channel, int64_t heads, hipStream_t st, int H, int Hqk, int dv, int layer,
                      int L, const int32_t* inv_row, float* states, int64_t n_pool,
                      const int32_t* slot, const uint16_t* k, const uint16_t* v, const float* g,
                      const float* beta, int W, int init_zero) {
  constexpr int CB = NT / (DK / kRows);
  const int cbs = (dv + CB - 1) / CB;
  for (int64_t h0 = 0; h0 < heads; h0 += kHeadsPerLaunch) {
    const dim3 grid(unsigned(std::min(heads - h0, kHeadsPerLaunch) * cbs));
    if (per_channel)
      hipLaunchKernelGGL((refresh_column_kernel<DK, true, NT>), grid, dim3(NT), 0, st, H, Hqk, dv, layer,
                         L, inv_row, states, n_pool, slot, k, v, g, beta, W, init_zero, int(h0), cbs);
    else
      hipLaunchKernelGGL((refresh_column_kernel<DK, false, NT>), grid, dim3(NT), 0, st, H, Hqk, dv, layer,
                         L, inv_row, states, n_pool, slot, k, v, g, beta, W, init_zero, int(h0), cbs);
  }
}

template <int DK, class... A>
void launch_column(bool per_channel, int64_t heads, hipStream_t st, int H, int Hqk, int dv, A... a) {
  if (DK <= 32 && heads >= kNarrowHeads) {
    const int lanes = dv * (DK / kRows);
    if (lanes <= 64) return launch_column_nt<DK, 64>(per_channel, heads, st, H, Hqk, dv, a...);
    if (lanes <= 128) return launch_column_nt<DK, 128>(per_channel, heads, st, H, Hqk, dv, a...);
  }
  launch_column_nt<DK, 256>(per_channel, heads, st, H, Hqk, dv, a...);
}

// Does this shape take the scalar-gate GDN kernel?
bool uses_gdn_kernel(const dasc_shape* shape) {
  return shape->arch == DASC_ARCH_GDN && dasc::refresh_wy_supported(shape->dk, shape->dv);
}

// The workspace the interface reserves for the GDN kernel: 4 KiB per 32-token chunk and head.
size_t gdn_workspace_bytes(int n_req, int H, int W) {
  return size_t(n_req) * size_t(H) * size_t((int64_t(W) + 31) / 32) * size_t(4096);
}
// Largest request list the GDN path takes: heads times groups of four chunks within 32 bits.
// Nothing in the kernels asks for it; it stays so that the same calls are taken and refused.
bool gdn_size_ok(int n_req, int H, int W) {
  return int64_t(n_req) * H * (((int64_t(W) + 31) / 32 + 3) / 4) <= INT32_MAX;
}

}  // namespace

extern "C" int dasc_refresh_workspace_bytes(const dasc_shape* shape, int32_t n_req, int32_t W,
                                            size_t* bytes) {
  if (!shape || !bytes || n_req < 1 || W < 1) return DASC_E_INVAL;
  if (!dasc::valid_shape(shape)) return DASC_E_SHAPE;
  *bytes = uses_gdn_kernel(shape) ? gdn_workspace_bytes(n_req, shape->n_heads, W) : 0;
  return DASC_OK;
}

namespace dasc {

// dasc_refresh with an explicit kernel choice (DASC_REFRESH_KERNEL_*): AUTO takes the
// chunked MFMA kernels at dk = dv = 128 (the scalar-gate one for GDN heads) and the
// per-column fp32 kernel for every other shape.
int refresh_impl(const dasc_shape* shape, int32_t layer, const int32_t* inv_row, float* states,
                 int64_t n_pool, const int32_t* slot, const uint16_t* k, const uint16_t* v,
                 const float* g, const float* beta, int32_t n_req, int32_t W, int32_t init_mode,
                 const void* workspace, size_t workspace_bytes, bool noalloc, int32_t kernel,
                 dasc_stream_t stream) {
  if (!shape) return DASC_E_INVAL;
  if (!dasc::valid_shape(shape) || shape->dv % 4 != 0) return DASC_E_SHAPE;
  if (layer < 0 || layer >= shape->n_layers || n_req < 1 || W < 1 || W > DASC_MAX_WINDOW ||
      n_pool < 1)
    return DASC_E_INVAL;
  if (init_mode != DASC_INIT_RESTORED && init_mode != DASC_INIT_ZERO) return DASC_E_INVAL;
  if (kernel != DASC_REFRESH_KERNEL_AUTO && kernel != DASC_REFRESH_KERNEL_COLUMN &&
      kernel != DASC_REFRESH_KERNEL_CHANNEL_WY)
    return DASC_E_INVAL;
  if (!inv_row || !states || !slot || !k || !v || !g || !beta) return DASC_E_INVAL;
  if (!dasc::aligned16(states) || !dasc::aligned16(k) || !dasc::aligned16(v)) return DASC_E_INVAL;
  const int dk = shape->dk, dv = shape->dv;
  if (dv > 256) return DASC_E_UNSUPPORTED;
  if (kernel == DASC_REFRESH_KERNEL_CHANNEL_WY && !dasc::refresh_wy_supported(dk, dv))
    return DASC_E_UNSUPPORTED;
  const bool gdn_kernel = kernel == DASC_REFRESH_KERNEL_AUTO && uses_gdn_kernel(shape);
  const size_t need = gdn_kernel && !noalloc ? gdn_workspace_bytes(n_req, shape->n_heads, W) : 0;
  if (workspace_bytes < need || (need > 0 && !workspace)) return DASC_E_WORKSPACE;
  if (need > 0 && !dasc::aligned16(workspace)) return DASC_E_INVAL;
  if (2 * int64_t(n_req) * shape->n_heads > INT32_MAX) return DASC_E_INVAL;

  const bool per_channel = shape->arch == DASC_ARCH_KDA;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const int zero = init_mode == DASC_INIT_ZERO;
  (void)hipGetLastError();
  if (gdn_kernel) {
    if (!gdn_size_ok(n_req, shape->n_heads, W)) return DASC_E_INVAL;
    dasc::launch_refresh_wy_gdn(n_req, shape->n_heads, shape->n_qk_heads, layer,
                                shape->n_layers, inv_row, states, n_pool, slot, k, v, g, beta, W,
                                zero, st);
    return dasc::launch_status();
  }
  if (kernel != DASC_REFRESH_KERNEL_COLUMN && dasc::refresh_wy_supported(dk, dv)) {
    dasc::launch_refresh_wy(per_channel, n_req, shape->n_heads, shape->n_qk_heads, layer,
                            shape->n_layers, inv_row, states, n_pool, slot, k, v, g, beta, W,
                            zero, st);
    return dasc::launch_status();
  }
  const int64_t heads = int64_t(n_req) * shape->n_heads;
  switch (dk) {
#define DASC_DK(D)                                                                              \
  case D:                                                                                       \
    launch_column<D>(per_channel, heads, st, shape->n_heads, shape->n_qk_heads, dv, layer,        \
                     shape->n_layers, inv_row, states, n_pool, slot, k, v, g, beta, W, zero);      \
    break;
    DASC_DK(16) DASC_DK(32) DASC_DK(64) DASC_DK(128)
#undef DASC_DK
    default: return DASC_E_UNSUPPORTED;
  }
  return dasc::launch_status();
}

}  // namespace dasc

extern "C" int dasc_refresh(const dasc_shape* shape, int32_t layer, const int32_t* inv_row,
                            float* states, int64_t n_pool, const int32_t* slot,
                            const uint16_t* k, const uint16_t* v, const float* g,
                            const float* beta, int32_t n_req, int32_t W, int32_t init_mode,
                            void* workspace, size_t workspace_bytes, dasc_stream_t stream) {
  return dasc::refresh_impl(shape, layer, inv_row, states, n_pool, slot, k, v, g, beta, n_req, W,
                            init_mode, workspace, workspace_bytes, false, DASC_REFRESH_KERNEL_AUTO,
                            stream);
}

extern "C" int dasc_refresh_select(const dasc_shape* shape, int32_t layer, const int32_t* inv_row,
                                   float* states, int64_t n_pool, const int32_t* slot,
                                   const uint16_t* k, const uint16_t* v, const float* g,
                                   const float* beta, int32_t n_req, int32_t W, int32_t init_mode,
                                   void* workspace, size_t workspace_bytes, int32_t kernel,
                                   dasc_stream_t stream) {
  return dasc::refresh_impl(shape, layer, inv_row, states, n_pool, slot, k, v, g, beta, n_req, W,
                            init_mode, workspace, workspace_bytes, false, kernel, stream);
}

extern "C" int dasc_restore_refresh(const dasc_shape* shape, int32_t layer, const float* ckpt,
                                    int64_t n_ckpt_slots, const int32_t* src_slot,
                                    int32_t n_ranks, int64_t slice_rows, int64_t n_rows,
                                    const int32_t* inv_row, float* states, int64_t n_pool,
                                    const int32_t* dst_slot, const uint16_t* k,
                                    const uint16_t* v, const float* g, const float* beta,
                                    int32_t n_req, int32_t W, int32_t init_mode,
                                    void* workspace, size_t workspace_bytes,
                                    dasc_stream_t stream) {
  if (!shape) return DASC_E_INVAL;
  if (!dasc::valid_shape(shape) || shape->dv % 4 != 0) return DASC_E_SHAPE;
  if (layer < 0 || layer >= shape->n_layers || n_req < 1 || W < 1 || W > DASC_MAX_WINDOW ||
      n_pool < 1 || n_ckpt_slots < 1 || n_ranks < 1 || n_rows < 0)
    return DASC_E_INVAL;
  if (n_rows > dasc::rows_per_state(shape)) return DASC_E_SHAPE;
  if (n_rows > 0 && (slice_rows < 1 || slice_rows > INT32_MAX || slice_rows * n_ranks < n_rows))
    return DASC_E_INVAL;
  if (init_mode != DASC_INIT_RESTORED && init_mode != DASC_INIT_ZERO) return DASC_E_INVAL;
  if (!inv_row || !states || !src_slot || !dst_slot || !k || !v || !g || !beta)
    return DASC_E_INVAL;
  if (n_rows > 0 && !ckpt) return DASC_E_INVAL;
  if (!dasc::aligned16(states) || !dasc::aligned16(ckpt) || !dasc::aligned16(k) ||
      !dasc::aligned16(v))
    return DASC_E_INVAL;
  size_t need = 0;
  int rc = dasc_refresh_workspace_bytes(shape, n_req, W, &need);
  if (rc != DASC_OK) return rc;
  if (workspace_bytes < need || (need > 0 && !workspace)) return DASC_E_WORKSPACE;
  if (need > 0 && !dasc::aligned16(workspace)) return DASC_E_INVAL;
  if (!dasc::refresh_wy_supported(shape->dk, shape->dv)) return DASC_E_UNSUPPORTED;
  if (2 * int64_t(n_req) * shape->n_heads > INT32_MAX) return DASC_E_INVAL;
  if (n_rows == 0) slice_rows = 1;  // nothing is read; keeps the divisor non-zero
  (void)hipGetLastError();
  // GDN heads take the scalar-gate kernel, as in dasc_refresh
  if (uses_gdn_kernel(shape)) {
    if (!gdn_size_ok(n_req, shape->n_heads, W)) return DASC_E_INVAL;
    dasc::launch_restore_refresh_wy_gdn(n_req, shape->n_heads, shape->n_qk_heads, layer,
                                        shape->n_layers, ckpt, n_ckpt_slots, src_slot, slice_rows,
                                        n_rows, inv_row, states, n_pool, dst_slot, k, v, g, beta,
                                        W, init_mode == DASC_INIT_ZERO,
                                        reinterpret_cast<hipStream_t>(stream));
  } else
    dasc::launch_restore_refresh_wy(n_req, shape->n_heads, shape->n_qk_heads, layer,
                                    shape->n_layers, ckpt, n_ckpt_slots, src_slot, slice_rows,
                                    n_rows, inv_row, states, n_pool, dst_slot, k, v, g, beta, W,
                                    init_mode == DASC_INIT_ZERO,
                                    reinterpret_cast<hipStream_t>(stream));
  return dasc::launch_status();
}
