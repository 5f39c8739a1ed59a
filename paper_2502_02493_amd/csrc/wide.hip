// Wide passes (gfx950, bf16 models): a calibration of more than 16 token columns — several sequences' accepted tokens,
// or their prompts' chunks — as ONE forward pass of up to 256 columns, every weight matrix read once.
//
// With that many columns a weight contraction is a matrix product between a memory-bound stream (a few dozen columns)
// and a compute-bound one (256 columns: two bf16 terms per activation, 512 MFMA columns).  One kernel covers both:
//   * A workgroup of eight waves takes 4 RW row tiles of 16 and CT column tiles of 16; its waves are four row groups
//     times two halves of every stage's k-tiles.  A wave keeps its own RW row tiles' weights in registers (each weight
//     fragment is loaded once, by one wave, straight from memory: the weights need no LDS) and multiplies them with all
//     CT column tiles, whose hi and lo fragments the waves share through LDS.  Per k-tile and wave that is RW weight
//     loads and 2 CT LDS reads for 2 RW CT MFMAs: with RW = 4, CT = 8 the LDS delivers 64 of its 128 bytes per clock
//     while the matrix pipe is full; the plain 16-column kernels (a wave per row tile, operands straight from the L2)
//     ask the L2 for as many operand bytes as weight bytes at 12 columns.  The halves put two waves on a SIMD
//     without a second reader of the same operand; their sums meet in LDS at the end.
//   * Stages of 2 KS k-tiles, the operand double-buffered in LDS, one barrier per stage; weights are requested two
//     stages ahead, the operand one, LDS fragments two steps ahead.
//   * Few row tiles (QKV, O, down: 256 to 384) are spread over the CUs by splitting K; the fp32 partial sums are added
//     in split order by the kernel that does what follows anyway (rotary and cache write; residual and norm operand).
// Measured at the 8B shape, a prefill of 16 x 16 tokens (256 columns): 41.8 -> 9.7 ms (eight pairs of 16-column passes
// before); gate/up 119 us a layer (120 GFLOP with both terms: 1.0 PFLOP/s), down 78, QKV 33, O 24.  4 x 6 tokens at
// contexts 4096 .. 32768 (24 columns): 6.57 -> 5.90 ms; gate/up 55 us there (4.3 TB/s).
// On the way there (256 columns): LDS fragments read next to their use 141 us for the mean of gate/up and QKV; read two
// steps ahead 100; weights two stages ahead but behind branches 94; unconditional requests 76.
#include "launch_common.hpp"

#include <math.h>
#include <string.h>

#include "../../include/easyspec_instrument.h"

namespace es {

enum { kEpiPartial = 0, kEpiSilu = 1, kEpiLogits = 2 };

struct WideArgs {
  const u32x4* w0;  // first matrix (gate; first rotary halves; or the only one)
  const u32x4* w1;  // second matrix of a pair, or null
  int rows;         // rows of one packed matrix (padded to whole tiles of R: every row can be read)
  int rows_out;     // rows of the result per matrix
  int R, nkt;
  int row_blocks, splits, per_split;  // k-tiles per split
  int col_blocks, col_tiles;          // column blocks of CT tiles; column tiles of the pass
  const u32x4* x;   // operand, 128 pieces per (column tile, k-tile)
  int n;            // columns
  int epi;
  float* out;       // kEpiPartial: [split][cols16][rows_out * matrices]; kEpiLogits: logits
  bf16_t* act;      // kEpiSilu: operand of width rows_out
  const float* rs;  // kEpiSilu, kEpiLogits: [cols]
};

// PAIR: the wave's row tiles are RW / 2 tiles of each of two matrices.  See the head of this file.
constexpr int kWideThreads = 512;  // four row groups x two halves of a stage's k-tiles
template <int RW, int CT, int KS, bool PAIR>
__global__ __launch_bounds__(kWideThreads) void wide_gemm_kernel(WideArgs a, Spans sp) {
  constexpr int SK = 2 * KS;                               // k-tiles per stage: KS for each half
  constexpr int NB = SK * CT * 128 / kWideThreads;         // 16-byte operand pieces a thread stages per stage
  static_assert(SK * CT * 128 % kWideThreads == 0, "whole pieces per thread");
  constexpr int RU = PAIR ? RW / 2 : RW;                   // row tiles of a matrix per wave
  constexpr int kStagePieces = SK * CT * 128;
  __shared__ u32x4 xs[2 * kStagePieces];                   // two stages of [column tile][k-tile of the stage][part][lane]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), rg = wave & 3, half = wave >> 2;
  const int unit = wide_unit(blockIdx.x, a.col_blocks), cb = wide_col_block(blockIdx.x, a.col_blocks);
  if (unit >= a.row_blocks * a.splits) return;
  const int rb = unit / a.splits, split = unit % a.splits;
  const int k0 = split * a.per_split, k1 = min(a.nkt, k0 + a.per_split);
  const int t0 = (rb * 4 + rg) * RU, ct0 = cb * CT;
  const u32x4* wp[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    const int t = PAIR ? t0 + r / 2 : t0 + r;
    wp[r] = (PAIR && (r & 1) ? a.w1 : a.w0) + wide_piece(lane, t, a.rows, a.R, a.nkt);
  }
  const int w_stride = fragment_pieces(a.R);
  // operand piece j of this thread: piece i = j * threads + tid of the stage, k-tile i % (SK * 128) / 128 of it, column
  // tile ct0 + i / (SK * 128) (a missing last tile re-reads its neighbour)
  const u32x4* xp[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int i = j * kWideThreads + tid, ct = min(ct0 + i / (SK * 128), a.col_tiles - 1);
    xp[j] = a.x + ((size_t)ct * a.nkt) * 128 + i % (SK * 128);
  }
  const u32x4 zero = {0u, 0u, 0u, 0u};
  f32x4 acc[RW][CT];
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Weights are requested two stages before they are used (they come from memory: a stage of products does not cover
  // that latency under load), operand pieces one stage (they come from the L2).  Requests of a stage are issued operand
  // first, so that waiting for the operand leaves the younger weight requests in flight.  All requests are unconditional
  // (no branch for the compiler to wait at): past the split's end they repeat its last stage (operand) or k-tile
  // (weights), whose lines are at hand; the products of k-tiles past the end are skipped.
  u32x4 w[3][KS][RW], xn[NB];
  auto load_w = [&](int kt, u32x4 (&d)[KS][RW]) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const size_t at = (size_t)min(kt + half * KS + ks, k1 - 1) * w_stride;
#pragma unroll
      for (int r = 0; r < RW; ++r) d[ks][r] = __builtin_nontemporal_load(wp[r] + at);
    }
  };
  auto load_x = [&](int kt) {
#pragma unroll
    for (int j = 0; j < NB; ++j) xn[j] = xp[j][(size_t)kt * 128];
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int j = 0; j < NB; ++j) xs[buf * kStagePieces + j * kWideThreads + tid] = xn[j];
  };
  // The products of one stage: KS * CT steps of (hi, lo) fragments, read from LDS two steps before they are used (the
  // scheduling barriers keep the compiler from moving a read next to its use, where its latency would be exposed)
  auto products = [&](int buf, const u32x4 (&wa)[KS][RW], int n_ks) {  // of the first n_ks of the half's k-tiles
    constexpr int AHEAD = CT < 2 ? CT : 2;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if (ks >= n_ks) break;  // uniform
      const u32x4* xb = xs + buf * kStagePieces + (half * KS + ks) * 128 + lane;
      u32x4 bh[AHEAD + 1], bl[AHEAD + 1];
#pragma unroll
      for (int c = -AHEAD; c < CT; ++c) {
        const int f = c + AHEAD;
        if (f < CT) {
          bh[f % (AHEAD + 1)] = xb[f * SK * 128];
          bl[f % (AHEAD + 1)] = xb[f * SK * 128 + 64];
        }
        if (c < 0) continue;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < RW; ++r) mma<bf16_t>(acc[r][c], wa[ks][r], bh[c % (AHEAD + 1)]);
#pragma unroll
        for (int r = 0; r < RW; ++r) mma<bf16_t>(acc[r][c], wa[ks][r], bl[c % (AHEAD + 1)]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  if (k0 < k1) {
    const int k_last = k0 + (k1 - k0 - 1) / SK * SK;  // first k-tile of the last stage
    int kt = k0, buf = 0;
    load_x(k0);
    load_w(k0, w[0]);
    load_w(k0 + SK, w[1]);
    put(0);
    __syncthreads();
    // one stage; the weight registers rotate by name (a copy would wait for the requests).  False: it was the last.
    auto step = [&](u32x4 (&now)[KS][RW], u32x4 (&later)[KS][RW]) {
      load_x(min(kt + SK, k_last));
      load_w(kt + 2 * SK, later);
      __builtin_amdgcn_sched_barrier(0);
      products(buf, now, k1 - kt - half * KS);
      kt += SK;
      if (kt >= k1) return false;
      buf ^= 1;
      put(buf);
      __syncthreads();
      return true;
    };
    while (step(w[0], w[2]) && step(w[1], w[0]) && step(w[2], w[1])) {
    }
  }
  // the second half's sums onto the first's, through the LDS of the operand stages, as many column tiles at a time as fit
  {
    constexpr int PER = 2 * kStagePieces / (4 * RW * 64), CC = PER < CT ? PER : CT;
    static_assert(PER >= 1, "a column tile's sums fit");
    f32x4* red = reinterpret_cast<f32x4*>(xs) + (size_t)rg * CC * RW * 64 + lane;
#pragma unroll
    for (int c0 = 0; c0 < CT; c0 += CC) {
      __syncthreads();
      if (half == 1) {
#pragma unroll
        for (int c = c0; c < c0 + CC && c < CT; ++c)
#pragma unroll
          for (int r = 0; r < RW; ++r) red[((c - c0) * RW + r) * 64] = acc[r][c];
      }
      __syncthreads();
      if (half == 0) {
#pragma unroll
        for (int c = c0; c < c0 + CC && c < CT; ++c)
#pragma unroll
          for (int r = 0; r < RW; ++r) acc[r][c] += red[((c - c0) * RW + r) * 64];
      }
    }
    if (half == 1) return;
  }

  const int row4 = (lane >> 4) * 4;
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int col = (ct0 + c) * 16 + (lane & 15);
    if (col >= a.n) continue;
    if (a.epi == kEpiPartial) {
      const int width = PAIR ? 2 * a.rows_out : a.rows_out;
      float* o = a.out + ((size_t)split * (a.col_tiles * 16) + col) * width;
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        const int row = (PAIR ? t0 + r / 2 : t0 + r) * 16 + row4;
        if (row < a.rows_out) *reinterpret_cast<f32x4*>(o + (PAIR && (r & 1) ? a.rows_out : 0) + row) = acc[r][c];
      }
    } else if (PAIR) {  // kEpiSilu
      const float rs = a.rs[col];
#pragma unroll
      for (int p = 0; p < RU; ++p) {
        const int row = (t0 + p) * 16 + row4;
        if (row >= a.rows_out) continue;
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float g = acc[PAIR ? 2 * p : 0][c][i] * rs, u = acc[PAIR ? 2 * p + 1 : 0][c][i] * rs;
          o[i] = (g / (1.0f + expf(-g))) * u;
        }
        store_act4<bf16_t>(a.act + wide_off(a.rows_out, col, row), kWidePart, o[0], o[1], o[2], o[3]);
      }
    } else {  // kEpiLogits
      const float rs = a.rs[col];
      const int e = span_entry(sp, col);
      float* o = a.out + ((size_t)sp.seq[e] * sp.tok_pitch + (col - sp.first[e])) * a.rows_out;
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        const int row = (t0 + r) * 16 + row4;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (row + i < a.rows_out) o[row + i] = acc[r][c][i] * rs;
      }
    }
  }
}

// Sum over the workgroup (up to 16 waves), every thread receiving the total; waves added in order.
__device__ __forceinline__ float wide_block_sum(float v) {
  __shared__ float sh[16];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = 0.f;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += sh[w];
  return t;
}

// Embedding: H = E[token], X = H * g_attn of layer 0, rs.  grid = columns.
__global__ __launch_bounds__(1024) void wide_embed_kernel(const bf16_t* __restrict__ E, const int32_t* __restrict__ tokens,
                                                          const float* __restrict__ gain, int d, int V, float inv_d, float eps,
                                                          WideBuffers w, Spans sp) {
  const int col = blockIdx.x, e = span_entry(sp, col);
  const int tok = min(max(tokens[(size_t)sp.seq[e] * sp.tok_pitch + (col - sp.first[e])], 0), V - 1);  // ids outside the vocabulary are clamped
  float ss = 0.f;
  for (int j = threadIdx.x * 4; j < d; j += 4096) {
    const u32x2 raw = *reinterpret_cast<const u32x2*>(E + (size_t)tok * d + j);
    const f32x4 h = {__uint_as_float(raw.x << 16), __uint_as_float(raw.x & 0xFFFF0000u), __uint_as_float(raw.y << 16),
                     __uint_as_float(raw.y & 0xFFFF0000u)};
    *reinterpret_cast<f32x4*>(w.H + (size_t)col * d + j) = h;
    const f32x4 g = *reinterpret_cast<const f32x4*>(gain + j);
    store_act4<bf16_t>((bf16_t*)w.X + wide_off(d, col, j), kWidePart, h[0] * g[0], h[1] * g[1], h[2] * g[2], h[3] * g[3]);
    ss += (h[0] * h[0] + h[1] * h[1]) + (h[2] * h[2] + h[3] * h[3]);
  }
  ss = wide_block_sum(ss);
  if (threadIdx.x == 0) w.rs[col] = 1.0f / sqrtf(ss * inv_d + eps);
}

// Partial sums of the QKV projection -> + bias, rotary, queries and cache.  Rows are numbered as the packed matrices
// are: pair = head * hd/2 + e, first halves, then second halves.  grid = (columns, pairs / 1024), four pairs a thread.
struct WideQkvArgs {
  const float* P;
  const float* rs;
  const float* bias;  // of the layer, or null
  const float2* rope;
  float* Q;
  bf16_t *kc, *vc;  // of the layer
  int splits, cols16, Hq, Hkv, hd, max_ctx;
};
__global__ __launch_bounds__(256) void wide_qkv_finish_kernel(WideQkvArgs a, Spans sp) {
  const int half = a.hd / 2, n_pairs = (a.Hq + 2 * a.Hkv) * half;
  const int col = blockIdx.x, pair = (blockIdx.y * 256 + threadIdx.x) * 4;
  if (pair >= n_pairs) return;
  const int en = span_entry(sp, col), pos = sp.pos0[en] + (col - sp.first[en]), seq = sp.seq[en];
  const int head = pair / half, e0 = pair % half;  // four pairs stay in one head: hd/2 is a multiple of 4
  f32x4 b_lo = {0.f, 0.f, 0.f, 0.f}, b_hi = b_lo, cs0 = {1.f, 0.f, 1.f, 0.f}, cs1 = cs0;
  if (a.bias) {
    b_lo = *reinterpret_cast<const f32x4*>(a.bias + head * a.hd + e0);
    b_hi = *reinterpret_cast<const f32x4*>(a.bias + head * a.hd + e0 + half);
  }
  if (head < a.Hq + a.Hkv) {
    const f32x4* rp = reinterpret_cast<const f32x4*>(a.rope + (size_t)pos * half + e0);
    cs0 = rp[0];
    cs1 = rp[1];
  }
  const float rs = a.rs[col];
  f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
  const float* p = a.P + (size_t)col * 2 * n_pairs + pair;
  const size_t pitch = (size_t)a.cols16 * 2 * n_pairs;
#pragma unroll 4
  for (int s = 0; s < a.splits; ++s) {
    lo += *reinterpret_cast<const f32x4*>(p + s * pitch);
    hi += *reinterpret_cast<const f32x4*>(p + s * pitch + n_pairs);
  }
  const float cosv[4] = {cs0[0], cs0[2], cs1[0], cs1[2]}, sinv[4] = {cs0[1], cs0[3], cs1[1], cs1[3]};
  float x[4], y[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float v0 = lo[i] * rs + b_lo[i], v1 = hi[i] * rs + b_hi[i];
    x[i] = v0 * cosv[i] - v1 * sinv[i];
    y[i] = v1 * cosv[i] + v0 * sinv[i];
  }
  if (head < a.Hq) {
    float* qo = a.Q + (size_t)col * (a.Hq * a.hd) + head * a.hd + e0;
    store4<float>(qo, x[0], x[1], x[2], x[3]);
    store4<float>(qo + half, y[0], y[1], y[2], y[3]);
  } else {
    const bool is_k = head < a.Hq + a.Hkv;
    const int kvh = head - a.Hq - (is_k ? 0 : a.Hkv);
    bf16_t* row = (is_k ? a.kc : a.vc) + (((size_t)seq * a.Hkv + kvh) * a.max_ctx + pos) * a.hd + e0;
    store4<bf16_t>(row, x[0], x[1], x[2], x[3]);
    store4<bf16_t>(row + half, y[0], y[1], y[2], y[3]);
  }
}

// Partial sums of an O or down projection -> residual, next operand, rs.  last != 0: the last column of entry e also
// goes, as column e of a pass of n_seq columns, into the operand xh / partial sums ssp of the 16-column head launch.
// grid = columns.
struct WideResidArgs {
  const float* P;
  const float* gain;
  int splits, cols16, d, last;
  float inv_d, eps;
  bf16_t* xh;
  float* ssp;
};
__global__ __launch_bounds__(1024) void wide_resid_kernel(WideResidArgs a, WideBuffers w, Spans sp) {
  const int col = blockIdx.x, d = a.d;
  int head_col = -1;
  if (a.last) {
    const int e = span_entry(sp, col);
    if (col == sp.first[e + 1] - 1) head_col = e;
  }
  const size_t pitch = (size_t)a.cols16 * d;
  float ss = 0.f;
  for (int j = threadIdx.x * 4; j < d; j += 4096) {
    const float* p = a.P + (size_t)col * d + j;
    f32x4 h = *reinterpret_cast<const f32x4*>(w.H + (size_t)col * d + j);
    const f32x4 g = *reinterpret_cast<const f32x4*>(a.gain + j);
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int s = 0; s < a.splits; ++s) sum += *reinterpret_cast<const f32x4*>(p + s * pitch);
    h += sum;
    *reinterpret_cast<f32x4*>(w.H + (size_t)col * d + j) = h;
    store_act4<bf16_t>((bf16_t*)w.X + wide_off(d, col, j), kWidePart, h[0] * g[0], h[1] * g[1], h[2] * g[2], h[3] * g[3]);
    if (head_col >= 0)
      store_act4<bf16_t>(a.xh + xoff<bf16_t>(sp.n_seq, d, head_col, j), (size_t)kMaxCols * d, h[0] * g[0], h[1] * g[1], h[2] * g[2], h[3] * g[3]);
    ss += (h[0] * h[0] + h[1] * h[1]) + (h[2] * h[2] + h[3] * h[3]);
  }
  ss = wide_block_sum(ss);
  if (threadIdx.x == 0) w.rs[col] = 1.0f / sqrtf(ss * a.inv_d + a.eps);
  if (head_col >= 0) {
    const int ntile = d / 16;
    for (int t = threadIdx.x; t < ntile; t += 1024) a.ssp[head_col * ntile + t] = t == 0 ? ss : 0.f;
  }
}

// Argmax of the logits row of every entry's last column (lowest index on ties).  grid = entries.
__global__ __launch_bounds__(1024) void wide_argmax_kernel(const float* __restrict__ logits, int V, int32_t* tokens_out, Spans sp) {
  __shared__ float sv[16];
  __shared__ int si[16];
  const int e = blockIdx.x, tid = threadIdx.x;
  const float* row = logits + ((size_t)sp.seq[e] * sp.tok_pitch + (sp.first[e + 1] - 1 - sp.first[e])) * V;
  float bv = -INFINITY;
  int bi = 0x7FFFFFFF;
  auto take = [&](float v, int i) {
    if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
  };
  for (int j0 = tid; j0 < V; j0 += 8 * 1024) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = j0 + u * 1024 < V ? row[j0 + u * 1024] : -INFINITY;
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + u * 1024 < V) take(v[u], j0 + u * 1024);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float ov = __shfl_xor(bv, off, 64);
    const int oi = __shfl_xor(bi, off, 64);
    take(ov, oi);
  }
  if ((tid & 63) == 0) { sv[tid >> 6] = bv; si[tid >> 6] = bi; }
  __syncthreads();
  if (tid == 0) {
    for (int k = 1; k < 16; ++k) take(sv[k], si[k]);
    tokens_out[sp.seq[e]] = bi;
  }
}

// ------------------------------------------------------------------------------------------
// Launches
// ------------------------------------------------------------------------------------------
// a stage is at most 8 k-tiles of 2 KB per column tile (kWideSlack): what the last stage of the last column tile may read past the end
constexpr size_t kWideSlack = 8 * 2048;
size_t wide_operand_bytes(int cols, int K) { return (size_t)cols * K * 2 * sizeof(bf16_t) + kWideSlack; }
size_t wide_partial_bytes(const Shape& s) {
  return (size_t)kWideSplitCols * std::max(s.RQKV, s.d) * sizeof(float);
}

static int col_tiles_of(const Spans& sp) { return (sp.n + 15) / 16; }

// How a product of `tiles` row tiles (per matrix) and nkt k-tiles is cut for a pass of ct column tiles.
struct WideCut {
  int RW, CT, col_blocks, row_blocks, splits, per_split;
};
static WideCut wide_cut(int tiles, int nkt, int ct, bool pair, bool split_k) {
  WideCut c;
  c.col_blocks = (ct + 7) / 8;
  c.CT = std::max(2, (ct + c.col_blocks - 1) / c.col_blocks);
  if (c.CT == 7) c.CT = 8;  // seven tiles of one k-tile are no whole number of pieces per thread
  // Four row tiles per wave where the columns make the product compute-bound (an LDS read then serves four MFMAs); two
  // where the weight stream bounds it: twice the workgroups.
  c.RW = c.CT >= 5 ? 4 : 2;
  const int per_wg = 4 * (pair ? c.RW / 2 : c.RW);
  c.row_blocks = (tiles + per_wg - 1) / per_wg;
  c.splits = 1;
  c.per_split = nkt;
  if (split_k) {
    // as many splits as fill the CUs once, at least 8 k-tiles each, within the room for the partial sums
    const int most = std::max(1, std::min(nkt / 8, kWideSplitCols / (ct * 16)));
    const int want = std::max(1, std::min(most, cu_count() / (c.row_blocks * c.col_blocks)));
    c.per_split = (nkt + want - 1) / want;
    c.splits = (nkt + c.per_split - 1) / c.per_split;
  }
  return c;
}

template <bool PAIR>
static void launch_wide_gemm_ct(const WideArgs& a, const Spans& sp, int CT, hipStream_t st) {
  const dim3 grid(wide_grid(a.row_blocks * a.splits, a.col_blocks)), blk(kWideThreads);
  switch (CT) {  // row tiles per wave as in wide_cut
    case 2: ES_LAUNCH((wide_gemm_kernel<2, 2, 4, PAIR>), grid, blk, 0, st, a, sp); break;
    case 3: ES_LAUNCH((wide_gemm_kernel<2, 3, 2, PAIR>), grid, blk, 0, st, a, sp); break;
    case 4: ES_LAUNCH((wide_gemm_kernel<2, 4, 2, PAIR>), grid, blk, 0, st, a, sp); break;
    case 5: ES_LAUNCH((wide_gemm_kernel<4, 5, 2, PAIR>), grid, blk, 0, st, a, sp); break;
    case 6: ES_LAUNCH((wide_gemm_kernel<4, 6, 1, PAIR>), grid, blk, 0, st, a, sp); break;
    default: ES_LAUNCH((wide_gemm_kernel<4, 8, 1, PAIR>), grid, blk, 0, st, a, sp); break;
  }
}

// Fills in the cut and launches; returns the number of splits.
static int launch_wide_gemm(WideArgs a, const Spans& sp, bool pair, bool split_k, hipStream_t st) {
  a.n = sp.n;
  a.col_tiles = col_tiles_of(sp);
  const WideCut c = wide_cut((a.rows_out + 15) / 16, a.nkt, a.col_tiles, pair, split_k);
  a.col_blocks = c.col_blocks;
  a.row_blocks = c.row_blocks;
  a.splits = c.splits;
  a.per_split = c.per_split;
  if (pair) launch_wide_gemm_ct<true>(a, sp, c.CT, st);
  else launch_wide_gemm_ct<false>(a, sp, c.CT, st);
  return c.splits;
}

static WideArgs wide_args(const void* w0, const void* w1, int rows_out, int R, int K, const void* x, int epi) {
  WideArgs a;
  memset(&a, 0, sizeof a);
  a.w0 = (const u32x4*)w0;
  a.w1 = (const u32x4*)w1;
  a.rows_out = rows_out;
  a.rows = (rows_out + R - 1) / R * R;
  a.R = R;
  a.nkt = K / 32;
  a.x = (const u32x4*)x;
  a.epi = epi;
  return a;
}

void launch_wide_embed(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, const int32_t* tokens, hipStream_t st) {
  ES_LAUNCH(wide_embed_kernel, dim3(sp.n), dim3(1024), 0, st, (const bf16_t*)b.embed, tokens, b.g_attn, s.d, s.V, 1.0f / (float)s.d, s.eps,
            w, sp);
}

void launch_wide_qkv(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, hipStream_t st) {
  const int n_pairs = s.RQKV / 2;
  const size_t half_pieces = tile_stride(n_pairs, s.d, s.dtype, s.R_qkv);
  const u32x4* wl = (const u32x4*)b.wqkv + (size_t)layer * 2 * half_pieces;
  WideArgs a = wide_args(wl, wl + half_pieces, n_pairs, s.R_qkv, s.d, w.X, kEpiPartial);
  a.out = w.P;
  WideQkvArgs q;
  q.splits = launch_wide_gemm(a, sp, true, true, st);
  q.P = w.P; q.rs = w.rs;
  q.bias = s.has_bias ? b.bqkv + (size_t)layer * s.RQKV : nullptr;
  q.rope = b.rope;
  q.Q = w.Q;
  const size_t cache = (size_t)layer * s.B * s.Hkv * s.max_ctx * s.hd;
  q.kc = (bf16_t*)b.kc + cache;
  q.vc = (bf16_t*)b.vc + cache;
  q.cols16 = col_tiles_of(sp) * 16; q.Hq = s.Hq; q.Hkv = s.Hkv; q.hd = s.hd; q.max_ctx = s.max_ctx;
  ES_LAUNCH(wide_qkv_finish_kernel, dim3(sp.n, (n_pairs + 1023) / 1024), dim3(256), 0, st, q, sp);
}

void launch_wide_proj(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, bool down, const float* gain,
                      bool last, hipStream_t st) {
  const int K = down ? s.F : s.HQ;
  const u32x4* wl = (const u32x4*)(down ? b.wd : b.wo) + (size_t)layer * tile_stride(s.d, K, s.dtype);
  WideArgs a = wide_args(wl, nullptr, s.d, 16, K, down ? w.ACT : w.AO, kEpiPartial);
  a.out = w.P;
  WideResidArgs r;
  r.splits = launch_wide_gemm(a, sp, false, true, st);
  r.P = w.P; r.gain = gain; r.cols16 = col_tiles_of(sp) * 16; r.d = s.d; r.last = last ? 1 : 0;
  r.inv_d = 1.0f / (float)s.d; r.eps = s.eps;
  r.xh = (bf16_t*)b.XA;
  r.ssp = b.ssp;
  ES_LAUNCH(wide_resid_kernel, dim3(sp.n), dim3(1024), 0, st, r, w, sp);
}

void launch_wide_gateup(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, hipStream_t st) {
  const size_t off = (size_t)layer * tile_stride(s.F, s.d, s.dtype, s.R_ffn);
  WideArgs a = wide_args((const u32x4*)b.wg + off, (const u32x4*)b.wu + off, s.F, s.R_ffn, s.d, w.X, kEpiSilu);
  a.act = (bf16_t*)w.ACT;
  a.rs = w.rs;
  launch_wide_gemm(a, sp, true, false, st);
}

void launch_wide_head(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, float* logits, int32_t* tokens_out,
                      hipStream_t st) {
  WideArgs a = wide_args(b.wlm, nullptr, s.V, 16, s.d, w.X, kEpiLogits);
  a.out = logits;
  a.rs = w.rs;
  launch_wide_gemm(a, sp, false, false, st);
  ES_LAUNCH(wide_argmax_kernel, dim3(sp.n_seq), dim3(1024), 0, st, logits, s.V, tokens_out, sp);
}

}  // namespace es
