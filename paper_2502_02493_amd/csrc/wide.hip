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
//   * Stages of 2 KS k-tiles, the operand in three LDS buffers filled in the stage before (at its begin or middle), one
//     barrier per stage, in its middle; weights are requested two stages ahead, the operand one, LDS fragments a step ahead.
//   * Packed tiles are taken as they are (14 rows for gate/up, 12 pairs for QKV at the 8B shape: the spare rows of the
//     MFMA idle).  Regrouped into 16 consecutive rows a fragment straddles two packed tiles and touches half as many
//     lines again: gate/up at 24 columns, where bytes bind, 55 us against 42 (not measured where products do).
//   * Few row tiles (QKV, O, down: 256 to 384) are spread over the CUs by splitting K; the fp32 partial sums are added
//     in split order by the kernel that does what follows anyway (rotary and cache write; residual and norm operand).
// Measured at the 8B shape.  A prefill of 16 x 16 tokens (256 columns): 41.8 -> 9.4 .. 9.5 ms (eight pairs of 16-column
// passes before); gate/up 111 us a layer (137 GFLOP with both terms and the idle rows: 1.2 PFLOP/s, where a loop of
// nothing but these MFMAs on random operands runs at 2.1 and the same kernel without its weight loads takes 0.77 of the
// time), down 52, QKV 33, O 23, and 22 for the launches that finish the split ones.  4 x 6 tokens at contexts 4096 .. 32768 (24
// columns): 6.57 -> 5.2 .. 5.4 ms, memory-bound: gate/up 40 us (5.8 TB/s), down 22.
// On the way there (256 columns, mean of gate/up and QKV): LDS fragments read next to their use 141 us; read ahead 100;
// weights two stages ahead but behind branches 94; unconditional requests 76; three operand buffers the same 76; weight
// requests spread over the stage, raised wave priority around the products: no change.
#include "launch_common.hpp"

#include <math.h>
#include <string.h>

#include <algorithm>
#include <vector>

#include "../../include/easyspec_instrument.h"

namespace es {

enum { kEpiPartial = 0, kEpiSilu = 1, kEpiLogits = 2 };

struct WideArgs {
  const u32x4* w0;  // first matrix (gate; first rotary halves; or the only one)
  const u32x4* w1;  // second matrix of a pair, or null
  int rows;         // rows of one matrix
  int R, tiles;     // rows per packed tile, tiles of one matrix
  int nkt;
  int row_blocks, splits, per_split;  // k-tiles per split
  int col_blocks, col_tiles;          // column blocks of CT tiles; column tiles of the pass
  const u32x4* x;   // operand, 128 pieces per (column tile, k-tile)
  int n;            // columns
  int epi;
  float* out;       // kEpiPartial: [split][cols16][rows * matrices]; kEpiLogits: logits
  bf16_t* act;      // kEpiSilu: operand of width rows
  const float* rs;  // kEpiSilu, kEpiLogits: [cols]
};

// PAIR: the wave's row tiles are RW / 2 tiles of each of two matrices.  See the head of this file.
constexpr int kWideThreads = 512;  // four row groups x two halves of a stage's k-tiles
template <int RW, int CT, int KS, bool PAIR, bool EARLY>
__global__ __launch_bounds__(kWideThreads) void wide_gemm_kernel(WideArgs a, Spans sp) {
  constexpr int SK = 2 * KS;                               // k-tiles per stage: KS for each half
  constexpr int NB = SK * CT * 128 / kWideThreads;         // 16-byte operand pieces a thread stages per stage
  static_assert(SK * CT * 128 % kWideThreads == 0, "whole pieces per thread");
  constexpr int RU = PAIR ? RW / 2 : RW;                   // row tiles of a matrix per wave
  constexpr int kStagePieces = SK * CT * 128;
  __shared__ u32x4 xs[3 * kStagePieces];                   // three stages of [column tile][k-tile of the stage][part][lane]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), rg = wave & 3, half = wave >> 2;
  const int unit = wide_unit(blockIdx.x, a.col_blocks), cb = wide_col_block(blockIdx.x, a.col_blocks);
  if (unit >= a.row_blocks * a.splits) return;
  const int rb = unit / a.splits, split = unit % a.splits;
  const int k0 = split * a.per_split, k1 = min(a.nkt, k0 + a.per_split);
  const int t0 = wide_row_tile(rb, rg, RU), ct0 = cb * CT;
  // Addresses are a wave-uniform base plus one 32-bit lane offset each (scalar registers, not vector ones).
  const u32x4* wb[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r)
    wb[r] = (PAIR && (r & 1) ? a.w1 : a.w0) + wide_tile(PAIR ? t0 + r / 2 : t0 + r, a.tiles, a.R, a.nkt);
  const int w_stride = fragment_pieces(a.R);
  const uint32_t w_lane = lane_piece(lane, a.R), x_lane = tid & 127;
  f32x4 acc[RW][CT];
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Weights are requested two stages before they are used (they come from memory: a stage of products does not cover
  // that latency under load), operand pieces from the middle of one stage to the middle of the next (they come from the
  // L2).  All requests are unconditional (no branch for the compiler to wait at): k-tiles past the split's end repeat
  // its last one, whose lines are at hand, and have their weights replaced by zeros before they are multiplied.
  u32x4 w[3][KS][RW], xn[NB];
  auto load_w = [&](int kt, u32x4 (&d)[KS][RW]) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const size_t at = (size_t)min(wide_k_tile(kt, half, ks, KS), k1 - 1) * w_stride;
#pragma unroll
      for (int r = 0; r < RW; ++r) d[ks][r] = __builtin_nontemporal_load(wb[r] + at + w_lane);
    }
  };
  // piece j of this thread: piece i = j * threads + tid of the stage, i.e. piece i % 128 of its (column tile, k-tile)
  // fragment pair i / 128 (a missing last column tile re-reads its neighbour)
  auto load_x = [&](int kt) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int f = j * (kWideThreads / 128) + (wave >> 1), ct = min(ct0 + f / SK, a.col_tiles - 1), k = min(kt + f % SK, k1 - 1);
      xn[j] = (a.x + wide_x_piece(ct, k, a.nkt))[x_lane];
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int j = 0; j < NB; ++j) xs[buf * kStagePieces + j * kWideThreads + tid] = xn[j];
  };
  // A stage is KS * CT steps of (hi, lo) fragments, each read from LDS a step before it is used, across the end of the
  // stage too (the scheduling barriers keep the compiler from moving a read next to its use, where its latency would be
  // exposed).  A stage puts the next stage's operand into LDS; the barrier in its middle is the only one,
  // and no wave has anything to wait for at the stage's end.  Three operand buffers: what is overwritten there was
  // last read in the stage before the one before, which every wave has left when any passes the barrier between.
  // EARLY (wide_early): the operand is put there, and the one after it requested, at the stage's begin and ahead of the
  // weights: loads return in order, and a wait for the operand in mid-stage waits for the weights requested half a stage
  // before it, of which only those of this stage are needed.
  constexpr int STEPS = KS * CT, AHEAD = 1, MID = STEPS / 2;
  static_assert(3 * STEPS % (AHEAD + 1) == 0, "fragment registers return to their place after three stages");
  const u32x4* const xl = xs + lane;
  u32x4 bh[AHEAD + 1], bl[AHEAD + 1];
  auto fetch = [&](int slot, int buf, int st) {
    const u32x4* f = xl + buf * kStagePieces + wide_step_fragment(st, half, CT, KS) * 128;
    bh[slot] = f[0];
    bl[slot] = f[64];
  };
  if (k0 < k1) {
    int kt = k0;
    load_x(k0);
    load_w(k0, w[0]);
    load_w(k0 + SK, w[1]);
    put(0);
    load_x(k0 + SK);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) fetch(i, 0, i);
    // the stage in buffer I, its weights in w[I] (registers rotate by name: a copy would wait for the requests)
    auto stage = [&](auto which) {
      constexpr int I = decltype(which)::value, N = (I + 1) % 3, L = (I + 2) % 3;
      if (EARLY) {
        put(N);
        load_x(kt + 2 * SK);
      }
      load_w(kt + 2 * SK, w[L]);
      if (kt + SK > k1) {  // uniform; only the last stage
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          if (wide_k_tile(kt, half, ks, KS) >= k1) {
#pragma unroll
            for (int r = 0; r < RW; ++r) w[I][ks][r] = u32x4{0u, 0u, 0u, 0u};
          }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int st = 0; st < STEPS; ++st) {
        const int ks = st / CT, c = st % CT, j = I * STEPS + st, at = j % (AHEAD + 1), to = (j + AHEAD) % (AHEAD + 1);
        if (st == MID) {
          if (!EARLY) put(N);
          __syncthreads();
          if (!EARLY) load_x(kt + 2 * SK);
        }
        if (st + AHEAD < STEPS) fetch(to, I, st + AHEAD);
        else fetch(to, N, st + AHEAD - STEPS);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < RW; ++r) mma<bf16_t>(acc[r][c], w[I][ks][r], bh[at]);
#pragma unroll
        for (int r = 0; r < RW; ++r) mma<bf16_t>(acc[r][c], w[I][ks][r], bl[at]);
        __builtin_amdgcn_sched_barrier(0);
      }
      kt += SK;
      return kt < k1;
    };
    while (stage(std::integral_constant<int, 0>{}) && stage(std::integral_constant<int, 1>{}) && stage(std::integral_constant<int, 2>{})) {
    }
  }
  // the second half's sums onto the first's, through the LDS of the operand stages, as many column tiles at a time as fit
  {
    constexpr int PER = 3 * kStagePieces / (4 * RW * 64), CC = PER < CT ? PER : CT;
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

  const int row4 = (lane >> 4) * 4;  // of the tile
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int col = (ct0 + c) * 16 + (lane & 15);
    if (col >= a.n) continue;
    if (a.epi == kEpiPartial) {  // R and the rows are multiples of four
      const int width = PAIR ? 2 * a.rows : a.rows;
      float* o = a.out + ((size_t)split * (a.col_tiles * 16) + col) * width;
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        const int t = PAIR ? t0 + r / 2 : t0 + r, row = t * a.R + row4;
        if (row4 < a.R && row < a.rows) *reinterpret_cast<f32x4*>(o + (PAIR && (r & 1) ? a.rows : 0) + row) = acc[r][c];
      }
    } else if (PAIR) {  // kEpiSilu
      const float rs = a.rs[col];
#pragma unroll
      for (int p = 0; p < RU; ++p) {
        const int row = (t0 + p) * a.R + row4;
        float o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float g = acc[PAIR ? 2 * p : 0][c][i] * rs, u = acc[PAIR ? 2 * p + 1 : 0][c][i] * rs;
          o[i] = (g / (1.0f + expf(-g))) * u;
        }
        if (a.R == 16) {
          if (row < a.rows) store_act4<bf16_t>(a.act + wide_off(a.rows, col, row), kWidePart, o[0], o[1], o[2], o[3]);
        } else if (((a.R | a.rows) & 1) == 0) {
          // pairs of rows lie in one tile and begin at an even k: half of the stores (gate/up and QKV at 256 columns 77.6 -> 76.4 us a launch)
#pragma unroll
          for (int i = 0; i < 4; i += 2)
            if (row4 + i < a.R && row + i < a.rows) store_act2<bf16_t>(a.act + wide_off(a.rows, col, row + i), kWidePart, o[i], o[i + 1]);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (row4 + i < a.R && row + i < a.rows) store_act1<bf16_t>(a.act + wide_off(a.rows, col, row + i), kWidePart, o[i]);
        }
      }
    } else {  // kEpiLogits
      const float rs = a.rs[col];
      const int e = span_entry(sp, col);
      float* o = a.out + ((size_t)sp.seq[e] * sp.tok_pitch + (col - sp.first[e])) * a.rows;
#pragma unroll
      for (int r = 0; r < RW; ++r) {
        const int row = (t0 + r) * a.R + row4;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (row + i < a.rows) o[row + i] = acc[r][c][i] * rs;
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
size_t wide_operand_bytes(int cols, int K) { return (size_t)cols * K * 2 * sizeof(bf16_t); }
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
  // Up to 64 columns the weight stream is what bounds the product: two row tiles per wave, the most workgroups.  More:
  // four row tiles per wave, so that an LDS read serves four MFMAs, and as many column blocks (on one XCD, reading the
  // same weights) as make the launch's rounds of one workgroup per CU, times the column tiles of each, the least.
  // gate/up and all, 8 layers, one column block against two: 8B shape (128 row blocks) 96 columns 1643 -> 1494 us, 128
  // columns 1927 -> 1590; Qwen2-7B shape (148) 1584 -> 1763 and 1784 -> 1889, hence the rule.  Split products fill the
  // CUs whatever the blocks.
  auto tiles_of = [&](int blocks) {
    const int t = std::max(2, (ct + blocks - 1) / blocks);
    return t == 7 ? 8 : t;  // seven tiles of one k-tile are no whole number of pieces per thread
  };
  c.RW = ct > 4 ? 4 : 2;
  c.col_blocks = ct > 4 && split_k ? 2 : (ct + 7) / 8;
  if (ct > 4 && !split_k) {
    const int rows = (tiles + (pair ? 7 : 15)) / (pair ? 8 : 16);
    auto cost = [&](int blocks) { return (rows * blocks + cu_count() - 1) / cu_count() * tiles_of(blocks); };
    for (int n = c.col_blocks + 1; n <= 4 && tiles_of(n) >= 3; ++n)
      if (cost(n) < cost(c.col_blocks)) c.col_blocks = n;
  }
  c.CT = tiles_of(c.col_blocks);
  const int per_wg = 4 * (pair ? c.RW / 2 : c.RW);
  c.row_blocks = (tiles + per_wg - 1) / per_wg;
  c.splits = 1;
  c.per_split = nkt;
  if (split_k) {
    // as many splits as fill the CUs once, at least 8 k-tiles each, within the room for the partial sums
    const int most = std::max(1, std::min(nkt / 8, kWideSplitCols / (ct * 16)));
    const int want = std::max(1, std::min(most, cu_count() / (c.row_blocks * c.col_blocks)));
    c.per_split = ((nkt + want - 1) / want + 1) & ~1;  // whole stages (of two k-tiles or more) if K allows
    c.splits = (nkt + c.per_split - 1) / c.per_split;
  }
  return c;
}

// the (RW, CT) there are kernels for: every cut that wide_cut makes
#define WIDE_KERNELS(X) X(2, 2) X(2, 3) X(2, 4) X(4, 3) X(4, 4) X(4, 5) X(4, 6) X(4, 8)

// Where a stage handles its operand before its weights: blocks of six and eight column tiles that share their weights with
// another block.  us, without and with: all products of the 8B shape in two blocks, 8 layers, 176 columns (six tiles) 1733 -> 1724,
// 248 columns (eight) 2132 -> 2089; gate/up alone at 256 columns 112 .. 123 -> 108 .. 114 a launch by box, down 51 .. 57 -> 50 .. 53.
// Shorter stages have no room for it (64 columns, four tiles: gate/up 49 -> 53), and a block of its own waits for weights that come
// from memory (gate/up of the Qwen2-7B shape at 84 columns, six tiles in one block, 8 layers: 1437 -> 1454 with it; heads of eight
// tiles in one block: no difference).
static bool wide_early(const WideCut& c) { return c.CT >= 6 && c.col_blocks > 1; }

template <bool PAIR>
static void launch_wide_gemm_ct(const WideArgs& a, const Spans& sp, const WideCut& c, hipStream_t st) {
  const dim3 grid(wide_grid(a.row_blocks * a.splits, a.col_blocks)), blk(kWideThreads);
#define WIDE_LAUNCH(RW, CT, EARLY) ES_LAUNCH((wide_gemm_kernel<RW, CT, wide_stage_tiles(CT), PAIR, EARLY>), grid, blk, 0, st, a, sp)
#define WIDE_CASE(RW, CT)                               \
  case RW * 10 + CT:                                    \
    if (wide_early(c)) WIDE_LAUNCH(RW, CT, (CT >= 6));  \
    else WIDE_LAUNCH(RW, CT, false);                    \
    break;
  switch (c.RW * 10 + c.CT) { WIDE_KERNELS(WIDE_CASE) }
#undef WIDE_CASE
#undef WIDE_LAUNCH
}

// What a wide product is of: rows of one matrix, rows per packed tile, K; two matrices side by side; partial sums per split.
struct WideShape {
  int rows, R, K;
  bool pair, split_k;
};
static WideShape wide_shape(const Shape& s, int op) {
  switch (op) {
    case EASYSPEC_OP_QKV: return {s.RQKV / 2, s.R_qkv, s.d, true, true};
    case EASYSPEC_OP_OPROJ: return {s.d, 16, s.HQ, false, true};
    case EASYSPEC_OP_GATEUP: return {s.F, s.R_ffn, s.d, true, false};
    case EASYSPEC_OP_DOWN: return {s.d, 16, s.F, false, true};
    default: return {s.V, 16, s.d, false, false};  // EASYSPEC_OP_HEAD
  }
}

// Fills in the cut and launches; returns the number of splits.
static int launch_wide_gemm(const Shape& s, int op, const void* w0, const void* w1, const void* x, int epi, void* out, const float* rs,
                            const Spans& sp, hipStream_t st) {
  const WideShape w = wide_shape(s, op);
  WideArgs a;
  memset(&a, 0, sizeof a);
  a.w0 = (const u32x4*)w0;
  a.w1 = (const u32x4*)w1;
  a.rows = w.rows;
  a.R = w.R;
  a.tiles = ceil_div(w.rows, w.R);
  a.nkt = w.K / 32;
  a.x = (const u32x4*)x;
  a.epi = epi;
  if (epi == kEpiSilu) a.act = (bf16_t*)out;
  else a.out = (float*)out;
  a.rs = rs;
  a.n = sp.n;
  a.col_tiles = col_tiles_of(sp);
  const WideCut c = wide_cut(a.tiles, a.nkt, a.col_tiles, w.pair, w.split_k);
  a.col_blocks = c.col_blocks;
  a.row_blocks = c.row_blocks;
  a.splits = c.splits;
  a.per_split = c.per_split;
  if (w.pair) launch_wide_gemm_ct<true>(a, sp, c, st);
  else launch_wide_gemm_ct<false>(a, sp, c, st);
  return c.splits;
}

// Host model of one product: every workgroup, wave and stage computes, through the kernel's own index functions, the weight
// and operand pieces it loads, the LDS fragments it multiplies and the partial sums it stores.
int wide_walk(const Shape& s, int op, int n_cols, WideWalk* r) {
  memset(r, 0, sizeof *r);
  const WideShape w = wide_shape(s, op);
  const int tiles = ceil_div(w.rows, w.R), nkt = w.K / 32, col_tiles = (n_cols + 15) / 16, n_mat = w.pair ? 2 : 1;
  const WideCut c = wide_cut(tiles, nkt, col_tiles, w.pair, w.split_k);
  const int KS = wide_stage_tiles(c.CT), per_wave = w.pair ? c.RW / 2 : c.RW, width = w.rows * n_mat;
  r->RW = c.RW; r->CT = c.CT; r->KS = KS;
  r->col_blocks = c.col_blocks; r->row_blocks = c.row_blocks; r->splits = c.splits; r->per_split = c.per_split;
  r->grid = wide_grid(c.row_blocks * c.splits, c.col_blocks);
  r->w_pieces = (long long)tiles * row_tile_pieces(nkt, w.R);
  r->x_pieces = (long long)wide_x_piece(col_tiles, 0, nkt);
  r->products = (long long)n_mat * tiles * nkt * col_tiles;
  r->out_room = w.split_k ? (long long)(wide_partial_bytes(s) / sizeof(float)) : 0;
#define WIDE_CASE(RW_, CT_) r->kernel |= c.RW == RW_ && c.CT == CT_;
  WIDE_KERNELS(WIDE_CASE)
#undef WIDE_CASE
  int most_lane = 0;
  for (int lane = 0; lane < 64; ++lane) most_lane = std::max(most_lane, (int)lane_piece(lane, w.R));
  for (int half = 0; half < 2; ++half)
    for (int st = 0; st < KS * c.CT; ++st) {
      const int f = wide_step_fragment(st, half, c.CT, KS);
      r->misplaced += f / (2 * KS) != st % c.CT || f % (2 * KS) != wide_k_tile(0, half, st / c.CT, KS);
    }
  std::vector<unsigned char> seen((size_t)r->products, 0);
  for (int id = 0; id < r->grid; ++id) {
    const int unit = wide_unit(id, c.col_blocks), ct0 = wide_col_block(id, c.col_blocks) * c.CT;
    if (unit >= c.row_blocks * c.splits) continue;
    const int rb = unit / c.splits, split = unit % c.splits, k0 = split * c.per_split, k1 = std::min(nkt, k0 + c.per_split);
    if (k0 >= k1) ++r->empty_splits;
    for (int rg = 0; rg < 4; ++rg)
      for (int i = 0; i < c.RW; ++i) {
        const int m = w.pair ? i & 1 : 0, t = wide_row_tile(rb, rg, per_wave) + (w.pair ? i / 2 : i);
        const long long base = (long long)wide_tile(t, tiles, w.R, nkt);
        for (int kt = k0; kt < k1; kt += 2 * KS)
          for (int half = 0; half < 2; ++half)
            for (int ks = 0; ks < KS; ++ks) {
              const int k = wide_k_tile(kt, half, ks, KS), at = std::min(k, k1 - 1);
              const long long piece = base + (long long)at * fragment_pieces(w.R) + most_lane;
              r->w_max = std::max(r->w_max, piece);
              r->w_out_of_range += piece - most_lane < 0 || piece >= r->w_pieces;
              for (int ct = ct0; ct < ct0 + c.CT; ++ct) {
                const long long x = (long long)wide_x_piece(std::min(ct, col_tiles - 1), at, nkt) + 127;
                r->x_max = std::max(r->x_max, x);
                r->x_out_of_range += x >= r->x_pieces;
                if (k >= k1 || t >= tiles || ct >= col_tiles) continue;  // zeroed, a repeat of the last tile, not stored
                unsigned char& n = seen[(((size_t)m * tiles + t) * nkt + k) * col_tiles + ct];
                if (n < 255) ++n;
              }
            }
        const int col = std::min((ct0 + c.CT) * 16, n_cols) - 1, row = std::min((t + 1) * w.R, w.rows) - 1;
        if (w.split_k && t < tiles)
          r->out_max = std::max(r->out_max, ((long long)split * (col_tiles * 16) + col) * width + (long long)m * w.rows + row);
      }
  }
  for (unsigned char n : seen) {
    r->missed += n == 0;
    r->repeated += n > 1;
  }
  return 0;
}

void launch_wide_embed(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, const int32_t* tokens, hipStream_t st) {
  ES_LAUNCH(wide_embed_kernel, dim3(sp.n), dim3(1024), 0, st, (const bf16_t*)b.embed, tokens, b.g_attn, s.d, s.V, 1.0f / (float)s.d, s.eps,
            w, sp);
}

void launch_wide_qkv(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, hipStream_t st) {
  const int n_pairs = s.RQKV / 2;
  const size_t half_pieces = tile_stride(n_pairs, s.d, s.dtype, s.R_qkv);
  const u32x4* wl = (const u32x4*)b.wqkv + (size_t)layer * 2 * half_pieces;
  WideQkvArgs q;
  q.splits = launch_wide_gemm(s, EASYSPEC_OP_QKV, wl, wl + half_pieces, w.X, kEpiPartial, w.P, nullptr, sp, st);
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
  WideResidArgs r;
  r.splits = launch_wide_gemm(s, down ? EASYSPEC_OP_DOWN : EASYSPEC_OP_OPROJ, wl, nullptr, down ? w.ACT : w.AO, kEpiPartial, w.P, nullptr, sp, st);
  r.P = w.P; r.gain = gain; r.cols16 = col_tiles_of(sp) * 16; r.d = s.d; r.last = last ? 1 : 0;
  r.inv_d = 1.0f / (float)s.d; r.eps = s.eps;
  r.xh = (bf16_t*)b.XA;
  r.ssp = b.ssp;
  ES_LAUNCH(wide_resid_kernel, dim3(sp.n), dim3(1024), 0, st, r, w, sp);
}

void launch_wide_gateup(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, hipStream_t st) {
  const size_t off = (size_t)layer * tile_stride(s.F, s.d, s.dtype, s.R_ffn);
  launch_wide_gemm(s, EASYSPEC_OP_GATEUP, (const u32x4*)b.wg + off, (const u32x4*)b.wu + off, w.X, kEpiSilu, w.ACT, w.rs, sp, st);
}

void launch_wide_head(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, float* logits, int32_t* tokens_out,
                      hipStream_t st) {
  launch_wide_gemm(s, EASYSPEC_OP_HEAD, b.wlm, nullptr, w.X, kEpiLogits, logits, w.rs, sp, st);
  ES_LAUNCH(wide_argmax_kernel, dim3(sp.n_seq), dim3(1024), 0, st, logits, s.V, tokens_out, sp);
}

}  // namespace es
