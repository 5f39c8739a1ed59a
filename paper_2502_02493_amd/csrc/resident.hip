// Resident passes (gfx950): a whole forward pass of a small model as ONE launch.
//
// A small model's pass is a chain of some twenty dependent kernels of a few dozen workgroups each, and what bounds it is
// not bytes or arithmetic but the chain: a launch of any size takes 4 to 6 us here (an empty one 2.5), and the host needs
// about as long to enqueue it.  Here the units of all those kernels (row tiles of a projection, heads of an attention) are
// worked through by workgroups that stay, and what one unit leaves for another goes through memory as tagged values:
//   * A value travels as an 8-byte granule, the float and the number of the pass (its epoch), stored and loaded by single
//     device-scope accesses.  A reader loads the granules it needs until all carry this pass's epoch: data and readiness
//     arrive in one trip, with no fence, no flag and no barrier over the grid (such a barrier alone costs 1.7 us with 64
//     workgroups, 2.8 to 3.2 with 256).  Every granule of a pass has a place of its own, so nothing is overwritten inside a
//     pass; from one pass to the next the kernel boundary orders.
//   * Units are numbered in the order of the launches they replace and handed out by a ticket counter.  A unit only waits
//     for units of smaller numbers, and those are done or in the hands of workgroups that run: the pass advances however few
//     of its workgroups the device has room for, whatever else runs beside it.  (Every wait also ends after a bounded
//     number of polls; a pass that gave up sets a host word, which the context's entry points look at.)
//   * A workgroup holds one ticket at a time and there are twice as many as the MLP or the head has units (at most one per CU),
//     so that the next phases' units are already waiting, their weights on the way into registers, when their operands
//     arrive.  Phases with more units than that (stacked QKV and O, many heads, large vocabularies) go in rounds.  A model is
//     "small" if a wave's share of a row tile fits there in one go (resident_model).
//   * The operand is put into LDS once per workgroup.  Up to four columns of an fp32 model are multiplied on the vector
//     ALUs (an fp32 MFMA takes 32 cycles for its 16 columns, used or not), everything else on the matrix cores.
// What is left is latency: of the 2.7 us a phase takes (one column, 256 wide), 0.4 are the products and their sum over the
// waves, 0.8 the tile's end in wave 0, the rest the trip of a store to the other XCDs and the poll that finds it.  So the code
// is straight-line: a request under a branch is waited for where the branch ends (a unit's start 1.4 -> 1.1 us, of a down
// projection 3.6 -> 2.3), an LDS read under one stands alone (products 0.9 -> 0.4), and a wave's lanes take an element of the
// tile each instead of four (end of a tile 1.5 -> 0.8).  In the attention the steps of all heads go side by side, the slots of
// this pass are part of the last run instead of a batch of their own, and with seven or eight heads half of the waves take half
// of them: 5.5 -> 3.2 us at 61 slots and seven heads.
// Where it is taken: resident_pass.  us a call, launches and resident: draft step of the 256-wide fp32 model of 4 layers 98 -> 56; an iteration of the 448-wide
// one of 5 layers (calibration of 5 tokens and three steps, vocabulary of 1000) 594 -> 380.
#include "launch_common.hpp"

#include <math.h>
#include <string.h>

#include <algorithm>

namespace es {

typedef unsigned long long granule_t;  // low half: the float, high half: the epoch

constexpr int kResThreads = 512, kResWaves = 8;
constexpr int kResRT2 = 6, kResRT1 = 12;  // k-tiles per wave that fit the registers: two row tiles side by side, one
constexpr int kResTiles = 96;             // row tiles of 16 of the model width (partial sums of squares in LDS)
constexpr int kResRedPitch = 20;          // floats per column of 16 rows in the reduction buffer (bank spread)
constexpr int kResPolls = 1 << 22;        // about a microsecond each

struct ResidentArgs {
  const u32x4 *wqkv, *wo, *wg, *wu, *wd, *wlm;
  const void* embed;
  const float *bqkv, *g_attn, *g_mlp, *g_final;
  const float2* rope;
  const float* g_any;  // as many floats as the widest operand
  void *kc, *vc;
  float* H;
  const int32_t* tokens;
  float* logits;
  int32_t* tokens_out;
  ResidentCtl* ctl;
  granule_t* ll;
  uint32_t* failed;
  int L, d, Hq, Hkv, F, V, HQ, RQKV, B, max_ctx, n_sets;
  float inv_d, eps, scale;
  uint8_t bounds[kResMaxLayers + 1];
  uint8_t col0[kMaxCols];  // first column of the column's sequence
};

// Places of the granules: per layer [16 columns][...] of q | k | v, attention output, residual before the MLP (its partial
// sums of squares behind every column's values), Attnoutput, MLP activations, residual after the MLP; then the argmax candidates.
struct ResidentMap {
  int qkv, ao, h1, a, act, h2, layer, hp;
};
ES_HD ResidentMap resident_map(int d, int HQ, int RQKV, int F) {
  ResidentMap m;
  m.hp = d + d / 16;
  m.qkv = 0;
  m.ao = m.qkv + kMaxCols * RQKV;
  m.h1 = m.ao + kMaxCols * HQ;
  m.a = m.h1 + kMaxCols * m.hp;
  m.act = m.a + kMaxCols * d;
  m.h2 = m.act + kMaxCols * F;
  m.layer = m.h2 + kMaxCols * m.hp;
  return m;
}

struct Poll {
  uint32_t epoch;
  int left;  // polls this wave may still make in vain (wave-uniform)
  uint32_t* failed;
  // after a poll: go on?  (all lanes have what they need, or the wave has waited too long)
  __device__ __forceinline__ bool done(bool ok) {
    if (__all(ok) || left <= 0) return true;
    if (--left == 0) __hip_atomic_store(failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __builtin_amdgcn_s_sleep(1);
    return left <= 0;
  }
};

__device__ __forceinline__ void ll_put(granule_t* p, float v, uint32_t epoch) {
  __hip_atomic_store(p, (granule_t)__float_as_uint(v) | ((granule_t)epoch << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// a uniform base and a 32-bit offset
__device__ __forceinline__ granule_t ll_load(const granule_t* base, int at) {
  return __hip_atomic_load(reinterpret_cast<granule_t*>(reinterpret_cast<char*>(const_cast<granule_t*>(base)) + (uint32_t)at * 8u), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// N granules of every lane; issue() requests them, finish() returns when all of the wave's carry the epoch.
template <int N>
struct Granules {
  granule_t v[N];
  __device__ __forceinline__ void issue(const granule_t* base, const int (&at)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = ll_load(base, at[i]);
  }
  __device__ __forceinline__ void finish(const granule_t* base, const int (&at)[N], Poll& w, float (&out)[N]) {
    while (true) {
      bool ok = true;
#pragma unroll
      for (int i = 0; i < N; ++i) ok = ok && (uint32_t)(v[i] >> 32) == w.epoch;
      if (w.done(ok)) break;
      issue(base, at);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = __uint_as_float((uint32_t)v[i]);
  }
};

// Sums without a trip through LDS: over the lanes l, l ^ 16, l ^ 32, l ^ 48 ...
__device__ __forceinline__ float quarter_sum(float v) {
  const uint32_t a = __float_as_uint(v);
  const auto h = __builtin_amdgcn_permlane32_swap(a, a, false, false);
  const uint32_t b = __float_as_uint(__uint_as_float(h[0]) + __uint_as_float(h[1]));
  const auto q = __builtin_amdgcn_permlane16_swap(b, b, false, false);
  return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}
// ... and of N = 16 or 32 consecutive lanes: sum, maximum
template <int N>
__device__ __forceinline__ float lanes_sum(float v) {
  v = group_sum<16>(v);
  if (N == 32) {
    const uint32_t a = __float_as_uint(v);
    const auto q = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    v = __uint_as_float(q[0]) + __uint_as_float(q[1]);
  }
  return v;
}
template <int N>
__device__ __forceinline__ float lanes_max(float v) {
  v = fmaxf(v, dpp_f32<0xB1>(v));
  v = fmaxf(v, dpp_f32<0x4E>(v));
  v = fmaxf(v, dpp_f32<0x141>(v));
  v = fmaxf(v, dpp_f32<0x140>(v));
  if (N == 32) {
    const uint32_t a = __float_as_uint(v);
    const auto q = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    v = fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
  }
  return v;
}

template <typename T>
__device__ __forceinline__ float load_elem(const void* p, size_t i) {
  return load1<T>(reinterpret_cast<const T*>(p) + i);
}

// x[col][k] into the LDS operand: pieces of EPL consecutive k, [k / EPL][column], per part
template <typename T>
__device__ __forceinline__ void put_operand(void* xs, int n, int K, int col, int k, float x);
template <>
__device__ __forceinline__ void put_operand<float>(void* xs, int n, int, int col, int k, float x) {
  reinterpret_cast<float*>(xs)[((k >> 2) * n + col) * 4 + (k & 3)] = x;
}
template <>
__device__ __forceinline__ void put_operand<bf16_t>(void* xs, int n, int K, int col, int k, float x) {
  uint16_t* p = reinterpret_cast<uint16_t*>(xs) + ((k >> 3) * n + col) * 8 + (k & 7);
  const uint32_t hi = float_to_bf16_bits(x);
  p[0] = (uint16_t)hi;
  p[K * n] = (uint16_t)float_to_bf16_bits(x - bf16_bits_to_float(hi));
}

// Where a product's operand comes from.
struct Operand {
  const granule_t* x;  // [column][pitch], or null: the embedding rows
  int pitch, K;
  const float* gain;   // of the norm in front, or null: taken as it is
  const float* some;   // any array of K floats
};

struct ResidentShared {
  float red[kResWaves * 2 * kMaxCols * kResRedPitch];
  float ss[kMaxCols * kResTiles];
  int tok[kMaxCols];
  int next;
};

// Granules tid + first + i * threads (i < N) of the operand into LDS, times the gain of the norm in front; normed ones with
// their K / 16 partial sums of squares.  Straight-line: a request under a branch would be waited for at the branch's end.
template <typename T, int N>
__device__ __forceinline__ void stage_part(const Operand& o, int row, int total, float inv_row, int first, int tid, int n, Poll& w, ResidentShared& sh,
                                           void* xs) {
  int at[N], col[N], k[N];
  float g[N], x[N];
  Granules<N> gr;
  const float* const gain = o.gain ? o.gain : o.some;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int f = min(first + tid + i * kResThreads, total - 1);
    col[i] = (int)(((float)f + 0.5f) * inv_row);  // f / row: off by less than half a step (f < 2^15, row < 2^12)
    k[i] = f - col[i] * row;
    at[i] = col[i] * o.pitch + k[i];
    g[i] = gain[min(k[i], o.K - 1)];
  }
  gr.issue(o.x, at);
  gr.finish(o.x, at, w, x);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (first + tid + i * kResThreads < total) {
      if (k[i] < o.K) put_operand<T>(xs, n, o.K, col[i], k[i], o.gain ? x[i] * g[i] : x[i]);
      else sh.ss[col[i] * kResTiles + k[i] - o.K] = x[i];
    }
  }
}

template <typename T>
__device__ __forceinline__ void stage(const ResidentArgs& a, const Operand& o, int tid, int n, Poll& w, ResidentShared& sh, void* xs) {
  if (o.x) {
    const int row = o.gain ? o.K + o.K / 16 : o.K, total = row * n;
    const float inv_row = 1.0f / (float)row;
    if (total <= kResThreads) {
      stage_part<T, 1>(o, row, total, inv_row, 0, tid, n, w, sh, xs);
    } else if (total <= 4 * kResThreads) {
      stage_part<T, 4>(o, row, total, inv_row, 0, tid, n, w, sh, xs);
    } else {
#pragma unroll 1
      for (int first = 0; first < total; first += 8 * kResThreads) stage_part<T, 8>(o, row, total, inv_row, first, tid, n, w, sh, xs);
    }
    return;
  }
  // embedding rows: whole groups of 16 lanes share a column and a group of 16 k
  const float inv_k = 1.0f / (float)o.K;
  for (int f = tid; f < o.K * n; f += kResThreads) {
    const int col = (int)(((float)f + 0.5f) * inv_k), k = f - col * o.K;
    const float h = load_elem<T>(a.embed, (size_t)sh.tok[col] * o.K + k);
    put_operand<T>(xs, n, o.K, col, k, h * o.gain[k]);
    const float s = group_sum<16>(h * h);
    if ((k & 15) == 0) sh.ss[col * kResTiles + (k >> 4)] = s;
  }
}

// One unit of a weight contraction: the partial sums of every wave into LDS.  Two row tiles side by side (w0, w1: their
// first pieces; k-tiles 64 pieces apart), or one whose k-tiles are dealt to the same two accumulators (w1 == null).  J:
// k-tiles per wave and accumulator.
template <typename T, int J>
__device__ __forceinline__ void resident_gemm(const ResidentArgs& a, int tid, int n, const u32x4* w0, const u32x4* w1, int nkt, const Operand& o,
                                              Poll& w, ResidentShared& sh, void* xs) {
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool pair = w1 != nullptr;
  const int step = pair ? kResWaves : 2 * kResWaves, other = pair ? 0 : kResWaves;
  auto tile = [&](int j, int r) { return wave + step * j + other * r; };  // this wave's k-tile j of accumulator r
  const u32x4* const ws[2] = {w0 + lane, (pair ? w1 : w0) + lane};
  u32x4 wr[J][2];
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int r = 0; r < 2; ++r) wr[j][r] = __builtin_nontemporal_load(ws[r] + (size_t)min(tile(j, r), nkt - 1) * 64);
  stage<T>(a, o, tid, n, w, sh, xs);
  __syncthreads();
  const int kg = lane >> 4, col = lane & 15;
  float* const red = sh.red + wave * 2 * (kMaxCols * kResRedPitch);
  if (std::is_same<T, float>::value && n <= 4) {
    const f32x4* const xf = reinterpret_cast<const f32x4*>(xs);
#pragma unroll 1
    for (int q = 0; q < n; ++q) {
      f32x4 x[J][2];
#pragma unroll
      for (int j = 0; j < J; ++j)
#pragma unroll
        for (int r = 0; r < 2; ++r) x[j][r] = xf[(min(tile(j, r), nkt - 1) * 4 + kg) * n + q];
      float s[2] = {0.f, 0.f};
#pragma unroll
      for (int j = 0; j < J; ++j)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const float p = __uint_as_float(wr[j][r].x) * x[j][r][0] + __uint_as_float(wr[j][r].y) * x[j][r][1] +
                          __uint_as_float(wr[j][r].z) * x[j][r][2] + __uint_as_float(wr[j][r].w) * x[j][r][3];
          s[r] += tile(j, r) < nkt ? p : 0.f;
        }
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const float v = quarter_sum(s[r]);
        if (lane < 16) red[(r * kMaxCols + q) * kResRedPitch + lane] = v;
      }
    }
  } else {
    f32x4 m[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    const u32x4* const xp = reinterpret_cast<const u32x4*>(xs) + min(col, n - 1);
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int p = (min(tile(j, r), nkt - 1) * 4 + kg) * n;
        const u32x4 hi = xp[p], lo = Tr<T>::PARTS == 2 ? xp[p + nkt * 4 * n] : hi;
        if (tile(j, r) < nkt) {
          mma<T>(m[r], wr[j][r], hi);
          if (Tr<T>::PARTS == 2) mma<T>(m[r], wr[j][r], lo);
        }
      }
    if (col < n) {
#pragma unroll
      for (int r = 0; r < 2; ++r) *reinterpret_cast<f32x4*>(red + (r * kMaxCols + col) * kResRedPitch + 4 * kg) = m[r];
    }
  }
  __syncthreads();
}

enum { kPhQkv, kPhAttn, kPhO, kPhGateUp, kPhDown, kPhHead, kPhArgmax, kPhEnd };

// POLLS: how many polls a wave may make in vain over the whole pass.  A constant: as an argument it costs a pass 0.6 .. 1 us.
template <typename T, int G, int POLLS = kResPolls>
__global__ __launch_bounds__(kResThreads) void resident_kernel(ResidentArgs a, Cols c) {
  constexpr int HD = 64, EPL = Tr<T>::EPL, KT = Tr<T>::KT, LPS = HD / EPL, SPW = 64 / LPS;
  __shared__ ResidentShared sh;
  void* const xs = dyn_red;
  const int d = a.d, ntile = d / 16;
  const ResidentMap map = resident_map(d, a.HQ, a.RQKV, a.F);
  const int nkt_d = d / KT, nkt_q = a.HQ / KT, nkt_f = a.F / KT;
  const int n_pairs = a.RQKV / 2, u_qkv = ceil_div(n_pairs, 16), u_f = ceil_div(a.F, 16), u_v = ceil_div(a.V, 16);
  granule_t* const cand = a.ll + (size_t)a.L * map.layer;  // [column][row tile of the head][value, index]
  Poll w;
  w.epoch = __hip_atomic_load(&a.ctl->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  w.left = POLLS;
  w.failed = a.failed;
  // A workgroup asks for its next unit when the sums of this one are on their way (wave 1; wave 0 finishes the unit).
  auto ask_next = [&] {
    if (threadIdx.x == 64) sh.next = (int)__hip_atomic_fetch_add(&a.ctl->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  ask_next();
  if ((int)threadIdx.x < c.n) sh.tok[threadIdx.x] = min(max(a.tokens[c.tok_idx[threadIdx.x]], 0), a.V - 1);  // ids outside the vocabulary are clamped
  __syncthreads();
  int ticket = __builtin_amdgcn_readfirstlane(sh.next);

  int set = 0, lo = 0, hi = a.bounds[1], layer = 0, ph = kPhQkv, first = 0;
  while (true) {
    // opaque in every round: what a unit derives from these is computed in it, not kept in registers over all others
    int n = c.n, tid = threadIdx.x;
    asm volatile("" : "+s"(n), "+v"(tid));
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), col = lane & 15, kg = lane >> 4;
    int units;
    while (true) {
      switch (ph) {
        case kPhQkv: units = (hi - lo) * u_qkv; break;
        case kPhAttn: units = (hi - lo) * n * a.Hkv; break;
        case kPhO: units = (hi - lo) * ntile; break;
        case kPhGateUp: units = u_f; break;
        case kPhDown: units = ntile; break;
        case kPhHead: units = u_v; break;
        case kPhArgmax: units = n; break;
        default: units = INT32_MAX;
      }
      if (ph == kPhEnd || ticket < first + units) break;
      first += units;
      if (ph == kPhDown && layer + 1 < hi) {
        ph = kPhGateUp;
        ++layer;
      } else if (ph == kPhDown && set + 1 < a.n_sets) {
        ph = kPhQkv;
        ++set;
        lo = layer = hi;
        hi = a.bounds[set + 1];
      } else {
        ++ph;
      }
    }
    if (ph == kPhEnd) break;
    const int unit = ticket - first;
    if (ph != kPhAttn && ph != kPhArgmax) {
      const bool qkv = ph == kPhQkv, gateup = ph == kPhGateUp, oproj = ph == kPhO, down = ph == kPhDown, head = ph == kPhHead;
      const int per = qkv ? u_qkv : ntile;  // QKV and O projections: the layers of the set one after the other
      const int li = qkv || oproj ? unit / per : 0, t = unit - li * per, l = qkv || oproj ? lo + li : layer;
      granule_t* const lay = a.ll + (size_t)l * map.layer;
      const granule_t* const before = lay - (size_t)(l - lo + 1) * map.layer + map.h2;  // the set's input (lo > 0)
      const int nkt = oproj ? nkt_q : down ? nkt_f : nkt_d;
      const size_t tile = row_tile_pieces(nkt, 16);
      const u32x4 *w0, *w1 = nullptr;
      Operand o;
      o.K = oproj ? a.HQ : down ? a.F : d;
      o.gain = nullptr;
      if (qkv) {
        w0 = a.wqkv + ((size_t)l * 2 * per + t) * tile;
        w1 = w0 + per * tile;
        o.x = lo ? before : nullptr;
        o.gain = a.g_attn + (size_t)l * d;
      } else if (gateup) {
        w0 = a.wg + ((size_t)l * u_f + t) * tile;
        w1 = a.wu + ((size_t)l * u_f + t) * tile;
        o.x = lay + map.h1;
        o.gain = a.g_mlp + (size_t)l * d;
      } else if (head) {
        w0 = a.wlm + (size_t)t * tile;
        o.x = lay + map.h2;
        o.gain = a.g_final;
      } else {
        w0 = (oproj ? a.wo : a.wd) + ((size_t)l * ntile + t) * tile;
        o.x = lay + (oproj ? map.ao : map.act);
      }
      o.pitch = o.gain ? map.hp : o.K;
      o.some = a.g_any;
      // Wave 0 finishes the tile, an element per lane: row lane % 16 of columns lane / 16 + 4 p.  What it needs besides the
      // sums is requested first: bias and rotation of a QKV tile, the residual an O or down tile adds to and the next
      // layer's Attnoutput (both were sent before the operand was).  Unconditional requests, of something that is there.
      const int row = t * 16 + col;  // col: here the lane's row of the tile
      const int hd_ = min(row, n_pairs - 1) / (HD / 2), e0 = row % (HD / 2);
      const bool is_q = hd_ < a.Hq, is_k = !is_q && hd_ < a.Hq + a.Hkv;
      const bool resid = (oproj && li == 0) || down, add_a = down && l + 1 < hi, h_sent = resid && (down || lo > 0);
      const granule_t* const hsrc = h_sent ? (down ? lay + map.h1 : before) : o.x ? o.x : a.ll;
      const granule_t* const asrc = add_a ? lay + map.layer + map.a : hsrc;  // of layer l + 1
      float b_lo = 0.f, b_hi = 0.f;
      float2 cs[4];
      float hv[4], av[4];
      int hat[4], aat[4];
      Granules<4> hg, ag;
      if (wave == 0) {
        if (qkv) {
          if (a.bqkv) {
            b_lo = a.bqkv[(size_t)l * a.RQKV + hd_ * HD + e0];
            b_hi = a.bqkv[(size_t)l * a.RQKV + hd_ * HD + e0 + HD / 2];
          }
#pragma unroll
          for (int p = 0; p < 4; ++p) cs[p] = a.rope[(size_t)c.rope_pos[min(kg + 4 * p, n - 1)] * (HD / 2) + e0];
        } else {
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const int q = min(kg + 4 * p, n - 1), at = min(row, d - 1);
            hat[p] = h_sent ? q * map.hp + at : 0;
            aat[p] = add_a ? q * d + at : 0;
            hv[p] = load_elem<T>(a.embed, (size_t)sh.tok[q] * d + at);
          }
          hg.issue(hsrc, hat);
          ag.issue(asrc, aat);
        }
      }
      if (nkt <= (w1 ? 2 : 4) * kResWaves) resident_gemm<T, 2>(a, tid, n, w0, w1, nkt, o, w, sh, xs);
      else resident_gemm<T, kResRT2>(a, tid, n, w0, w1, nkt, o, w, sh, xs);
      if (wave == 0) {
        if (h_sent) hg.finish(hsrc, hat, w, hv);
        if (add_a) ag.finish(asrc, aat, w, av);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          if (4 * p >= n) break;
          const int q = min(kg + 4 * p, n - 1);
          const bool ok = kg + 4 * p < n;
          float s0 = 0.f, s1 = 0.f, r = 1.f;
          {
            float v0[kResWaves], v1[kResWaves];
#pragma unroll
            for (int v = 0; v < kResWaves; ++v) {
              v0[v] = sh.red[(v * 2 * kMaxCols + q) * kResRedPitch + col];
              v1[v] = sh.red[((v * 2 + 1) * kMaxCols + q) * kResRedPitch + col];
            }
            if (o.gain) {  // the 16 lanes of a column add up its partial sums
              float ss = 0.f;
              for (int i = col; i < ntile; i += 16) ss += sh.ss[q * kResTiles + i];
              r = 1.0f / sqrtf(group_sum<16>(ss) * a.inv_d + a.eps);
            }
#pragma unroll
            for (int v = 0; v < kResWaves; ++v) {
              s0 += v0[v];
              s1 += v1[v];
            }
          }
          if (qkv) {
            const float v0 = s0 * r + b_lo, v1 = s1 * r + b_hi, cosv = is_q || is_k ? cs[p].x : 1.f, sinv = is_q || is_k ? cs[p].y : 0.f;
            float x = v0 * cosv - v1 * sinv, y = v1 * cosv + v0 * sinv;
            if (sizeof(T) == 2 && !is_q) {  // the other columns see the stored values
              x = bf16_bits_to_float(float_to_bf16_bits(x));
              y = bf16_bits_to_float(float_to_bf16_bits(y));
            }
            if (ok) {
              granule_t* g = lay + map.qkv + q * a.RQKV + hd_ * HD + e0;
              ll_put(g, x, w.epoch);
              ll_put(g + HD / 2, y, w.epoch);
              if (!is_q) {
                T* out = reinterpret_cast<T*>(is_k ? a.kc : a.vc) +
                         ((((size_t)l * a.B + c.seq[q]) * a.Hkv + (hd_ - a.Hq - (is_k ? 0 : a.Hkv))) * a.max_ctx + c.pos[q]) * HD + e0;
                store1<T>(out, x);
                store1<T>(out + HD / 2, y);
              }
            }
          } else if (gateup) {
            const float g = s0 * r, u = s1 * r;
            if (ok) ll_put(lay + map.act + q * a.F + row, (g / (1.0f + expf(-g))) * u, w.epoch);
          } else if (resid) {
            // goes to the MLP of layer l (O projection) or l + 1 (down projection inside a set), or is the set's output
            granule_t* const dst = lay + (oproj ? map.h1 : add_a ? map.layer + map.h1 : map.h2) + q * map.hp;
            float h = hv[p] + (s0 + s1);
            if (add_a) h += av[p];
            if (ok) ll_put(dst + row, h, w.epoch);
            const float ss = group_sum<16>(h * h);
            if (ok && col == 0) ll_put(dst + d + t, ss, w.epoch);
            if (ok && down && l + 1 == a.L) a.H[(size_t)q * d + row] = h;
          } else if (oproj) {
            if (ok) ll_put(lay + map.a + q * d + row, s0 + s1, w.epoch);
          } else {
            const float v = (s0 + s1) * r;
            const bool in = ok && row < a.V;
            if (in && a.logits && c.logit_row[q] >= 0) a.logits[(size_t)c.logit_row[q] * a.V + row] = v;
            float bv = -INFINITY;
            int bi = 0x7FFFFFFF;
            if (in && better(v, row, bv, bi)) { bv = v; bi = row; }
#pragma unroll
            for (int off = 1; off <= 8; off <<= 1) {
              const float ov = __shfl_xor(bv, off, 64);
              const int oi = __shfl_xor(bi, off, 64);
              if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
            }
            if (ok && col == 0) {
              granule_t* g = cand + ((size_t)q * u_v + t) * 2;
              ll_put(g, bv, w.epoch);
              ll_put(g + 1, __uint_as_float((uint32_t)bi), w.epoch);
            }
          }
        }
      }
    } else if (ph == kPhAttn) {
      const int per = n * a.Hkv, li = unit / per, ac = (unit - li * per) / a.Hkv, kvh = unit % a.Hkv, l = lo + li;
      const int c0 = a.col0[ac], pos = c.pos[ac], n_old = c.pos[c0], n_new = pos + 1 - n_old;
      const int vbase = c.vis_base[ac];
      const unsigned long long vmask = c.vis_mask[ac];
      const int sub = lane / LPS, e0 = (lane % LPS) * EPL;
      const size_t rowbase = (((size_t)l * a.B + c.seq[ac]) * a.Hkv + kvh) * (size_t)a.max_ctx;
      const u32x4* const kb = reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(a.kc) + rowbase * HD + e0);
      const u32x4* const vb = reinterpret_cast<const u32x4*>(reinterpret_cast<const T*>(a.vc) + rowbase * HD + e0);
      float* const qs = reinterpret_cast<float*>(xs);      // [G][HD]
      float* const kn = qs + G * HD;                       // [new slot][HD]
      float* const vn = kn + kMaxCols * HD;
      float* const accs = vn + kMaxCols * HD;              // [32 slot groups][G][HD]
      float* const ms = accs + 32 * G * HD;                // [G][32] maxima, then sums
      // The waves share the slots, the cached ones and behind them those of this pass, in runs of whole loads; with seven or
      // eight query heads half of them takes half of the heads.  The first batch of rows is requested before the queries
      // are there.
      constexpr int IT = 4, HS = G >= 7 ? 2 : 1, GW = (G + HS - 1) / HS, NSP = kResWaves / HS, NGRP = NSP * 4;
      const int g0 = wave / NSP * GW, part = wave % NSP, n_all = n_old + n_new;
      const int groups = ceil_div(n_all, SPW), w0 = part * groups / NSP * SPW, w1 = min((part + 1) * groups / NSP * SPW, n_all);
      u32x4 kr[IT], vr[IT];
      auto fetch = [&](int base) {  // unconditional: slots past the cached ones fetch the last of them, or the first row
#pragma unroll
        for (int j = 0; j < IT; ++j) {
          const int s = max(min(base + j * SPW + sub, n_old - 1), 0);
          kr[j] = kb[(size_t)s * LPS];
          vr[j] = vb[(size_t)s * LPS];
        }
      };
      fetch(w0);
      {
        const granule_t* src = a.ll + (size_t)l * map.layer + map.qkv;
        const int total = G * HD + 2 * n_new * HD;
        constexpr int NS = 5;  // sixteen new slots of the most query heads in one go
#pragma unroll 1
        for (int f0 = 0; f0 < total; f0 += NS * kResThreads) {
          int at[NS];
          float x[NS];
          Granules<NS> gr;
#pragma unroll
          for (int i = 0; i < NS; ++i) {
            const int f = min(f0 + tid + i * kResThreads, total - 1), r = (f - G * HD) / HD;  // 64-element row of k, v
            at[i] = f < G * HD ? ac * a.RQKV + kvh * G * HD + f
                               : (c0 + (r < n_new ? r : r - n_new)) * a.RQKV + (a.Hq + (r < n_new ? 0 : a.Hkv) + kvh) * HD + (f & (HD - 1));
          }
          gr.issue(src, at);
          gr.finish(src, at, w, x);
#pragma unroll
          for (int i = 0; i < NS; ++i) {
            const int f = f0 + tid + i * kResThreads;
            if (f >= total) continue;
            const int r = (f - G * HD) / HD;
            if (f < G * HD) qs[f] = x[i];
            else if (r < n_new) kn[r * HD + (f & (HD - 1))] = x[i];
            else vn[(r - n_new) * HD + (f & (HD - 1))] = x[i];
          }
        }
      }
      __syncthreads();
      float q[GW][EPL], acc[GW][EPL], m[GW], sum[GW];
#pragma unroll
      for (int g = 0; g < GW; ++g) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          q[g][e] = qs[min(g0 + g, G - 1) * HD + e0 + e];
          acc[g][e] = 0.f;
        }
        m[g] = -INFINITY;
        sum[g] = 0.f;
      }
      // Batches of IT slots of every slot group, running maximum and sum of the group as in the vector attention kernel
      auto visible = [&](int s) { return s < vbase || ((vmask >> ((s - vbase) & 63)) & 1ull) != 0; };
#pragma unroll 1
      for (int base = w0; base < w1; base += IT * SPW) {
        float kf[IT][EPL], vf[IT][EPL], sc[IT][GW];
#pragma unroll
        for (int j = 0; j < IT; ++j) {
          unpack<T>(kr[j], kf[j]);
          unpack<T>(vr[j], vf[j]);
        }
        if (base + IT * SPW > n_old) {  // uniform: some of this pass's slots
#pragma unroll
          for (int j = 0; j < IT; ++j) {
            const int s = base + j * SPW + sub, at = max(min(s - n_old, n_new - 1), 0) * HD + e0;
#pragma unroll
            for (int e = 0; e < EPL; ++e) {
              kf[j][e] = s >= n_old ? kn[at + e] : kf[j][e];
              vf[j][e] = s >= n_old ? vn[at + e] : vf[j][e];
            }
          }
        }
        fetch(base + IT * SPW);
#pragma unroll
        for (int j = 0; j < IT; ++j)
#pragma unroll
          for (int g = 0; g < GW; ++g) {
            float dot = 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) dot += q[g][e] * kf[j][e];
            sc[j][g] = dot;
          }
#pragma unroll
        for (int j = 0; j < IT; ++j) {
          const int s = base + j * SPW + sub;
          const bool valid = s < w1 && visible(s);
#pragma unroll
          for (int g = 0; g < GW; ++g) {
            const float dot = group_sum<LPS>(sc[j][g]);
            sc[j][g] = valid ? dot * a.scale : -INFINITY;
          }
        }
#pragma unroll
        for (int g = 0; g < GW; ++g) {
          float bm = sc[0][g];
#pragma unroll
          for (int j = 1; j < IT; ++j) bm = fmaxf(bm, sc[j][g]);
          const float m_new = fmaxf(m[g], bm), m_ref = m_new == -INFINITY ? 0.f : m_new, alpha = __expf(m[g] - m_ref);
          m[g] = m_new;
          sum[g] *= alpha;
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[g][e] *= alpha;
#pragma unroll
          for (int j = 0; j < IT; ++j) {
            sc[j][g] = __expf(sc[j][g] - m_ref);  // 0 for slots past the end or masked
            sum[g] += sc[j][g];
          }
        }
#pragma unroll
        for (int j = 0; j < IT; ++j)
#pragma unroll
          for (int g = 0; g < GW; ++g)
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[g][e] += sc[j][g] * vf[j][e];
      }
      // down to four slot groups a wave (eight lanes a slot: lanes 8 apart, inside rows of 16, meet first)
      if (SPW == 8) {
#pragma unroll
        for (int g = 0; g < GW; ++g) {
          const float mm = fmaxf(m[g], dpp_f32<0x128>(m[g])), ref = mm == -INFINITY ? 0.f : mm, f = __expf(m[g] - ref);
          sum[g] *= f;
          sum[g] += dpp_f32<0x128>(sum[g]);
          m[g] = mm;
#pragma unroll
          for (int e = 0; e < EPL; ++e) {
            acc[g][e] *= f;
            acc[g][e] += dpp_f32<0x128>(acc[g][e]);
          }
        }
      }
      const int grp = part * 4 + (SPW == 8 ? sub >> 1 : sub);
      if (SPW == 4 || (sub & 1) == 0) {
#pragma unroll
        for (int g = 0; g < GW; ++g) {
          if (g0 + g >= G) break;
#pragma unroll
          for (int e = 0; e < EPL; e += 4)
            *reinterpret_cast<f32x4*>(accs + (grp * G + g0 + g) * HD + e0 + e) = f32x4{acc[g][e], acc[g][e + 1], acc[g][e + 2], acc[g][e + 3]};
          if (lane % LPS == 0) {
            ms[(g0 + g) * 32 + grp] = m[g];
            ms[G * 32 + (g0 + g) * 32 + grp] = sum[g];
          }
        }
      }
      __syncthreads();
      if (wave < G) {  // a wave per query head: the groups' weights, then an element per lane
        const float gm = ms[wave * 32 + (lane & (NGRP - 1))], gs = ms[G * 32 + wave * 32 + (lane & (NGRP - 1))];
        float x[NGRP];
#pragma unroll
        for (int i = 0; i < NGRP; ++i) x[i] = accs[(i * G + wave) * HD + lane];
        const float mm = lanes_max<NGRP>(gm);
        float f = __expf(gm - mm);
        f /= lanes_sum<NGRP>(gs * f);
        float out = 0.f;
#pragma unroll
        for (int i = 0; i < NGRP; ++i) out += __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), i)) * x[i];
        ll_put(a.ll + (size_t)l * map.layer + map.ao + ac * a.HQ + (kvh * G + wave) * HD + lane, out, w.epoch);
      }
    } else {  // argmax of one column (lowest index on ties)
      float bv = -INFINITY;
      int bi = 0x7FFFFFFF;
      const granule_t* src = cand + (size_t)unit * u_v * 2;
      for (int t0 = 0; t0 < u_v; t0 += kResThreads) {
        const int t = min(t0 + tid, u_v - 1);
        const int at[2] = {2 * t, 2 * t + 1};
        float x[2];
        Granules<2> gr;
        gr.issue(src, at);
        gr.finish(src, at, w, x);
        const int ix = (int)__float_as_uint(x[1]);
        if (better(x[0], ix, bv, bi)) { bv = x[0]; bi = ix; }
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        const float ov = __shfl_xor(bv, off, 64);
        const int oi = __shfl_xor(bi, off, 64);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
      }
      if (lane == 0) {
        sh.red[wave] = bv;
        sh.red[kResWaves + wave] = __uint_as_float((uint32_t)bi);
      }
      __syncthreads();
      if (tid == 0) {
        for (int v = 1; v < kResWaves; ++v) {
          const float ov = sh.red[v];
          const int oi = (int)__float_as_uint(sh.red[kResWaves + v]);
          if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
        }
        if (c.out_idx[unit] >= 0) a.tokens_out[c.out_idx[unit]] = bi;
      }
    }
    ask_next();
    __syncthreads();  // the unit's LDS is free again
    ticket = __builtin_amdgcn_readfirstlane(sh.next);
  }
  // The last workgroup out sets the counters for the next pass: by then every workgroup has read the epoch and has taken
  // its last ticket.
  if (threadIdx.x == 0) {
    const uint32_t out = __hip_atomic_fetch_add(&a.ctl->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (out == gridDim.x - 1) {
      const uint32_t e = w.epoch + 1;
      __hip_atomic_store(&a.ctl->ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&a.ctl->done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&a.ctl->epoch, e == 0u || e == 0xFFFFFFFFu ? 1u : e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Which models and passes, and the launch
// ------------------------------------------------------------------------------------------
bool resident_model(const Shape& s) {
  const int kt = s.dtype == 1 ? 32 : 16;
  return s.hd == 64 && s.R_ffn == 16 && s.R_qkv == 16 && s.L <= kResMaxLayers && s.V <= kResMaxVocab && s.d / 16 <= kResTiles &&
         s.d / kt <= kResRT2 * kResWaves && s.HQ / kt <= kResRT1 * kResWaves && s.F / kt <= kResRT1 * kResWaves;
}

size_t resident_granule_bytes(const Shape& s) {
  const ResidentMap m = resident_map(s.d, s.HQ, s.RQKV, s.F);
  return ((size_t)s.L * m.layer + (size_t)kMaxCols * ceil_div(s.V, 16) * 2) * sizeof(granule_t);
}

static size_t resident_lds(const Shape& s, int n) {
  const int G = s.Hq / s.Hkv;
  const size_t operand = (size_t)std::max(std::max(s.d, s.HQ), s.F) * n * 4;  // fp32, or two bf16 terms
  const size_t attn = ((size_t)G * 64 + 2 * kMaxCols * 64 + 32 * G * 64 + 2 * 32 * G) * sizeof(float);
  return std::max(operand, attn);
}

static int resident_grid(const Shape& s) {
  // two workgroups per unit of the MLP or the head, whichever has more (one works, one waits for the next phase), up to one per CU
  const int widest = std::max(ceil_div(s.F, 16), ceil_div(s.V, 16));
  return std::min(cu_count(), 2 * widest);
}

// Which passes.  Contexts: one workgroup walks a KV head's slots, where the launches split them from 256 on: up to 80 KB of keys
// (fp32 320 slots, bf16 640).  us a step, launches and resident, the 448-wide model of 5 layers with its seven heads per KV head:
// fp32 30 slots 140 / 75, 300 slots 150 / 100; bf16 30 slots 134 / 81, 300 slots 134 / 97, 600 slots 135 / 113.  Columns: the
// operands of a layer, 2 d_model + n_q_heads * head_dim + d_ffn granules a column, up to 24576 of them.
// Inside these limits the route is chosen by a cost in ns, fitted to both routes' times of 2900 calls (400 models of the admitted
// sizes: 2 .. 32 layers, vocabularies of 500 .. 16384, 1 .. 16 columns, sets of 1 .. 8 layers).  A launch saved is worth 2300 (the
// fit's 2600 less a margin for its scatter of 5 % of a call), a merge of split attention 1200.  Against that stand granules staged,
// by every unit for itself: 0.4 each, those of the head 1.6; units that find no workgroup free and follow in a further round: 3000 a
// round; slots that a unit of the attention walks, times its heads: 1.6.  Of those calls one is slower here than as launches
// (1.04x); by the limits above alone 144 were, up to 1.18x.  us a step, launches and resident: fp32 19 layers 576 / 608 wide, sets of
// seven, ten columns 329 / 388; bf16 8 layers 1536 / 3072 wide, vocabulary 16384, sets of eight, three columns 230 / 262.  A third of the
// calls refused are slower resident, the others would gain up to 1.2x, 1.03x on average over all of them.  Of 1311 calls of 260 other
// models that the rule takes, one timed slower (1.05x).
bool resident_pass(const Shape& s, const Cols& c, const int32_t* bounds, int n_sets) {
  const int most = s.dtype == 1 ? 640 : 320;
  int ctx = 0;
  for (int i = 0; i < c.n; ++i) ctx = std::max(ctx, c.pos[i] + 1);
  if (ctx > most || c.n * (2 * s.d + s.HQ + s.F) > 24576 || sizeof(ResidentShared) + resident_lds(s, c.n) > 150 * 1024) return false;
  const long grid = resident_grid(s), ntile = s.d / 16, head = ceil_div(s.V, 16);
  auto rounds = [&](long units) { return (units + grid - 1) / grid; };
  const long r_gu = rounds(s.F / 16), r_down = rounds(ntile), r_head = rounds(head);
  long launches = 3 + 2 * s.L, merges = 0, staged = s.L * (r_gu * s.d + r_down * s.F) + 4 * r_head * s.d, late = s.L * (r_gu + r_down - 2) + r_head - 1, walked = 0;
  for (int j = 0; j < n_sets; ++j) {
    const long k = bounds[j + 1] - bounds[j], r_qkv = rounds(k * (s.RQKV / 32)), r_attn = rounds(k * c.n * s.Hkv), r_o = rounds(k * ntile);
    launches += 3;
    merges += ctx > 256;
    staged += r_qkv * s.d + r_o * s.HQ;
    late += r_qkv + r_attn + r_o - 3;
    walked += r_attn * ctx * (s.Hq / s.Hkv);
  }
  return 2300 * launches + 1200 * merges > (2 * c.n * staged + 8 * walked) / 5 + 3000 * late;
}

#define RESIDENT_G(X) X(1) X(2) X(4) X(7) X(8)
template <typename T>
static const void* resident_fn(int G) {
#define RES_CASE(G_) case G_: return (const void*)resident_kernel<T, G_>;
  switch (G) { RESIDENT_G(RES_CASE) }
#undef RES_CASE
  return nullptr;
}

bool resident_hasty_model(const Shape& s) { return resident_model(s) && s.dtype == 0 && s.Hq == 2 * s.Hkv; }

hipError_t resident_prepare(const Shape& s) {
  const void* f = s.dtype == 1 ? resident_fn<bf16_t>(s.Hq / s.Hkv) : resident_fn<float>(s.Hq / s.Hkv);
  const int lds = 150 * 1024 - (int)sizeof(ResidentShared);
  if (resident_hasty_model(s)) {
    const hipError_t e = hipFuncSetAttribute((const void*)resident_kernel<float, 2, 1>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

void launch_resident(const Shape& s, const Buffers& b, const Resident& r, const Cols& c, const int32_t* tokens, const int32_t* bounds, int n_sets,
                     float* logits, int32_t* tokens_out, hipStream_t st) {
  ResidentArgs a;
  memset(&a, 0, sizeof a);
  a.wqkv = (const u32x4*)b.wqkv; a.wo = (const u32x4*)b.wo; a.wg = (const u32x4*)b.wg; a.wu = (const u32x4*)b.wu; a.wd = (const u32x4*)b.wd;
  a.wlm = (const u32x4*)b.wlm;
  a.embed = b.embed; a.bqkv = s.has_bias ? b.bqkv : nullptr; a.g_attn = b.g_attn; a.g_mlp = b.g_mlp; a.g_final = b.g_final; a.rope = b.rope;
  a.g_any = (const float*)r.granules;
  a.kc = b.kc; a.vc = b.vc; a.H = b.H;
  a.tokens = tokens; a.logits = logits; a.tokens_out = tokens_out;
  a.ctl = r.ctl; a.ll = (granule_t*)r.granules; a.failed = r.failed;
  a.L = s.L; a.d = s.d; a.Hq = s.Hq; a.Hkv = s.Hkv; a.F = s.F; a.V = s.V; a.HQ = s.HQ; a.RQKV = s.RQKV; a.B = s.B; a.max_ctx = s.max_ctx;
  a.n_sets = n_sets;
  a.inv_d = 1.0f / (float)s.d; a.eps = s.eps; a.scale = 1.0f / sqrtf((float)s.hd);
  for (int j = 0; j <= n_sets; ++j) a.bounds[j] = (uint8_t)bounds[j];
  for (int i = 0; i < c.n; ++i) a.col0[i] = (uint8_t)(i > 0 && c.seq[i] == c.seq[i - 1] ? a.col0[i - 1] : i);
  const dim3 grid(resident_grid(s)), blk(kResThreads);
  const size_t lds = resident_lds(s, c.n);
  if (r.hasty) {
    ES_LAUNCH((resident_kernel<float, 2, 1>), grid, blk, lds, st, a, c);
    return;
  }
#define RES_CASE(G_) \
  case G_: \
    if (s.dtype == 1) ES_LAUNCH((resident_kernel<bf16_t, G_>), grid, blk, lds, st, a, c); \
    else ES_LAUNCH((resident_kernel<float, G_>), grid, blk, lds, st, a, c); \
    break;
  switch (s.Hq / s.Hkv) { RESIDENT_G(RES_CASE) }
#undef RES_CASE
}

}  // namespace es
