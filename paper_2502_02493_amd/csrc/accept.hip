// Acceptance by speculative sampling (paper Alg. 3; bonus distribution of Sec. 2.1) on the
// device, in double precision: the decisions (accept or reject, which token the bonus draw
// lands on) are integers decided by floating-point comparisons, so the arithmetic is kept wide
// enough that summation order cannot move a decision except within ~1e-13 of its threshold.
//
//   p'_i = softmax(draft_logits[i] / T),  p_i = softmax(target_logits[i] / T)
//   position i is rejected when r_i * p'_i(x'_i) > p_i(x'_i);  m = first rejected position or gamma
//   bonus ~ max(0, p_m - p'_m) / sum  (m < gamma),  p_gamma  (m = gamma), drawn by inverse CDF in
//   index order with the given uniform u: the lowest v whose running sum exceeds u * sum.
//
// Two launches, both spread over the vocabulary so that no single workgroup has to evaluate 10^5 double-precision
// exponentials:
//   (1) accept_stats_kernel    per logit row and vocabulary slice: slice maximum and sum exp((l - max) / T)  (combined by
//                              the readers); a thread holds its logits in registers, so the slice is read once;
//   (2) accept_draw_kernel     every workgroup repeats the gamma accept decisions (a few exponentials a thread), then adds up
//                              the unnormalised bonus weights q(v) of its vocabulary chunk.  The last workgroup of a
//                              sequence to have done so draws: running sum over the chunk sums in index order, then over the
//                              weights of the chunk the draw lands in, worked out once more (no weight is ever stored).
// "Last" is told by a counter; it says whose sums have been sent, and (1) marks them all as missing, so the last workgroup sees
// when they are there.  (No fence, which would write back the L2, and no wait for a store's acknowledgement.)  In a call that has its
// workspace to itself they always come, some of them already on the way when the counter says so.  Another call on the same workspace at
// the same time can mark them as missing again, for good: the wait ends after kPolls looks, and the call reports -1.
// Bound by fp64 latency and two dependent launches, not by the 5.6 MB of logits.  gamma 5, vocabulary 128 256, one sequence: three
// launches (8 slices of 1024 threads with sixteen exponentials each, weights, draw) 21.1 us a call, two 14.0.  Of these the first
// launch takes 4.6 (two workgroups of 24 exponentials a SIMD on the busiest CUs), the boundary 1.2, and of the second the statistics
// 2.0, decisions 0.7, weights and their sum 0.7, the two counters 1.75 (one for all workgroups: 2.7), the sums 0.95 and the draw 1.55
// (0.25 of it for the one thread that the draw lies with being told by its rank, not by its bounds (first_past), and for the bound).
// Requesting a thread's entries of all positions at the start, instead of those of the position that the decisions leave, does not
// pay: 14.2 (statistics 2.5 us, weights 0.75).
#include "kernels.h"

#include <mutex>
#include <type_traits>

namespace es {

constexpr int kMinSlices = 8, kMaxSlices = 64;  // workgroups per logit row in (1), a power of two (accept_plan)
constexpr int kStatThreads = 512;
constexpr int kStatRegs = 8;       // logits a thread of (1) holds at a time
constexpr int kDrawThreads = 256;  // threads of (2); 2 or 8 vocabulary entries each
constexpr int kPolls = 1 << 18;    // looks for a chunk sum, about a microsecond each: a quarter of a second
constexpr int kWsChunk = 2048;     // the workspace has room for a double per so many entries besides one for each

// Reductions over 8, 16, 32 or 64 neighbouring lanes (n, uniform) by operand swizzles, every lane receiving the result; a shuffle
// through LDS per step would stand in the chain that these kernels are.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
// f of the values of lanes l and l ^ 16 (l ^ 32)
template <bool HALF, class F>
__device__ __forceinline__ float across(float v, const F& f) {
  const uint32_t a = __builtin_bit_cast(uint32_t, v);
  const auto s = HALF ? __builtin_amdgcn_permlane32_swap(a, a, false, false) : __builtin_amdgcn_permlane16_swap(a, a, false, false);
  return f(__builtin_bit_cast(float, (uint32_t)s[0]), __builtin_bit_cast(float, (uint32_t)s[1]));
}
template <bool HALF, class F>
__device__ __forceinline__ double across(double v, const F& f) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
  const auto l = HALF ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false) : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto h = HALF ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false) : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return f(__builtin_bit_cast(double, (uint64_t)l[0] | ((uint64_t)h[0] << 32)), __builtin_bit_cast(double, (uint64_t)l[1] | ((uint64_t)h[1] << 32)));
}
template <typename V, class F>
__device__ __forceinline__ V lanes_fold(V v, int n, const F& f) {
  v = f(v, dpp<0xB1>(v));   // quad_perm [1,0,3,2]
  v = f(v, dpp<0x4E>(v));   // quad_perm [2,3,0,1]
  v = f(v, dpp<0x141>(v));  // row_half_mirror
  if (n >= 16) v = f(v, dpp<0x140>(v));  // row_mirror
  if (n >= 32) v = across<false>(v, f);
  if (n >= 64) v = across<true>(v, f);
  return v;
}
template <typename V>
__device__ __forceinline__ V lanes_sum(V v, int n) {
  return lanes_fold(v, n, [](V a, V b) { return a + b; });
}
__device__ __forceinline__ float lanes_max(float v, int n) {
  return lanes_fold(v, n, [](float a, float b) { return fmaxf(a, b); });
}

// Over the workgroup of NW waves: the waves' results in order, the same bits in every thread.
template <int NW>
__device__ __forceinline__ double block_sum(double v, double* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = lanes_sum(v, 64);
  __syncthreads();  // sh may still be read from the previous call
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) t += sh[w];
  return t;
}
template <int NW>
__device__ __forceinline__ float block_max(float v, float* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = lanes_max(v, 64);
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  float t = -INFINITY;
#pragma unroll
  for (int w = 0; w < NW; ++w) t = fmaxf(t, sh[w]);
  return t;
}

// How a call is cut.  Slices: more than kMinSlices while the workgroups of (1) are fewer than the CUs or a slice is longer
// than its threads hold, as long as a slice has two entries a thread and (2) can take a row's slices side by side, four
// terms a thread at most.  us a call, gamma 5, vocabulary 128 256, with 8 / 16 / 32 / 64 slices: one sequence 19.0 / 15.3 / 15.0 /
// 15.4, four 27.0 / 23.2 / 23.5 / 25.8, sixteen 67.0 / 61.9 / 59.7 / 68.0; gamma 1, 152 064, one 21.2 / 17.1 / 15.1 / 13.7.
// Entries per thread of (2): two, eight where chunks of two would make more than four workgroups per CU (each repeats the
// decisions): one sequence 15.4 us with two, 18.7 with eight; four 23.5 and 25.8; sixteen 61.5 and 59.8.
// us a call of the three launches and of these two, gamma 5: vocabulary 900, one sequence 14.0 and 11.3; 4000, one, four and sixteen
// 13.9, 17.3, 25.4 and 10.9, 11.2, 13.4; 32 000, four, sixteen and 64 20.0, 31.9, 86.7 and 13.5, 22.9, 61.3; 128 256, one, four and
// sixteen 22.2, 31.4, 69.1 and 13.9, 23.7, 60.6; gamma 10, 152 064, one and sixteen 26.4, 130.0 and 20.5, 118.9.
struct AcceptPlan {
  int slices, per, chunks;
};
static AcceptPlan accept_plan(int batch, int gamma, int V) {
  AcceptPlan p;
  const long rows = 2 * (long)gamma + 1, cus = 256;
  p.slices = kMinSlices;
  while (p.slices < kMaxSlices && rows * 2 * p.slices <= 4 * kDrawThreads && V >= 2 * p.slices * 2 * kStatThreads &&
         (V > p.slices * kStatRegs * kStatThreads || rows * p.slices * batch < cus))
    p.slices *= 2;
  p.per = batch * (((long)V + 2 * kDrawThreads - 1) / (2 * kDrawThreads)) > 4 * cus ? 8 : 2;
  p.chunks = (V + p.per * kDrawThreads - 1) / (p.per * kDrawThreads);
  return p;
}

// Workspace of one sequence (doubles): [rows][slices][2] slice statistics, then the chunk sums; in its last double the
// counter of (2).  Room for kMinSlices slices and V + V / kWsChunk doubles more: what accept_plan asks for fits (more slices
// than kMinSlices take at most 2048 doubles and V is at least 16 384 then, the chunks are at most V / 512 + 1 and the lines of
// their groups' counters, from V = 8193 on, V / 512 + 32 doubles).
// kNoSum: a chunk sum that is not there yet, a NaN with a payload that arithmetic does not make.
typedef unsigned long long sum_bits;
constexpr sum_bits kNoSum = 0x7FFC5A3C96E1B482ull;
struct AcceptWs {
  double* stats;
  sum_bits* chunk_sum;
  int* done;
};
__host__ __device__ inline size_t accept_ws_doubles(int gamma, int V) {
  const size_t rows = 2 * (size_t)gamma + 1, nchunk = ((size_t)V + kWsChunk - 1) / kWsChunk;
  return rows * kMinSlices * 2 + nchunk + (size_t)V + 1;
}
__device__ __forceinline__ AcceptWs accept_ws(double* base, int b, int gamma, int V, int slices) {
  const size_t rows = 2 * (size_t)gamma + 1, all = accept_ws_doubles(gamma, V);
  AcceptWs w;
  w.stats = base + (size_t)b * all;
  w.chunk_sum = reinterpret_cast<sum_bits*>(w.stats + rows * slices * 2);
  w.done = reinterpret_cast<int*>(w.stats + all - 1);
  return w;
}
// The counter of the group of kGroup chunks that c belongs to: a line of its own each, in front of the last double (a call of more
// than one group has a vocabulary of more than 8192).
constexpr int kGroup = 16;
__device__ __forceinline__ int* group_counter(const AcceptWs& w, int c) { return w.done - 32 * (c / kGroup + 1); }

// x / T as the division rounds it, without one: y = 1 / T rounded to nearest, q = x y, then one step q + (x - q T) y with
// fused multiply-adds (Markstein 1990: correctly rounded if y is).  Infinities and NaNs keep the product.
__device__ __forceinline__ double quotient(double x, double T, double y) {
  const double q = x * y;
  return fabs(q) < INFINITY ? fma(fma(-q, T, x), y, q) : q;
}

// rows 0..gamma are the target's, rows gamma+1..2*gamma the draft's.  grid (slices, rows, batch)
__global__ __launch_bounds__(kStatThreads) void accept_stats_kernel(const float* __restrict__ draft_logits,
                                                                     const float* __restrict__ target_logits, int gamma, int V,
                                                                     double T, int slices, int chunks,
                                                                     double* __restrict__ ws_base) {
  __shared__ double sh_d[kStatThreads / 64];
  __shared__ float sh_f[kStatThreads / 64];
  const int slice = blockIdx.x, j = blockIdx.y, b = blockIdx.z;
  const float* row = j <= gamma ? target_logits + ((size_t)b * (gamma + 1) + j) * V
                                : draft_logits + ((size_t)b * gamma + (j - gamma - 1)) * V;
  const int per = (V + slices - 1) / slices;
  const int v0 = min(V, slice * per), v1 = min(V, v0 + per);
  const bool held = v1 - v0 <= kStatRegs * kStatThreads;  // uniform: the slice stays in registers between the two passes over it
  float l[kStatRegs];
  auto load = [&](int base) {
#pragma unroll
    for (int i = 0; i < kStatRegs; ++i) {
      const int v = base + i * kStatThreads + threadIdx.x;
      l[i] = v < v1 ? row[v] : -INFINITY;
    }
  };
  float mx = -INFINITY;
  for (int base = v0; base < v1; base += kStatRegs * kStatThreads) {
    load(base);
#pragma unroll
    for (int i = 0; i < kStatRegs; ++i) mx = fmaxf(mx, l[i]);
  }
  mx = block_max<kStatThreads / 64>(mx, sh_f);
  const double ref = mx == -INFINITY ? 0.0 : (double)mx;  // nothing but minus infinities: they add exp(-inf) = 0
  const double inv_T = 1.0 / T;
  double z = 0.0;
  for (int base = v0; base < v1; base += kStatRegs * kStatThreads) {
    if (!held) load(base);
#pragma unroll
    for (int i = 0; i < kStatRegs; ++i)
      if (base + i * kStatThreads < v1) z += exp(quotient((double)l[i] - ref, T, inv_T));  // uniform; slots past the end add 0
  }
  z = block_sum<kStatThreads / 64>(z, sh_d);
  const AcceptWs ws = accept_ws(ws_base, b, gamma, V, slices);
  if (threadIdx.x == 0) {
    double* o = ws.stats + ((size_t)j * slices + slice) * 2;
    o[0] = (double)mx;  // -inf for an empty slice; its sum is 0
    o[1] = z;
  }
  if (j == 0)
    for (int c = slice * kStatThreads + threadIdx.x; c < chunks; c += slices * kStatThreads) {
      ws.chunk_sum[c] = kNoSum;
      if (c % kGroup == 0 && chunks > kGroup) *group_counter(ws, c) = 0;
      if (c == 0) *ws.done = 0;
    }
}

// Inclusive running sum over the workgroup's threads: inside rows of 16 lanes by operand swizzles, then the rows' and the waves' totals
// in order.  incl[] holds every thread's afterwards.  Neighbours add the same terms in different orders, so incl[] rises and falls by
// last bits where the terms in between are small or nothing: a threshold can lie between several neighbouring entries.
__device__ __forceinline__ double lane_value(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
__device__ __forceinline__ void block_scan(double v, double* incl, double* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = lane >> 4;
  v += dpp<0x111>(v);  // row_shr by 1, 2, 4, 8: zeros come in
  v += dpp<0x112>(v);
  v += dpp<0x114>(v);
  v += dpp<0x118>(v);
  const double t0 = lane_value(v, 15), t1 = t0 + lane_value(v, 31), t2 = t1 + lane_value(v, 47);
  v += row == 0 ? 0.0 : row == 1 ? t0 : row == 2 ? t1 : t2;
  __syncthreads();  // sh and incl may still be read from the previous call
  if (lane == 63) sh[wave] = v;
  __syncthreads();
  double before = 0.0;
  for (int k = 0; k < wave; ++k) before += sh[k];
  incl[threadIdx.x] = before + v;
  __syncthreads();
}

// grid (chunks, batch); PER: vocabulary entries per thread, POLLS: looks for a chunk sum before the sequence is given up.  Every
// workgroup takes the same decisions from the same numbers: a row's slices in as many neighbouring lanes, their terms added by
// shuffles; then, in every wave, the test of each position in a lane.
constexpr int kMaxAcceptRows = 2 * 64 + 1;
template <int PER, int POLLS>
__global__ __launch_bounds__(kDrawThreads) void accept_draw_kernel(const int32_t* __restrict__ draft, const float* __restrict__ draft_logits,
                                                                    const float* __restrict__ target_logits, const float* __restrict__ r,
                                                                    const float* __restrict__ u, int gamma, int V, double T, int slices,
                                                                    double* ws_base, int32_t* __restrict__ accept_len,
                                                                    int32_t* __restrict__ bonus) {
  constexpr int kChunk = PER * kDrawThreads;
  __shared__ double s_incl[kDrawThreads], s_wave[kDrawThreads / 64], s_mx[kMaxAcceptRows], s_z[kMaxAcceptRows];
  __shared__ double s_lo[kDrawThreads / 64];
  __shared__ int s_flag, s_at[kDrawThreads / 64];
  __shared__ int s_lost[2];  // a chunk sum did not come: while they were added up, while the draw's chunk was looked for
  const int chunk = blockIdx.x, nchunk = gridDim.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const AcceptWs ws = accept_ws(ws_base, b, gamma, V, slices);
  const float* tl = target_logits + (size_t)b * (gamma + 1) * V;
  const float* dl = draft_logits + (size_t)b * gamma * V;
  const double inv_T = 1.0 / T;
  // Requested in the order of need: loads return in it.  First the drafted tokens, then the statistics, then the tokens' logits.
  int token = -1;
  float t_logit = 0.f, d_logit = 0.f, r_in = 0.f;
  if (lane < gamma) {
    token = draft[(size_t)b * gamma + lane];
    r_in = r[(size_t)b * gamma + lane];
  }
  const float u_in = u[b];
  auto others = [&] {
    asm volatile("" ::: "memory");  // behind the statistics
    if (token >= 0 && token < V) {
      t_logit = tl[(size_t)lane * V + token];
      d_logit = dl[(size_t)lane * V + token];
    }
    asm volatile("" ::: "memory");
  };
  if (tid < 2) s_lost[tid] = 0;
  const int terms = (2 * gamma + 1) * slices;
  auto combine = [&](auto side_by_side, int first, const auto& others) {  // that many terms a thread, their chains interleaved
    constexpr int N = decltype(side_by_side)::value;
    double mine[N], sum[N], m[N], t[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const size_t i = min(first + tid + k * kDrawThreads, terms - 1);
      mine[k] = ws.stats[2 * i];
      sum[k] = ws.stats[2 * i + 1];
    }
    others();
    // the slices are a power of two and divide 64: a row's lie in one wave
#pragma unroll
    for (int k = 0; k < N; ++k) m[k] = lanes_max((float)mine[k], slices);  // maxima of floats
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const double e = sum[k] * exp(quotient(mine[k] - m[k], T, inv_T));
      t[k] = sum[k] > 0.0 ? e : 0.0;
    }
#pragma unroll
    for (int k = 0; k < N; ++k) t[k] = lanes_sum(t[k], slices);
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int i = first + tid + k * kDrawThreads;
      if (i < terms && (i & (slices - 1)) == 0) {
        s_mx[i / slices] = m[k];
        s_z[i / slices] = t[k];
      }
    }
  };
  if (terms <= kDrawThreads) {
    combine(std::integral_constant<int, 1>{}, 0, others);
  } else if (terms <= 2 * kDrawThreads) {
    combine(std::integral_constant<int, 2>{}, 0, others);
  } else {
    combine(std::integral_constant<int, 4>{}, 0, others);
    for (int first = 4 * kDrawThreads; first < terms; first += 4 * kDrawThreads) combine(std::integral_constant<int, 4>{}, first, [] {});
  }
  __syncthreads();
  bool rejected = false;
  if (lane < gamma && token >= 0 && token < V) {
    const double p = exp(quotient((double)t_logit - s_mx[lane], T, inv_T)) / s_z[lane];
    const double pd = exp(quotient((double)d_logit - s_mx[gamma + 1 + lane], T, inv_T)) / s_z[gamma + 1 + lane];
    rejected = (double)r_in * pd > p;
  }
  const bool bad = lane < gamma && !(token >= 0 && token < V);
  const unsigned long long stop = __ballot(rejected || bad), bads = __ballot(bad);
  const int m = stop ? __ffsll((long long)stop) - 1 : gamma;
  auto report = [&](int len, int token) {
    if (tid == 0) {
      accept_len[b] = len;
      bonus[b] = token;
    }
  };
  if ((bads >> (m & 63)) & 1 & (unsigned long long)(m < gamma)) {  // not a token
    if (chunk == 0) report(-1, -1);
    return;
  }
  const double tm = s_mx[m], tz = s_z[m], inv_tz = 1.0 / tz;
  bool residual = m < gamma;
  const double dm = residual ? s_mx[gamma + 1 + m] : 0.0, dz = residual ? s_z[gamma + 1 + m] : 1.0, inv_dz = 1.0 / dz;
  const float* trow = tl + (size_t)m * V;
  const float* drow = residual ? dl + (size_t)m * V : trow;
  auto weight = [&](float t, float dd) {
    double q = quotient(exp(quotient((double)t - tm, T, inv_T)), tz, inv_tz);
    if (residual) {
      q -= quotient(exp(quotient((double)dd - dm, T, inv_T)), dz, inv_dz);
      q = q > 0.0 ? q : 0.0;
    }
    return q;
  };
  // each thread owns a contiguous run, so that every sum below is in index order
  auto run_of = [&](int c, double (&q)[PER]) {
    const int v0 = c * kChunk + tid * PER;
    float t[PER], dd[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int v = min(v0 + i, V - 1);
      t[i] = trow[v];
      dd[i] = drow[v];
    }
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      q[i] = v0 + i < V ? weight(t[i], dd[i]) : 0.0;
      s += q[i];
    }
    return s;
  };
  auto load_sum = [&](int c) { return __hip_atomic_load(&ws.chunk_sum[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  auto send_sum = [&](int c, double v) {
    __hip_atomic_store(&ws.chunk_sum[c], v == v ? __builtin_bit_cast(sum_bits, v) : 0x7FF8000000000000ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  double q[PER];
  const double tot = block_sum<kDrawThreads / 64>(run_of(chunk, q), s_wave);
  // every thread's first chunk sum comes with the counter: for the last workgroup it is there, but for those under way
  const int cper = (nchunk + kDrawThreads - 1) / kDrawThreads, c0 = min(nchunk, tid * cper), c1 = min(nchunk, c0 + cper);
  const sum_bits early = load_sum(min(c0, nchunk - 1));
  if (tid == 0) {
    send_sum(chunk, tot);
    // Raising one counter takes 11 ns a workgroup, one after the other (2.7 us for 251): a counter for every sixteen
    // chunks, and one for those that were a group's last.
    auto raise = [](int* p) { return __hip_atomic_fetch_add(p, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    const int group = min(kGroup, nchunk - chunk / kGroup * kGroup), groups = (nchunk + kGroup - 1) / kGroup;
    s_flag = (groups == 1 || raise(group_counter(ws, chunk)) == group - 1) && raise(ws.done) == (groups == 1 ? nchunk : groups) - 1;
  }
  __syncthreads();
  if (!s_flag) return;

  // The sequence's last workgroup: every thread takes a run of chunks
  auto chunk_sum = [&](int c, int stage, sum_bits x = kNoSum) {  // it has been sent: there at the first look or a few later
    for (int looks = 0; x == kNoSum && looks < POLLS; ++looks) x = load_sum(c);
    if (x == kNoSum) s_lost[stage] = 1;  // a NaN, and the thread looks no further
    return __builtin_bit_cast(double, x);
  };
  double own = 0.0;  // this thread's part of s_incl
  auto scan_chunks = [&](sum_bits first) {
    own = 0.0;
    for (int c = c0; c < c1 && own == own; ++c) own += chunk_sum(c, 0, c == c0 ? first : kNoSum);
    block_scan(own, s_incl, s_wave);
    return s_incl[kDrawThreads - 1];
  };
  double total = scan_chunks(early);
  if (!(total > 0.0)) {
    if (s_lost[0]) return report(-1, -1);
    // identical distributions leave no residual (a rejection is then impossible for r < 1): fall
    // back to the target distribution of that position (rare, slow, correct)
    residual = false;
    for (int c = 0; c < nchunk; ++c) {
      const double s = block_sum<kDrawThreads / 64>(run_of(c, q), s_wave);
      if (tid == 0) send_sum(c, s);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the old sums are gone when the other waves look
    __syncthreads();
    total = scan_chunks(kNoSum);
    if (s_lost[0]) return report(-1, -1);
  }
  const double thr = lane_value((double)u_in * total, 0);  // uniform
  // The draw lies with the first thread that has weight and whose running sum, on top of `before`, is past the threshold; find(lo), called
  // for it (and for the first such thread of every other wave), gives the place in its run and moves lo to the sum in front of it.
  auto first_past = [&](double before, double* at_lo, auto&& find) {
    const int wave = tid >> 6;
    const double below = s_incl[max(tid - 1, 0)];  // side by side with the thread's own
    const unsigned long long past = __ballot(own > 0.0 && thr < before + s_incl[tid]);
    if (lane == (past ? __ffsll((long long)past) - 1 : 0)) {
      double lo = before + (tid ? below : 0.0);
      s_at[wave] = past ? find(lo) : -1;
      s_lo[wave] = lo;
    }
    __syncthreads();
    int at[kDrawThreads / 64], first = -1;
    double lo[kDrawThreads / 64];
#pragma unroll
    for (int w = 0; w < kDrawThreads / 64; ++w) {
      at[w] = s_at[w];
      lo[w] = s_lo[w];
    }
#pragma unroll
    for (int w = kDrawThreads / 64 - 1; w >= 0; --w) {
      first = at[w] >= 0 ? at[w] : first;
      *at_lo = at[w] >= 0 ? lo[w] : *at_lo;
    }
    *at_lo = lane_value(*at_lo, 0);
    return __builtin_amdgcn_readfirstlane(first);
  };
  double before = 0.0, unused = 0.0;
  const int pick_chunk = first_past(0.0, &before, [&](double& lo) {
    int c = c0;
    for (; c < c1 - 1; ++c) {
      const double w = chunk_sum(c, 1);
      if (w != w || (w > 0.0 && lo + w > thr)) break;
      lo += w;
    }
    return c;
  });  // -1: u * total rounded up to the total
  if (cper > 1 && s_lost[1]) return report(-1, -1);
  int pick = -1;
  if (pick_chunk >= 0) {
    own = run_of(pick_chunk, q);
    block_scan(own, s_incl, s_wave);
    pick = first_past(before, &unused, [&](double& lo) {
      int at = -1;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        if (at >= 0 && lo > thr) continue;  // found: the running sum is past the threshold
        if (q[i] > 0.0) at = pick_chunk * kChunk + tid * PER + i;
        lo += q[i];
      }
      return at;
    });
  }
  if (pick < 0) {
    // the sums disagreed in the last bit, or the threshold reached the total: the last token with
    // positive weight up to the chunk's end (of the vocabulary), or the first
    if (tid == 0) s_flag = -1;
    int end = min(V, pick_chunk >= 0 ? (pick_chunk + 1) * kChunk : V);
    for (; pick < 0 && end > 0; end -= kDrawThreads) {
      const int v = end - 1 - tid;
      const bool positive = v >= 0 && weight(trow[max(v, 0)], drow[max(v, 0)]) > 0.0;
      __syncthreads();
      if (positive) atomicMax(&s_flag, v);
      __syncthreads();
      pick = s_flag;
    }
    pick = max(pick, 0);
  }
  report(m, pick);
}

size_t sample_accept_workspace_bytes(int batch, int gamma, int V) {
  return (size_t)batch * accept_ws_doubles(gamma, V) * sizeof(double);
}

void launch_sample_accept(const int32_t* draft, const float* draft_logits, const float* target_logits, const float* r,
                          const float* u, int batch, int gamma, int V, double T, double* ws, int32_t* accept_len,
                          int32_t* bonus, bool give_up, hipStream_t st) {
  const AcceptPlan p = accept_plan(batch, gamma, V);
  hipLaunchKernelGGL(accept_stats_kernel, dim3(p.slices, 2 * gamma + 1, batch), dim3(kStatThreads), 0, st, draft_logits, target_logits,
                     gamma, V, T, p.slices, p.chunks, ws);
  const auto draw = give_up ? (p.per == 2 ? accept_draw_kernel<2, 0> : accept_draw_kernel<8, 0>)
                            : (p.per == 2 ? accept_draw_kernel<2, kPolls> : accept_draw_kernel<8, kPolls>);
  hipLaunchKernelGGL(draw, dim3(p.chunks, batch), dim3(kDrawThreads), 0, st, draft, draft_logits, target_logits, r, u, gamma, V, T,
                     p.slices, ws, accept_len, bonus);
}

// ------------------------------------------------------------------------------------------
// The same two launches for callers that cannot allocate and bring no workspace: the
// workspace is a file-scope device array.  Its name is a host-side stand-in, not a device
// address: the address comes from hipGetSymbolAddress, once per device with that device
// current (every GPU holds its own copy), and only that pointer is handed to kernels.
// ------------------------------------------------------------------------------------------
constexpr size_t kStaticWsDoubles = (size_t)1 << 20;  // 8 MiB per GPU, held until the process ends
static __device__ __align__(256) double scratch[kStaticWsDoubles];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static double* g_scratch_ptr[kMaxDevices];  // per device, filled at the first call on it

size_t sample_accept_static_capacity_bytes() { return kStaticWsDoubles * sizeof(double); }

hipError_t sample_accept_static_workspace(double** out) {
  *out = nullptr;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    double* p = nullptr;
    e = hipGetSymbolAddress((void**)&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace es
