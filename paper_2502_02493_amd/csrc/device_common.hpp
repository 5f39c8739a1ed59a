// gfx950 (CDNA4, wave64) kernels of the EasySpec draft hot path.
//
// Every weight contraction of the model is the same shape of work: a matrix that is far larger
// than any cache is streamed from HBM exactly once and multiplied with at most 16 token
// columns (1 per live sequence in a fuzzy draft step, paper Alg. 2; the accepted tokens plus
// the bonus token in calibration, paper Sec. 3.2).  All of them therefore share one core:
//
//   * Weights are repacked at load time into 1 KB tiles of 16 rows x KT columns (KT = 32 bf16
//     or 16 fp32).  Inside a tile, lane l of a wavefront owns 16 contiguous bytes: row l%16,
//     columns (l/16)*EPL .. +EPL-1.  That is exactly the A-operand register layout of the
//     16x16 MFMA instructions, so one fully coalesced 1 KB wave load feeds one MFMA with no
//     shuffling, and a row tile's K sweep is one contiguous ascending address stream.
//   * The token columns are the MFMA's N dimension (B operand, 16 bytes per lane read from a
//     small L2-resident activation array, only lanes of live columns load).
//   * The waves of a workgroup split K between them (interleaved, so the workgroup reads
//     consecutive KBs), partial accumulators are summed through LDS in a fixed order, and a
//     thread per element runs the epilogue that the operation needs (bias + rotary + cache
//     write, residual update + next norm input, SiLU*up, logits + argmax).
//
// RMSNorm is split so that no kernel has to normalise before it can start streaming: the
// producer of a residual vector h writes T(h * gain) for the consumer's gain and the partial
// sums of squares of h per 16-row tile; the consumer multiplies its accumulators by
// rsqrt(mean(h^2) + eps).  Both sides of the parity tests use this order of roundings.
#pragma once
#include "kernels.h"
#include "tile_index.hpp"

#include <algorithm>
#include <type_traits>

namespace es {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct bf16_t {
  uint16_t bits;
};

template <typename T>
struct Tr;
template <>
struct Tr<float> {
  static constexpr int EPL = 4, KT = 16, PARTS = 1;
};
// bf16 activations are carried as two bf16 terms, hi = bf16(x) and lo = bf16(x - hi), stored as
// two arrays [hi | lo]; the contraction runs one MFMA per term.  MFMA issue slots are idle in
// this HBM-bound work, so the second term is free and keeps activations at ~16 mantissa bits.
template <>
struct Tr<bf16_t> {
  static constexpr int EPL = 8, KT = 32, PARTS = 2;
};

// Layout of an activation operand: see tile_index.hpp (xoff_elems), here by element type.
static_assert(kOperandCols == kMaxCols, "operand slots hold kMaxCols columns");
template <typename T>
__device__ __forceinline__ size_t xoff(int ncols, int K, int col, int k) {
  return xoff_elems(Tr<T>::EPL, ncols, K, col, k);
}
// u32x4 between the fragments of consecutive k-tiles
template <typename T>
__device__ __forceinline__ int xtile_stride(int ncols) {
  return xtile_fragments(ncols);
}

__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ uint32_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest, ties to even
  return u >> 16;
}

// two floats to two bf16 (a in the low half), round to nearest even: one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
// x[0..7] as two bf16 terms, hi = bf16(x), lo = bf16(x - hi)
__device__ __forceinline__ void split_bf16x8(const float (&x)[8], bf16x8& hi, bf16x8& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    h[j] = pack_bf16x2(x[2 * j], x[2 * j + 1]);
    l[j] = pack_bf16x2(x[2 * j] - __uint_as_float(h[j] << 16), x[2 * j + 1] - __uint_as_float(h[j] & 0xFFFF0000u));
  }
  const u32x4 hv = {h[0], h[1], h[2], h[3]}, lv = {l[0], l[1], l[2], l[3]};
  hi = __builtin_bit_cast(bf16x8, hv);
  lo = __builtin_bit_cast(bf16x8, lv);
}

// ... and what those two terms leave of x, as a third: with it all 24 bits
__device__ __forceinline__ bf16x8 third_bf16x8(const float (&x)[8], bf16x8 hi, bf16x8 lo) {
  const u32x4 hv = __builtin_bit_cast(u32x4, hi), lv = __builtin_bit_cast(u32x4, lo);
  uint32_t r[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    r[j] = pack_bf16x2((x[2 * j] - __uint_as_float(hv[j] << 16)) - __uint_as_float(lv[j] << 16),
                       (x[2 * j + 1] - __uint_as_float(hv[j] & 0xFFFF0000u)) - __uint_as_float(lv[j] & 0xFFFF0000u));
  const u32x4 rv = {r[0], r[1], r[2], r[3]};
  return __builtin_bit_cast(bf16x8, rv);
}

// Is any of eight packed bf16 infinite or NaN (all exponent bits set: adding one to the exponent carries into the sign)?
__device__ __forceinline__ bool any_nonfinite(u32x4 v) {
  uint32_t carry = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) carry |= (v[i] & 0x7F807F80u) + 0x00800080u;
  return (carry & 0x80008000u) != 0;
}
// ... and the same with those that are cleared
__device__ __forceinline__ u32x4 clear_nonfinite(u32x4 v) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    v[i] &= ((v[i] & 0x7F80u) == 0x7F80u ? 0xFFFF0000u : 0xFFFFFFFFu) & ((v[i] & 0x7F800000u) == 0x7F800000u ? 0x0000FFFFu : 0xFFFFFFFFu);
  return v;
}

template <typename T>
__device__ __forceinline__ float load1(const T* p);
template <>
__device__ __forceinline__ float load1<float>(const float* p) {
  return *p;
}
template <>
__device__ __forceinline__ float load1<bf16_t>(const bf16_t* p) {
  return bf16_bits_to_float(p->bits);
}

template <typename T>
__device__ __forceinline__ void store1(T* p, float v);
template <>
__device__ __forceinline__ void store1<float>(float* p, float v) {
  *p = v;
}
template <>
__device__ __forceinline__ void store1<bf16_t>(bf16_t* p, float v) {
  p->bits = (uint16_t)float_to_bf16_bits(v);
}

// four consecutive elements, p aligned to 4 elements
template <typename T>
__device__ __forceinline__ void store4(T* p, float a, float b, float c, float d);
template <>
__device__ __forceinline__ void store4<float>(float* p, float a, float b, float c, float d) {
  f32x4 v = {a, b, c, d};
  *reinterpret_cast<f32x4*>(p) = v;
}
template <>
__device__ __forceinline__ void store4<bf16_t>(bf16_t* p, float a, float b, float c, float d) {
  u32x2 v = {float_to_bf16_bits(a) | (float_to_bf16_bits(b) << 16), float_to_bf16_bits(c) | (float_to_bf16_bits(d) << 16)};
  *reinterpret_cast<u32x2*>(p) = v;
}

// Activation stores: p points into the "hi" array, the "lo" array starts part elements later.
template <typename T>
__device__ __forceinline__ void store_act1(T* p, size_t part, float v);
template <>
__device__ __forceinline__ void store_act1<float>(float* p, size_t, float v) {
  *p = v;
}
template <>
__device__ __forceinline__ void store_act1<bf16_t>(bf16_t* p, size_t part, float v) {
  const uint32_t hi = float_to_bf16_bits(v);
  p->bits = (uint16_t)hi;
  p[part].bits = (uint16_t)float_to_bf16_bits(v - bf16_bits_to_float(hi));
}
// two consecutive elements, p aligned to two
template <typename T>
__device__ __forceinline__ void store_act2(T* p, size_t part, float a, float b);
template <>
__device__ __forceinline__ void store_act2<float>(float* p, size_t, float a, float b) {
  *reinterpret_cast<float2*>(p) = make_float2(a, b);
}
template <>
__device__ __forceinline__ void store_act2<bf16_t>(bf16_t* p, size_t part, float a, float b) {
  const uint32_t ha = float_to_bf16_bits(a), hb = float_to_bf16_bits(b);
  *reinterpret_cast<uint32_t*>(p) = ha | (hb << 16);
  *reinterpret_cast<uint32_t*>(p + part) = float_to_bf16_bits(a - bf16_bits_to_float(ha)) | (float_to_bf16_bits(b - bf16_bits_to_float(hb)) << 16);
}
template <typename T>
__device__ __forceinline__ void store_act4(T* p, size_t part, float a, float b, float c, float d);
template <>
__device__ __forceinline__ void store_act4<float>(float* p, size_t, float a, float b, float c, float d) {
  store4<float>(p, a, b, c, d);
}
template <>
__device__ __forceinline__ void store_act4<bf16_t>(bf16_t* p, size_t part, float a, float b, float c, float d) {
  const uint32_t ha = float_to_bf16_bits(a), hb = float_to_bf16_bits(b), hc = float_to_bf16_bits(c), hd = float_to_bf16_bits(d);
  u32x2 hi = {ha | (hb << 16), hc | (hd << 16)};
  *reinterpret_cast<u32x2*>(p) = hi;
  store4<bf16_t>(p + part, a - bf16_bits_to_float(ha), b - bf16_bits_to_float(hb), c - bf16_bits_to_float(hc),
                 d - bf16_bits_to_float(hd));
}

// unpack the EPL elements of one 16-byte fragment
template <typename T>
__device__ __forceinline__ void unpack(const u32x4& r, float (&out)[Tr<T>::EPL]);
template <>
__device__ __forceinline__ void unpack<float>(const u32x4& r, float (&out)[4]) {
  out[0] = __uint_as_float(r.x); out[1] = __uint_as_float(r.y); out[2] = __uint_as_float(r.z); out[3] = __uint_as_float(r.w);
}
template <>
__device__ __forceinline__ void unpack<bf16_t>(const u32x4& r, float (&out)[8]) {
  out[0] = __uint_as_float(r.x << 16); out[1] = __uint_as_float(r.x & 0xFFFF0000u);
  out[2] = __uint_as_float(r.y << 16); out[3] = __uint_as_float(r.y & 0xFFFF0000u);
  out[4] = __uint_as_float(r.z << 16); out[5] = __uint_as_float(r.z & 0xFFFF0000u);
  out[6] = __uint_as_float(r.w << 16); out[7] = __uint_as_float(r.w & 0xFFFF0000u);
}

// One k-tile of multiply-accumulate: acc[16 rows x 16 cols] += A[16 x KT] * B[KT x 16].
template <typename T>
__device__ __forceinline__ void mma(f32x4& acc, const u32x4& a, const u32x4& b);
template <>
__device__ __forceinline__ void mma<bf16_t>(f32x4& acc, const u32x4& a, const u32x4& b) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
template <>
__device__ __forceinline__ void mma<float>(f32x4& acc, const u32x4& a, const u32x4& b) {
  // four K=4 steps; step e contracts element e of every lane's fragment (same k on both sides)
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
}

// ------------------------------------------------------------------------------------------
// The shared core.  w[r]: first tile of row tile r (tiles of one row tile are consecutive,
// 64 u32x4 each).  x: activation operand in T (layout: xoff).  The calling wave accumulates k-tiles
// wave, wave+NW, ... into acc.
//
// NB = B fragments (and MFMAs) per weight tile.  With two-term activations and at most 8
// columns, the lo terms ride in MFMA columns ncols..2*ncols-1 of the same instruction
// ("folded", NB = 1) and tile_sum() adds the two halves at the end; with more columns the
// hi and lo terms take one MFMA each (NB = 2).  A wave keeps one batch of 8 KB in flight; two
// batches per wave were measured slower (the registers cost more occupancy than they hide).
// ------------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ bool folded(int ncols) {
  return Tr<T>::PARTS == 2 && 2 * ncols <= kMaxCols;
}

// NP = forward passes served by one launch (1, or 2: a calibration of more columns than one pass holds runs
// its passes two at a time).  Every weight fragment a wave loads is then used for both passes' columns: the
// passes have their own activation operands, accumulators and epilogues, the weights leave HBM once.
//
// What the code around the loads costs shows in the launches whose waves hold the most registers.  Addresses of single tiles in
// vector registers and a branch for every operand fragment spilled registers in the two-fragment O and down projections and
// took about a hundred instructions a batch; with uniform addresses and one branch a batch: prefill of 16 tokens at context
// 8192 4120 -> 4071 us, Qwen2-7B step 2692 -> 2636, 6-token calibration 3372 -> 3340 (runs of one build differ by 0.4 to 1.5 %).
//
// meanwhile(0) is called once, by every wave, when its first batch of weights has been requested: whatever else a kernel has to
// fetch or work out before its stream ends belongs there.  meanwhile(1) follows when its second batch has been requested (what
// was fetched has arrived by then), or at the end if there is none.  NW, the waves of the workgroup, is an argument of the kernels:
// blockDim lies behind the arguments, in a cache line of its own that a wave would wait for a second time before its first load.
template <typename T, int RT, int NB, int NP, class Meanwhile>
__device__ __forceinline__ void gemm_loop(const u32x4* const (&w)[RT], const u32x4* const (&x)[NP], const uint32_t (&x_lane)[NB], int xs, const bool& colok,
                                          int nkt, int NW, f32x4 (&acc)[NP][RT], int w_lane, int w_stride, const Meanwhile& meanwhile) {
  constexpr int U = batch_len(RT);  // k-tiles per batch: 8 KB of weights in flight per wave
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // w_lane: the lane's 16-byte piece of a weight fragment, w_stride: pieces per fragment (lane and 64 for tiles of 16 rows).
  // A tile's address is a uniform base and the lane's 32-bit offset: no vector registers per tile.
  const uint32_t w_byte = (uint32_t)w_lane * 16;
  auto piece = [](const u32x4* base, uint32_t byte) { return reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(base) + byte); };
  const u32x4 zero = {0u, 0u, 0u, 0u};
  // One batch.  The last, partial one has the same shape with the loads past the end switched off (wave-uniform), so
  // that the remaining tiles are still fetched together instead of one latency at a time.
  auto batch = [&](int kt, auto partial, auto&& requested) {
    constexpr bool PARTIAL = decltype(partial)::value;
    u32x4 a[RT][U], b[NP][NB][U];
    uint32_t wb = w_byte;
    asm volatile("" : "+v"(wb));  // keeps the sum with the uniform base, which is different for every load, out of vector registers
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = !PARTIAL || batch_tile(kt, u, NW) < nkt;
#pragma unroll
      for (int r = 0; r < RT; ++r) a[r][u] = in ? __builtin_nontemporal_load(piece(w[r] + (size_t)batch_tile(kt, u, NW) * w_stride, wb)) : zero;
    }
    requested();
    // the lanes of columns that are not there leave their registers as they are: what they hold only reaches those columns of the product
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < NB; ++q) b[p][q][u] = __builtin_nondeterministic_value(zero);
    if (colok) {
      uint32_t xb[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        xb[q] = x_lane[q];
        asm volatile("" : "+v"(xb[q]));
      }
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const bool in = !PARTIAL || batch_tile(kt, u, NW) < nkt;
#pragma unroll
          for (int q = 0; q < NB; ++q) b[p][q][u] = in ? *piece(x[p] + (size_t)batch_tile(kt, u, NW) * xs, xb[q]) : zero;
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int r = 0; r < RT; ++r) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int q = 0; q < NB; ++q) mma<T>(acc[p][r], a[r][u], b[p][q][u]);
      }
    }
  };
  int kt = wave;
  const auto first = [&] {
    asm volatile("" ::: "memory");  // the requests stay ahead of it
    meanwhile(std::integral_constant<int, 0>{});
  };
  const auto second = [&] {
    asm volatile("" ::: "memory");
    meanwhile(std::integral_constant<int, 1>{});
  };
  const auto nothing = [] {};
  if (batch_is_full(kt, U, NW, nkt)) {
    batch(kt, std::false_type{}, first);
    kt = next_batch(kt, U, NW);
    if (batch_is_full(kt, U, NW, nkt)) {
      batch(kt, std::false_type{}, second);
      kt = next_batch(kt, U, NW);
      for (; batch_is_full(kt, U, NW, nkt); kt = next_batch(kt, U, NW)) batch(kt, std::false_type{}, nothing);
      if (kt < nkt) batch(kt, std::true_type{}, nothing);
    } else {
      if (kt < nkt) batch(kt, std::true_type{}, nothing);
      second();
    }
  } else {
    if (kt < nkt) batch(kt, std::true_type{}, first);
    else first();
    second();
  }
}

// NB is chosen by the host per launch: 1 when the activations have one term (fp32) or the
// columns fold (at most 8), else 2.  Separate instantiations keep the common one-fragment path
// free of the second path's registers.  x[p]: the operand of pass p (all passes have ncols columns).
template <typename T, int RT, int NB, int NP, class Meanwhile>
__device__ __forceinline__ void gemm_accumulate(const u32x4* const (&w)[RT], const T* const (&x)[NP], int K, int ncols, int NW,
                                                f32x4 (&acc)[NP][RT], int w_lane, int w_stride, const Meanwhile& meanwhile) {
  constexpr int EPL = Tr<T>::EPL, KT = Tr<T>::KT, PARTS = Tr<T>::PARTS;
  const int lane = threadIdx.x & 63;
  const int nkt = K / KT;
  const u32x4* xp[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) xp[p] = reinterpret_cast<const u32x4*>(x[p]);
  uint32_t x_lane[NB];
  bool colok = false;
  const u32x4* const(&xc)[NP] = xp;
  const uint32_t(&xl)[NB] = x_lane;
  gemm_loop<T, RT, NB, NP>(w, xc, xl, xtile_stride<T>(ncols), colok, nkt, NW, acc, w_lane, w_stride, [&](auto when) {
    meanwhile(when);
    if (decltype(when)::value != 0) return;
    // NB == 1: lane column c < ncols reads the hi term of column c, column ncols + c its lo term
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const long o = x_fragment_elems(EPL, PARTS, NB, ncols, K, lane, q);
      colok = o >= 0;  // the same for every q
      x_lane[q] = (uint32_t)(colok ? o : 0) * sizeof(T);
    }
  });
}

// After its stream a workgroup's waves put their partial tiles into LDS, [wave][row tile][16 columns][kRedPitch] floats, and a thread
// each adds up and finishes the elements (row, column) of the tiles: element i has row i % 16, column i / 16.
// A launch's start and end are bound by instructions: a wave issues one in four cycles or more, so a hundred of them in a row
// are a fifth of a microsecond that nothing hides.  One wave that finished four elements a lane and folded the terms by
// shuffles did four times the instructions at a launch's end; operands of the end, the norm's scale and the kernel's own
// dimensions stood in front of its first load (215 to 447 instructions, now 70 to 120).  us a call, before and after both: 6-token calibration
// of the 8B shape 3354 -> 3225 (195 launches), draft step 2698 -> 2642 (107), prefill of 16 tokens 4055 -> 3983, tree levels of 4 and
// 12 nodes 5986 -> 5828, Qwen2-7B step 2660 -> 2617.
constexpr int kRedPitch = 20;  // bank spread; rows of four stay 16-byte pieces
ES_HD constexpr int red_floats(int nw, int rt) { return nw * rt * (kMaxCols * kRedPitch); }
template <int RT>
__device__ __forceinline__ void put_partials(const f32x4 (&acc)[RT], float* red) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* d = red + red_floats(wave, RT) + (lane & 15) * kRedPitch + (lane >> 4) * 4;
#pragma unroll
  for (int r = 0; r < RT; ++r) *reinterpret_cast<f32x4*>(d + red_floats(r, 1)) = acc[r];
}
// Element (row, col) of row tile r: the waves in order, the lo-term column (when the contraction ran folded) onto the hi-term one.
template <typename T, int RT>
__device__ __forceinline__ float tile_sum(const float* red, int NW, int r, int row, int col, int ncols) {
  const float* p = red + red_floats(r, 1) + col * kRedPitch + row;
  const bool fold = folded<T>(ncols);
  const int lo = fold ? ncols * kRedPitch : 0;
  float s = 0.f, l = 0.f;
  auto add = [&](auto n, const float* q) {  // straight-line: the reads go out together
    float v[decltype(n)::value], u[decltype(n)::value];
#pragma unroll
    for (int w = 0; w < decltype(n)::value; ++w) {
      v[w] = q[red_floats(w, RT)];
      if (Tr<T>::PARTS == 2) u[w] = q[red_floats(w, RT) + lo];
    }
#pragma unroll
    for (int w = 0; w < decltype(n)::value; ++w) {
      s += v[w];
      if (Tr<T>::PARTS == 2) l += u[w];
    }
  };
  if (NW == 8) {
    add(std::integral_constant<int, 8>{}, p);
  } else if (NW == 4) {
    add(std::integral_constant<int, 4>{}, p);
  } else if (NW == 7) {
    add(std::integral_constant<int, 7>{}, p);
  } else {
#pragma unroll 1
    for (int w = 0; w < NW; ++w) add(std::integral_constant<int, 1>{}, p + red_floats(w, RT));
  }
  return fold ? s + l : s;
}

// Sum over aligned groups of N lanes (8, 16 or 32), every lane of a group receiving the total,
// with data-parallel-primitive operand swizzles (lane^1 and lane^2 inside quads, then the
// mirrored lane of the other half of 8 and of 16 lanes) instead of LDS permutes.  Same operand
// pairs as an xor butterfly, hence the same bits.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int N>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(N == 8 || N == 16 || N == 32, "group size");
  v += dpp_f32<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_f32<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_f32<0x141>(v);  // row_half_mirror
  if (N >= 16) v += dpp_f32<0x140>(v);  // row_mirror
  if (N >= 32) v += __shfl_xor(v, 16, 64);
  return v;
}
// ... and over all 64, without a trip through LDS; the maximum likewise
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_f32<0xB1>(v));
  v = fmaxf(v, dpp_f32<0x4E>(v));
  v = fmaxf(v, dpp_f32<0x141>(v));
  v = fmaxf(v, dpp_f32<0x140>(v));
  const uint32_t a = __float_as_uint(v);
  const auto q = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  const uint32_t b = __float_as_uint(fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1])));
  const auto h = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
}
__device__ __forceinline__ float wave_sum(float v) {
  const uint32_t a = __float_as_uint(group_sum<16>(v));
  const auto q = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  const uint32_t b = __float_as_uint(__uint_as_float(q[0]) + __uint_as_float(q[1]));
  const auto h = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}

// rstd[col] = rsqrt(sum_t ssp[col][t] / d + eps), summed in a fixed order; a barrier has to follow.
__device__ __forceinline__ void compute_rstd(const float* __restrict__ ssp, int ntile, int ncols, int NW, float inv_d, float eps,
                                             float* s_rstd) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int col = wave; col < ncols; col += NW) {
    float s = 0.f;
    for (int t = lane; t < ntile; t += 64) s += ssp[col * ntile + t];
    s = wave_sum(s);
    if (lane == 0) s_rstd[col] = 1.0f / sqrtf(s * inv_d + eps);
  }
}

// The same quantity with its loads issued behind the first batch of weights and its arithmetic done
// behind the second's requests (gemm_loop, meanwhile): neither stands in front of the stream, and the L2
// latency of the partial sums does not sit in the tail of the kernel.  Covers d <= 4096 and up to two columns per
// wave (the common cases); otherwise rstd_finish falls back to compute_rstd.  Same summation
// order as compute_rstd, so both give identical bits.
struct RstdPre {
  float v[2][4];
  bool fast;
};

__device__ __forceinline__ void rstd_issue(const float* __restrict__ ssp, int ntile, int ncols, int NW, RstdPre& p) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  p.fast = ntile <= 256 && ncols <= 2 * NW;
  if (!p.fast) return;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int col = wave + i * NW;
#pragma unroll
    for (int j = 0; j < 4; ++j) p.v[i][j] = 0.f;
    if (col >= ncols) continue;  // uniform
    const float* row = ssp + col * ntile;
#pragma unroll
    for (int j = 0; j < 4; ++j) p.v[i][j] = lane + 64 * j < ntile ? row[lane + 64 * j] : 0.f;
  }
}

// A barrier has to follow.
__device__ __forceinline__ void rstd_finish(const float* __restrict__ ssp, int ntile, int ncols, int NW, float inv_d, float eps,
                                            const RstdPre& p, float* s_rstd) {
  if (!p.fast) {
    compute_rstd(ssp, ntile, ncols, NW, inv_d, eps, s_rstd);
    return;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int col = wave + i * NW;
    if (col >= ncols) break;  // uniform
    const float s = wave_sum(p.v[i][0] + p.v[i][1] + p.v[i][2] + p.v[i][3]);
    if (lane == 0) s_rstd[col] = 1.0f / sqrtf(s * inv_d + eps);
  }
}

// argmax order: the lowest index on ties
__device__ __forceinline__ bool better(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }

// the entry of a wide pass that column col belongs to
__device__ __forceinline__ int span_entry(const Spans& sp, int col) {
  int e = 0;
#pragma unroll
  for (int i = 1; i < kWideSeqs; ++i) e += (int)(i < sp.n_seq) & (int)(col >= sp.first[i]);
  return e;
}

extern __shared__ f32x4 dyn_red[];

// Kernel argument of a launch that serves two passes: their arguments and columns side by side.  Those kernels
// are compiled for workgroups of at most kTwinThreads threads (room for 256 registers per lane).
constexpr int kTwinThreads = 512;
template <typename Args>
struct Twin {
  Args a[2];
  Cols c[2];
};
// pass p's piece of the reduction buffer
template <int RT>
__device__ __forceinline__ float* red_of_pass(int p, int NW) {
  return reinterpret_cast<float*>(dyn_red) + p * red_floats(NW, RT);
}

}  // namespace es
