// Decode attention kernels of the EasySpec draft hot path (gfx950): the vector-ALU split-KV kernel,
// the matrix-core kernel for groups of columns of one sequence, the merge of split-KV partials;
// how a launch cuts the contexts; and their launch wrappers.
#include "launch_common.hpp"

#include <limits.h>

#include "../../include/easyspec.h"

namespace es {

// ------------------------------------------------------------------------------------------
// Decode attention over the KV caches of a set's layers, split along the context.
// One workgroup = (column and context chunk, KV head, layer); it serves the G query heads that
// share the KV head.  A K or V row (hd elements) is spread over LPS lanes, 16 bytes each, so a
// wave load covers SPW = 64/LPS consecutive slots (1 KB, coalesced).  Each wave walks its own
// contiguous run of slots in batches of IT loads per operand, all issued before the first is
// used, with a running (max, sum, accumulator) per query head: scores and probabilities never
// leave registers, since K and V fragments of a slot sit in the same lanes.  The four waves'
// states are combined through LDS; if the context has more than one chunk the workgroup
// writes a partial (max, sum, accumulator) per head and attn_merge_kernel combines the chunks.
// For bf16 caches with 128-element heads and four to eight query heads per KV head the scores come
// from the matrix cores instead (K rows staged through the wave's own LDS into MFMA A fragments,
// the queries as two bf16 terms): the vector ALUs keep the softmax of one head per lane and P.V.
// ------------------------------------------------------------------------------------------
struct AttnArgs {
  const float* Q;
  const void* kc;
  const void* vc;
  float* PO;
  float* PM;
  float* PL;
  void* AO;
  int layer0, Hq, Hkv, B, max_ctx;
  int even;        // vector kernel: every column has the same number of chunks
  int n;           // columns, or groups of them
  float inv_n;     // 1 / n
  int CH;       // matrix-core kernel: slots per chunk (0: the vector kernel)
  int nch_ref;  // wide passes: partials of a head
  int log2_nwv; // vector kernel: waves per workgroup, 4 or 8
  int direct;   // vector kernel: LDS holds the state of every slot group (see the kernel's last part)
  float scale;
};

// The split-KV cut of one column for the vector kernel: its nb units (of `unit` slots, the smallest step of a wave) are dealt to
// nch = round(nb * nch_ref / nb_ref) chunks whose unit counts differ by at most one, the longer ones first, so that a context of
// a power-of-two length plus a few drafted tokens does not leave a sliver of a chunk.  The host works out count, quotient and
// remainder for every column (ChunkMap): the kernels divide by nothing.  Four divisions by run-time numbers, two of them in 64 bits, the
// grid's decoding and the launch's own dimensions stood before a wave's first load of K, 870 instructions in all, and behind the
// chunk the slot groups were folded one LDS read after the other.  Attention and merge, us a call, before and after: 8B draft step
// 139 -> 129, 6-token calibration 457 -> 440, 16 tokens at context 8192 (matrix cores) 770 -> 744, tree levels 384 -> 370,
// Qwen2-7B step 144 -> 136; contexts 4096 .. 32768 unchanged.
struct ColumnCut {
  int32_t nch, quot, rest;
};
inline ColumnCut column_cut(int nch_ref, int nb_ref, int n_slots, int unit) {
  const int nb = (n_slots + unit - 1) / unit;
  int nch = (int)(((long)nb * nch_ref + nb_ref / 2) / nb_ref);
  nch = nch > nb ? nb : nch;
  nch = nch < 1 ? 1 : nch;
  return ColumnCut{nch, nb / nch, nb % nch};
}
// slots [s0, s1) of chunk `chunk` < nch
__host__ __device__ __forceinline__ void chunk_range(const ColumnCut& cut, int n_slots, int unit, int chunk, int& s0, int& s1) {
  const int u0 = chunk * cut.quot + (chunk < cut.rest ? chunk : cut.rest);
  s0 = u0 * unit;
  s1 = (u0 + cut.quot + (chunk < cut.rest ? 1 : 0)) * unit;
  s1 = s1 < n_slots ? s1 : n_slots;
}

// The run [w0, w1) of wave `wave` of 2^log2_nwv inside the chunk [s0, s1): the chunk's units dealt evenly.
__host__ __device__ __forceinline__ void wave_range(int s0, int s1, int unit, int wave, int log2_nwv, int& w0, int& w1) {
  const int n_units = (s1 - s0 + unit - 1) / unit;
  w0 = s0 + (wave * n_units >> log2_nwv) * unit;
  w1 = s0 + ((wave + 1) * n_units >> log2_nwv) * unit;
  w1 = w1 < s1 ? w1 : s1;
}

constexpr int kAttnIT = 8;       // loads in flight per operand per lane
constexpr int kAttnSmallIT = 2;  // the same for the short steps that finish a wave's share

template <typename T, int HD>
struct AttnGeom {
  static constexpr int EPL = Tr<T>::EPL, LPS = HD / EPL, SPW = 64 / LPS;
  static constexpr int WAVE_SLOTS = kAttnIT * SPW;    // slots one wave covers per batch
  static constexpr int UNIT = kAttnSmallIT * SPW;     // and per small step: the granularity of the split
};

extern __shared__ float dyn_f[];

// The chunks of a launch's columns: column i has col[i].cut.nch of them, and its workgroups, [KV head][chunk], are
// those from first[i] on of the grid's first extent.  Columns of unequal length have unequal numbers of chunks; a
// grid of (longest column's chunks) x KV heads x columns left its empty workgroups on the same XCDs again and again
// (workgroup ids go to the eight XCDs in turn): contexts 4096 / 8192 / 16384 / 32768, attention and merge of a one-layer
// set 64 -> 48 us, of a four-layer set 173 -> 166 (Qwen2-7B shape 37 -> 32, 112 -> 89).  Columns of one sequence keep
// the distance of whole columns, a multiple of eight with eight KV heads, and so the XCD on which they meet each
// other's K and V.
// Columns of equal chunk counts (AttnArgs::even: one sequence, most batches of like lengths) keep the plain grid (chunk,
// KV head, layer x column), which needs no division to find its place.
// What a workgroup has to know of its column lies together: one scalar load.
struct ColumnWork {
  ColumnCut cut;
  int32_t n_slots, seq, pad[3];
};
struct ChunkMap {
  int32_t first[kMaxCols];  // first workgroup of a column (its first chunk's number times Hkv); INT_MAX: no such column
  ColumnWork col[kMaxCols];
};
// layer and column (group) of a grid index layer * n + column: no division (both are small: off by far less than half a step)
__device__ __forceinline__ void layer_and_column(const AttnArgs& a, int z, int& li, int& col) {
  li = __builtin_amdgcn_readfirstlane((int)(((float)z + 0.5f) * a.inv_n));
  col = z - li * a.n;
}

// TREE: the columns are nodes of token trees and carry a visibility mask; without it every
// slot up to the column's own is visible and the mask logic costs no registers.
template <typename T, int HD, int G, bool TREE>
__global__ __launch_bounds__(512) void attn_kernel(AttnArgs a, Cols c, ChunkMap map) {
  typedef AttnGeom<T, HD> Geo;
  constexpr int EPL = Geo::EPL, LPS = Geo::LPS, SPW = Geo::SPW, IT = kAttnIT;
  int li, col, kvh, chunk;
  if (a.even) {
    chunk = blockIdx.x;
    kvh = blockIdx.y;
    layer_and_column(a, blockIdx.z, li, col);
  } else {
    li = blockIdx.y;
    col = 0;
#pragma unroll
    for (int i = 1; i < kMaxCols; ++i) col += (int)blockIdx.x >= map.first[i];
    const int of_col = blockIdx.x - map.first[col], chunks = map.col[col].cut.nch;
    kvh = (int)(((float)of_col + 0.5f) / (float)chunks);  // of_col < kMaxChunks * Hkv: off by far less than half a step
    kvh = __builtin_amdgcn_readfirstlane(kvh);
    chunk = of_col - kvh * chunks;
  }
  const ColumnWork cw = map.col[col];
  const int n_slots = cw.n_slots;
  // slots below vis_base are all visible; slot vis_base + i (i < 64) only if bit i is set (the
  // column's row of a token tree's mask).  Causal columns have vis_base = n_slots.
  const int vbase = TREE ? c.vis_base[col] : 0;
  const unsigned long long vmask = TREE ? c.vis_mask[col] : 0;
  const int nch = cw.cut.nch;
  if (chunk >= nch) return;
  int s0, s1;
  chunk_range(cw.cut, n_slots, Geo::UNIT, chunk, s0, s1);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), NWV = 1 << a.log2_nwv;  // 4 or 8 waves
  const int sub = lane / LPS, e0 = (lane % LPS) * EPL;

  const size_t rowbase = (((size_t)(a.layer0 + li) * a.B + cw.seq) * a.Hkv + kvh) * (size_t)a.max_ctx;
  // wave-uniform row bases; a lane's fragment of slot s lies s * HD + e0 elements further (32-bit offsets)
  const char* kb = reinterpret_cast<const char*>(reinterpret_cast<const T*>(a.kc) + rowbase * HD);
  const char* vb = reinterpret_cast<const char*>(reinterpret_cast<const T*>(a.vc) + rowbase * HD);
  constexpr uint32_t ROW_BYTES = HD * sizeof(T);
  const uint32_t lane_byte = e0 * sizeof(T);
  const int HQ = a.Hq * HD;

  float q[G][EPL], acc[G][EPL], m_run[G], l_run[G];
  // one head per lane (see the batch code): running maximum and sum of that head only
  // ... and, for bf16 caches and four to eight query heads per KV head, the scores themselves from the
  // matrix cores: a tile of 16 slots x 32 elements of K is the A operand, the queries (two bf16 terms,
  // hi and lo, one product each) the B operand with the heads repeated over the 16 columns.  With four
  // heads lane l receives the score of head 2 (l & 1) + ((l >> 1) & 1), the head the vector path leaves
  // there, and probabilities travel as quad broadcasts; with more, lane l has head l % 8 and the
  // probabilities of a batch go through a few hundred bytes of the wave's LDS, where every lane of a
  // slot's row reads all heads' values back (same address for the whole row: a broadcast).
  constexpr bool kScoresByMfma = LPS == 16 && G >= 4 && std::is_same<T, bf16_t>::value;
  constexpr bool kHeadPerLane = (G == 4 && LPS == 16) || kScoresByMfma;
  constexpr bool kQuadHeads = G == 4;
  constexpr int QKT = kScoresByMfma ? HD / 32 : 1;
  // per slot row (sub): 8 heads x 8 probabilities, 8 rescale factors, 4 floats of padding (bank spread)
  constexpr int kShareRow = 76;
  bf16x8 qh[QKT], ql[QKT];
  float m1 = -INFINITY, l1 = 0.f;
  const bool odd1 = lane & 1, odd2 = lane & 2;
  const int head_l = kQuadHeads ? 2 * (lane & 1) + ((lane >> 1) & 1) : min(lane & 7, G - 1);  // this lane's head
  // the lane's B fragments of the queries: requested here, split into their two bf16 terms only after the
  // wave's first K and V rows have been requested too (split_q), so that the two latencies overlap
  float q_raw[QKT][8];
  if constexpr (kScoresByMfma) {
    const float* qp = a.Q + ((size_t)li * kMaxCols + col) * HQ + (kvh * G + head_l) * HD + (lane >> 4) * 8;
#pragma unroll
    for (int kt = 0; kt < QKT; ++kt)
#pragma unroll
      for (int e = 0; e < 8; ++e) q_raw[kt][e] = qp[kt * 32 + e];
  }
  auto split_q = [&] {
#pragma unroll
    for (int kt = 0; kt < QKT; ++kt) {
      // the compiler would move the conversions, and with them the wait for the queries, in front of the requests for K and V
#pragma unroll
      for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(q_raw[kt][e]));
      split_bf16x8(q_raw[kt], qh[kt], ql[kt]);
    }
  };
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const float* qp = a.Q + ((size_t)li * kMaxCols + col) * HQ + (kvh * G + g) * HD + e0;
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      if constexpr (!kScoresByMfma) q[g][j] = qp[j];
      acc[g][j] = 0.f;
    }
    m_run[g] = -INFINITY;
    l_run[g] = 0.f;
  }

  // The chunk's units are dealt evenly to the waves, each taking a contiguous run [w0, w1): full
  // batches of IT loads per operand (all issued before the first is used) while more than two
  // small steps' worth is left, then small steps, so that a wave's arithmetic follows its share
  // of the slots.  Slots past w1 fetch the run's last row instead (their scores are discarded
  // below): unconditional loads, no branch per load.
  int w0, w1;
  wave_range(s0, s1, Geo::UNIT, wave, a.log2_nwv, w0, w1);
  auto fetch_k = [&](auto n_loads, int base, u32x4* kr) {
#pragma unroll
    for (int j = 0; j < decltype(n_loads)::value; ++j) {
      const int s = min(base + j * SPW + sub, w1 - 1);
      kr[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kb + ((uint32_t)s * ROW_BYTES + lane_byte)));
    }
  };
  auto fetch_v = [&](auto n_loads, int base, u32x4* vr) {
#pragma unroll
    for (int j = 0; j < decltype(n_loads)::value; ++j) {
      const int s = min(base + j * SPW + sub, w1 - 1);
      vr[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vb + ((uint32_t)s * ROW_BYTES + lane_byte)));
    }
  };
  // One batch: kr, vr hold its K and V rows.  `staged` runs once the K registers are free again (matrix-core
  // scores only: the rows sit in LDS by then), which is where the next batch is requested.
  auto consume = [&](auto n_loads, int base, u32x4* kr, const u32x4* vr, auto&& staged) {
    constexpr int N = decltype(n_loads)::value;
    // K for the matrix cores: tile t holds 16 slots; A row r = lane % 16 carries slot
    // (r % 4) * 4 + r / 4 of the tile, so that the score of the slot this lane's V load j = 4 t + i
    // brings (slot 4 i + sub of the tile) comes out in this lane, element i of the tile's result.
    // The rows are loaded whole (coalesced, as for the vector products) and turned into A fragments
    // through the wave's own 8 KB of LDS, the 16-byte pieces of slot row s XORed by s % 16 so that
    // neither the row-wise stores nor the fragment reads meet a bank twice.
    constexpr int NT = kScoresByMfma ? (N + 3) / 4 : 1;
    u32x4 ka[NT][QKT];
    if constexpr (kScoresByMfma) {
      u32x4* stage = reinterpret_cast<u32x4*>(dyn_f) + wave * (IT * SPW * LPS);
#pragma unroll
      for (int j = 0; j < N; ++j) stage[stage_store_piece(lane, j)] = kr[j];
      __builtin_amdgcn_wave_barrier();  // LDS operations of one wave execute in order: no wait is needed
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int kt = 0; kt < QKT; ++kt) ka[t][kt] = stage[stage_fetch_piece(lane, t, kt)];
      __builtin_amdgcn_wave_barrier();  // the reads are issued before the next batch's stores
      staged();
    }
    if constexpr (kHeadPerLane) {
      // Four query heads over a 16-lane row: instead of four row-wide sums per slot, the lanes
      // trade partial dot products pairwise so that lane l ends up with the row's total for head
      // 2 (l & 1) + ((l >> 1) & 1) alone; the softmax arithmetic is then done once per lane
      // (one head) and the probability of head g comes back to the row's other lanes as a
      // quad broadcast on its way into the P.V products.
      float sc1[N];
      f32x4 st[NT];
      if constexpr (kScoresByMfma) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          f32x4 s_hi = {0.f, 0.f, 0.f, 0.f}, s_lo = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kt = 0; kt < QKT; ++kt) {
            s_hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[t][kt]), qh[kt], s_hi, 0, 0, 0);
            s_lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[t][kt]), ql[kt], s_lo, 0, 0, 0);
          }
          st[t] = s_hi + s_lo;
        }
      }
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const int s = base + j * SPW + sub;
        const bool valid = (int)(s < w1) & (int)(!TREE || (int)(s < vbase) | (int)((vmask >> ((s - vbase) & 63)) & 1ull));  // straight-line
        if constexpr (kScoresByMfma) {
          sc1[j] = valid ? st[j / 4][j % 4] * a.scale : -INFINITY;
        } else {
          float kv[EPL];
          unpack<T>(kr[j], kv);
          float d[4];
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            d[g] = 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) d[g] += q[g][e] * kv[e];
          }
          const float t0 = (odd1 ? d[2] : d[0]) + dpp_f32<0xB1>(odd1 ? d[0] : d[2]);  // lane ^ 1
          const float t1 = (odd1 ? d[3] : d[1]) + dpp_f32<0xB1>(odd1 ? d[1] : d[3]);
          float v = (odd2 ? t1 : t0) + dpp_f32<0x4E>(odd2 ? t0 : t1);                  // lane ^ 2
          v += dpp_f32<0x124>(v);  // row_ror:4
          v += dpp_f32<0x128>(v);  // row_ror:8
          sc1[j] = valid ? v * a.scale : -INFINITY;
        }
      }
      float bm = sc1[0];
#pragma unroll
      for (int j = 1; j < N; ++j) bm = fmaxf(bm, sc1[j]);
      const float m_new = fmaxf(m1, bm);
      const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // see the general path below
      const float alpha = __expf(m1 - m_ref);
      m1 = m_new;
      l1 *= alpha;
      if constexpr (kQuadHeads) {
        const float al[4] = {dpp_f32<0x00>(alpha), dpp_f32<0xAA>(alpha), dpp_f32<0x55>(alpha), dpp_f32<0xFF>(alpha)};
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[g][e] *= al[g];
#pragma unroll
        for (int j = 0; j < N; ++j) {
          float vv[EPL];
          unpack<T>(vr[j], vv);
          const float p = __expf(sc1[j] - m_ref);  // 0 for slots past the end or masked
          l1 += p;
          // head g sits in quad lane 0, 2, 1, 3 for g = 0 .. 3
          const float pg[4] = {dpp_f32<0x00>(p), dpp_f32<0xAA>(p), dpp_f32<0x55>(p), dpp_f32<0xFF>(p)};
#pragma unroll
          for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[g][e] += pg[g] * vv[e];
        }
      } else {
        // lanes 0..7 of a slot row put their head's probabilities and rescale factor into the wave's LDS
        // (the K tiles are in registers by now); every lane then reads all heads' values of its row
        constexpr int NP = (N + 3) / 4;  // 16-byte pieces of probabilities per head
        float* share = dyn_f + wave * (IT * SPW * LPS * 4) + sub * kShareRow;
        float pj[4 * NP];
#pragma unroll
        for (int j = 0; j < 4 * NP; ++j) {
          pj[j] = j < N ? __expf(sc1[j < N ? j : 0] - m_ref) : 0.f;  // 0 for slots past the end or masked
          l1 += pj[j];
        }
        if ((lane & 8) == 0) {
#pragma unroll
          for (int q4 = 0; q4 < NP; ++q4)
            *reinterpret_cast<f32x4*>(share + (lane & 7) * 8 + 4 * q4) = f32x4{pj[4 * q4], pj[4 * q4 + 1], pj[4 * q4 + 2], pj[4 * q4 + 3]};
          share[64 + (lane & 7)] = alpha;
        }
        __builtin_amdgcn_wave_barrier();  // LDS operations of one wave execute in order
        const f32x4 al0 = *reinterpret_cast<const f32x4*>(share + 64), al1 = *reinterpret_cast<const f32x4*>(share + 68);
        const float al[8] = {al0[0], al0[1], al0[2], al0[3], al1[0], al1[1], al1[2], al1[3]};
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int e = 0; e < EPL; ++e) acc[g][e] *= al[g];
#pragma unroll
        for (int q4 = 0; q4 < NP; ++q4) {  // four slots' probabilities of every head at a time (registers)
          f32x4 pg[G];
#pragma unroll
          for (int g = 0; g < G; ++g) pg[g] = *reinterpret_cast<const f32x4*>(share + g * 8 + 4 * q4);
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const int j = 4 * q4 + jj;
            if (j < N) {
              float vv[EPL];
              unpack<T>(vr[j], vv);
#pragma unroll
              for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[g][e] += pg[g][jj] * vv[e];
            }
          }
        }
        __builtin_amdgcn_wave_barrier();  // the reads are issued before the next batch's K rows overwrite the place
      }
      return;
    }
    float sc[N][G], m_use[G];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const int s = base + j * SPW + sub;
      const bool valid = (int)(s < w1) & (int)(!TREE || (int)(s < vbase) | (int)((vmask >> ((s - vbase) & 63)) & 1ull));  // straight-line
      float kv[EPL];
      unpack<T>(kr[j], kv);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float dot = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) dot += q[g][e] * kv[e];
        dot = group_sum<LPS>(dot);
        sc[j][g] = valid ? dot * a.scale : -INFINITY;
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float bm = sc[0][g];
#pragma unroll
      for (int j = 1; j < N; ++j) bm = fmaxf(bm, sc[j][g]);
      // The running maximum belongs to the slot group (the LPS lanes that share slots), not to the
      // wave: no cross-lane traffic per batch; the groups are brought to a common reference once,
      // after the loop.  A group whose slots so far were all past the end or masked still has
      // -inf: the exponentials then take 0 as reference and give 0 instead of exp(-inf + inf).
      const float m_new = fmaxf(m_run[g], bm);
      const float m_ref = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = __expf(m_run[g] - m_ref);  // exp(-inf) = 0 on the first batch
      m_run[g] = m_new;
      m_use[g] = m_ref;
      l_run[g] *= alpha;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[g][e] *= alpha;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      float vv[EPL];
      unpack<T>(vr[j], vv);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float p = __expf(sc[j][g] - m_use[g]);  // 0 for slots past the end or masked
        l_run[g] += p;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] += p * vv[e];
      }
    }
  };
  auto process = [&](auto n_loads, int base) {
    u32x4 kr[decltype(n_loads)::value], vr[decltype(n_loads)::value];
    fetch_k(n_loads, base, kr);
    fetch_v(n_loads, base, vr);
    consume(n_loads, base, kr, vr, [] {});
  };
  int base = w0;  // wave-uniform, like the loop conditions
  constexpr std::integral_constant<int, IT> kFull{};
  auto full_batch_at = [&](int b) { return w1 - b > 2 * Geo::UNIT; };
  if constexpr (kScoresByMfma) {
    if (full_batch_at(base)) {
      u32x4 kr[IT], vr[IT];
      fetch_k(kFull, base, kr);
      fetch_v(kFull, base, vr);
      split_q();
      if constexpr (kQuadHeads) {
        // With the scores on the matrix cores the vector arithmetic of a batch no longer hides the
        // latency of the next one's loads behind other waves' work, so a wave keeps two batches in
        // flight: K of the next batch goes into the registers the staging has just freed, V into a
        // second set of registers.  (More heads: no registers left for that set.)
        u32x4 vn[IT];
        while (full_batch_at(base + Geo::WAVE_SLOTS)) {  // another full batch follows: request it, work on this one
          const int next = base + Geo::WAVE_SLOTS;
          consume(kFull, base, kr, vr, [&] {
            fetch_k(kFull, next, kr);
            fetch_v(kFull, next, vn);
            asm volatile("" ::: "memory");  // the requests stay here: the compiler would sink them to their first use
          });
          base = next;
#pragma unroll
          for (int j = 0; j < IT; ++j) vr[j] = vn[j];
        }
      }
      consume(kFull, base, kr, vr, [] {});  // four heads: the wave's last full batch
      base += Geo::WAVE_SLOTS;
    } else {
      split_q();
    }
  }
  for (; full_batch_at(base); base += Geo::WAVE_SLOTS) process(kFull, base);
  // At most two units are left.  Vector scores: both in one step (one latency instead of two).  Scores from the matrix
  // cores: a step each; a third shape of the batch code costs the 7-head instantiation more than the latency
  // (Qwen2-7B shape, context 4096: 2677 us a draft step against 2651).
  if constexpr (kScoresByMfma) {
    for (; base < w1; base += Geo::UNIT) process(std::integral_constant<int, kAttnSmallIT>{}, base);
  } else {
    if (w1 - base > Geo::UNIT) process(std::integral_constant<int, 2 * kAttnSmallIT>{}, base);
    else if (base < w1) process(std::integral_constant<int, kAttnSmallIT>{}, base);
  }

  if constexpr (kHeadPerLane && !kQuadHeads) {  // back to every lane holding all heads' maximum and sum: through LDS
    float* share = dyn_f + wave * (IT * SPW * LPS * 4) + sub * kShareRow;
    if ((lane & 8) == 0) {
      share[lane & 7] = m1;
      share[8 + (lane & 7)] = l1;
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int g = 0; g < G; ++g) {
      m_run[g] = share[g];
      l_run[g] = share[8 + g];
    }
  }
  if constexpr (kScoresByMfma) __syncthreads();  // the combination below reuses the LDS the K tiles went through
  if constexpr (kHeadPerLane && kQuadHeads) {  // back to every lane holding all four heads' maximum and sum
    const float mm[4] = {dpp_f32<0x00>(m1), dpp_f32<0xAA>(m1), dpp_f32<0x55>(m1), dpp_f32<0xFF>(m1)};
    const float ll[4] = {dpp_f32<0x00>(l1), dpp_f32<0xAA>(l1), dpp_f32<0x55>(l1), dpp_f32<0xFF>(l1)};
#pragma unroll
    for (int g = 0; g < G; ++g) {
      m_run[g] = mm[g & 3];
      l_run[g] = ll[g & 3];
    }
  }

  // Combine the NWV * SPW slot groups of the workgroup (l_run counts each slot once per group,
  // every lane of a group holds the same value).  A group, or a whole chunk of a tree column,
  // may have seen no visible slot: its maximum is -inf, its sums 0, and its weight below 0.
  const size_t arow = (size_t)li * kMaxCols + col;
  auto emit = [&](int g, int e, float m, float l, float o0, float o1) {  // outputs e, e + 1 of head g
    const int head = kvh * G + g;
    if (nch == 1) {
      T* dst = reinterpret_cast<T*>(a.AO) + (size_t)li * Tr<T>::PARTS * kMaxCols * HQ;
      store_act1<T>(dst + xoff<T>(c.n, HQ, col, head * HD + e), (size_t)kMaxCols * HQ, o0 / l);
      store_act1<T>(dst + xoff<T>(c.n, HQ, col, head * HD + e + 1), (size_t)kMaxCols * HQ, o1 / l);
    } else {
      const size_t row = arow * a.Hq + head;
      *reinterpret_cast<float2*>(a.PO + (row * kMaxChunks + chunk) * HD + e) = make_float2(o0, o1);
      if (e == 0) {
        a.PM[row * kMaxChunks + chunk] = m;
        a.PL[row * kMaxChunks + chunk] = l;
      }
    }
  };
  if (a.direct) {
    // every group's state goes to LDS as it stands; each thread then folds all groups for two
    // adjacent outputs (no cross-lane traffic at all)
    const int P = NWV * SPW, p = wave * SPW + sub;
    float* w_acc = dyn_f;              // [P][G][HD]
    float* w_m = dyn_f + P * G * HD;   // [G][P]
    float* w_l = w_m + G * P;          // [G][P]
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int e = 0; e < EPL; e += 4)
        *reinterpret_cast<f32x4*>(w_acc + (p * G + g) * HD + e0 + e) = f32x4{acc[g][e], acc[g][e + 1], acc[g][e + 2], acc[g][e + 3]};
    }
    if (lane % LPS == 0) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        w_m[g * P + p] = m_run[g];
        w_l[g * P + p] = l_run[g];
      }
    }
    __syncthreads();
    auto fold = [&](auto n_groups) {
      constexpr int N = decltype(n_groups)::value;
      for (int idx = tid; idx < G * HD / 2; idx += 64 * NWV) {
        const int g = idx / (HD / 2), e = (idx % (HD / 2)) * 2;
        // sixteen groups at a time, everything of theirs read before it is used (all 32 or 64 of heads of 64 elements at once
        // took 168 to 312 bytes of scratch a lane with four to eight heads, and 148 instead of 123 registers with two)
        constexpr int PER = N < 16 ? N : 16;
        float m = -INFINITY, mm[PER], ll[PER];
        float2 v[PER];
        auto maxima = [&](int q0) {
#pragma unroll
          for (int q = 0; q < PER; q += 4) {
            const f32x4 m4 = *reinterpret_cast<const f32x4*>(w_m + g * N + q0 + q);
#pragma unroll
            for (int i = 0; i < 4; ++i) mm[q + i] = m4[i];
          }
        };
        auto sums = [&](int q0) {
#pragma unroll
          for (int q = 0; q < PER; q += 4) {
            const f32x4 l4 = *reinterpret_cast<const f32x4*>(w_l + g * N + q0 + q);
#pragma unroll
            for (int i = 0; i < 4; ++i) ll[q + i] = l4[i];
          }
#pragma unroll
          for (int q = 0; q < PER; ++q) v[q] = *reinterpret_cast<const float2*>(w_acc + ((q0 + q) * G + g) * HD + e);
        };
        auto largest = [&] {
#pragma unroll
          for (int q = 0; q < PER; ++q) m = fmaxf(m, mm[q]);
        };
        maxima(0);
        if constexpr (N == PER) sums(0);
        largest();
        if constexpr (N > PER) {
#pragma unroll 1
          for (int q0 = PER; q0 < N; q0 += PER) {
            maxima(q0);
            largest();
          }
        }
        const float m_ref = m == -INFINITY ? 0.f : m;
        float l = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll 1
        for (int q0 = 0; q0 < N; q0 += PER) {
          if constexpr (N > PER) {
            maxima(q0);
            sums(q0);
          }
#pragma unroll
          for (int q = 0; q < PER; ++q) {  // in group order: the result does not depend on timing
            const float wgt = __expf(mm[q] - m_ref);
            l += ll[q] * wgt;
            o0 += v[q].x * wgt;
            o1 += v[q].y * wgt;
          }
        }
        emit(g, e, m, l, o0, o1);
      }
    };
    if (NWV == 4) fold(std::integral_constant<int, 4 * SPW>{});
    else fold(std::integral_constant<int, 8 * SPW>{});
  } else {
    // LDS too small for every group: the groups of a wave are combined with shuffles first
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float mw = m_run[g];
#pragma unroll
      for (int off = LPS; off < 64; off <<= 1) mw = fmaxf(mw, __shfl_xor(mw, off, 64));
      const float rescale = m_run[g] == -INFINITY ? 0.f : __expf(m_run[g] - mw);
      m_run[g] = mw;
      l_run[g] *= rescale;
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[g][e] *= rescale;
#pragma unroll
      for (int off = LPS; off < 64; off <<= 1) {
        l_run[g] += __shfl_xor(l_run[g], off, 64);
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[g][e] += __shfl_xor(acc[g][e], off, 64);
      }
    }
    float* w_acc = dyn_f;                 // [NWV][G][HD]
    float* w_m = dyn_f + NWV * G * HD;    // [NWV][G]
    float* w_l = w_m + NWV * G;           // [NWV][G]
    if (sub == 0) {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < EPL; ++e) w_acc[(wave * G + g) * HD + e0 + e] = acc[g][e];
    }
    if (lane == 0) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        w_m[wave * G + g] = m_run[g];
        w_l[wave * G + g] = l_run[g];
      }
    }
    __syncthreads();
    for (int idx = tid; idx < G * HD / 2; idx += 64 * NWV) {
      const int g = idx / (HD / 2), e = (idx % (HD / 2)) * 2;
      float m = w_m[g];
      for (int w = 1; w < NWV; ++w) m = fmaxf(m, w_m[w * G + g]);
      const float m_ref = m == -INFINITY ? 0.f : m;
      float l = 0.f, o0 = 0.f, o1 = 0.f;
      for (int w = 0; w < NWV; ++w) {
        const float wgt = __expf(w_m[w * G + g] - m_ref);
        l += w_l[w * G + g] * wgt;
        o0 += w_acc[(w * G + g) * HD + e] * wgt;
        o1 += w_acc[(w * G + g) * HD + e + 1] * wgt;
      }
      emit(g, e, m, l, o0, o1);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Attention on the matrix cores (bf16 caches).  The query rows that share one KV head — the G
// heads of up to 16 NW / G columns of one sequence (the tokens of a calibration, the nodes of a tree
// level) — are the columns of NW MFMA tiles of 16, one tile per wave of the workgroup, so K and V
// are read once per group of columns and the per-slot arithmetic leaves the vector ALUs:
//   S^T[slot][row]  = K[slot][:] . Q[row][:]      A = K (rows = slots), B = Q^T, two-term bf16 q (queries_in_fp32: three)
//   O^T[e][row]    += V^T[e][slot] P^T[slot][row]  A = V^T, B = P^T, two-term bf16 p (wide passes, AttnCut::three: three)
// A workgroup walks its chunk of the context in super tiles of 64 slots: its waves load the K and V
// rows of a tile together (coalesced) and put them into LDS (XOR-swizzled 16-byte pieces; V is read
// back with the transposing LDS read), each wave then takes its own 16 query rows through scores,
// softmax and P.V.  One split-KV partial per query row and chunk (merged by attn_merge_kernel;
// written out directly if the column's whole context is one chunk).  The slots of a super tile are
// dealt to the four S^T tiles so that lane (row r, quarter q) ends up with the 16 CONSECUTIVE slots
// q*16 .. q*16+15: the accumulator layout of S^T is then the B-operand layout of the P.V
// instruction, and a V^T fragment is 8 consecutive slots.
// What bounds it is the dependent chain of one tile in a wave (loads, LDS, scores, softmax, P.V).
// Sharing the tile between the waves reads K and V once for up to 64 query rows and leaves a wave
// few enough registers (its share of the tile instead of all of it) that two or more run on a SIMD.
// Before (every wave alone with up to 16 query rows and a tile of its own, one wave per SIMD) and now: prefill of
// 16 tokens at context 8192 4482 -> 4098 us; tree levels of 4 and 12 nodes at context 2048 6089 -> 5970 us together on one
// box, 6075 -> 6018 on another.  (4 x 6 tokens at contexts 4096 .. 32768 as two passes of 12 columns, which they no
// longer run as: 7353 -> 6570 us.)  Two row tiles per wave instead (one chain for 32 rows): 4553 us for the prefill, 6171 for
// the levels; the registers of a private 64-slot tile leave one wave per SIMD.
// grid = (chunks, Hkv, k * groups), block = 64 * NW.
// ------------------------------------------------------------------------------------------
struct ColGroups {
  int32_t n;  // groups
  struct Group {
    int32_t first, count, seq;  // columns (consecutive, same sequence); count * G <= 16 NW
    int32_t n_max, n_all;       // slots the longest of them attends to; slots below this one are visible to all
    int32_t pad[3];
  } g[kMaxCols];
};
// What the kernel asks about its columns: those of a pass of at most kMaxCols (PassCols), or of a wide pass, whose
// columns are given by sequence (SpanCols).
template <int PT>
struct PassCols {
  Cols c;
  ColGroups cg;
  static constexpr bool kWide = false;
  static constexpr int kQueryTerms = 2;
  static constexpr int kProbTerms = PT;  // bf16 terms of a probability: two or three (AttnCut::three)
};
template <int QT>
struct SpanCols {
  Spans sp;
  int32_t n;                       // groups
  int32_t first_group[kWideSeqs];  // first group of entry e (INT_MAX: no such entry)
  int32_t most;                    // columns of a full group
  static constexpr bool kWide = true;
  static constexpr int kQueryTerms = QT;  // bf16 terms of a query: two or three (queries_in_fp32)
  static constexpr int kProbTerms = 3;
};
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));

template <int HD, bool TREE, int NW, class Src>
__global__ __launch_bounds__(64 * NW, NW == 1 ? 1 : 2) void attn_mfma_kernel(AttnArgs a, Src src, int G) {
  constexpr int KT = HD / 32, ET = HD / 16, PIECES = HD / 8, NL = PIECES / NW;
  __shared__ u32x4 kt_lds[64 * PIECES], vt[64 * PIECES];  // [64 slots][PIECES] 16-byte pieces each, swizzled
  __shared__ bool s_odd[NW];  // causal columns: a wave's part of the V tile holds something that is not finite
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int chunk = blockIdx.x, kvh = blockIdx.y;
  int li = 0, grp = blockIdx.z;  // wide passes are one layer
  if constexpr (!Src::kWide) layer_and_column(a, blockIdx.z, li, grp);
  int first, cnt, seq, pos_first = 0;  // the group's columns, their sequence, the position of its first (wide passes)
  int n_max;  // slots the longest column of the group attends to
  int n_all;  // slots below this one are visible to every column of the group
  if constexpr (Src::kWide) {
    int e = 0;
#pragma unroll
    for (int i = 1; i < kWideSeqs; ++i) e += grp >= src.first_group[i];
    const int skip = (grp - src.first_group[e]) * src.most;
    first = src.sp.first[e] + skip;
    cnt = min(src.most, src.sp.first[e + 1] - first);
    seq = src.sp.seq[e];
    pos_first = src.sp.pos0[e] + skip;
    n_max = pos_first + cnt;
    n_all = pos_first + 1;
  } else {
    const ColGroups::Group w = src.cg.g[grp];  // the host has gone through the columns: one scalar load instead of two a column
    first = w.first; cnt = w.count; seq = w.seq; n_max = w.n_max; n_all = w.n_all;
  }
  const int r = lane & 15, q4 = lane >> 4;  // query row (MFMA column) and quarter / k-group
  const int row = wave * 16 + r;
  const bool active = wave * 16 < cnt * G;  // wave-uniform: a wave without query rows only helps to load the tiles
  const bool row_ok = row < cnt * G;
  const int col = first + (row_ok ? row / G : 0), g = row_ok ? row % G : 0;
  const int ws0 = chunk * a.CH;
  if (ws0 >= n_max) return;  // whole workgroup
  const int ws1 = min(ws0 + a.CH, n_max);
  int n_slots, vbase = 0;  // of this lane's row
  unsigned long long vmask = 0;
  if constexpr (Src::kWide) {
    n_slots = pos_first + (col - first) + 1;
  } else {
    n_slots = src.c.pos[col] + 1;
    vbase = src.c.vis_base[col];
    vmask = src.c.vis_mask[col];
  }
  const int HQ = a.Hq * HD;
  const size_t rowbase = (((size_t)(a.layer0 + li) * a.B + seq) * a.Hkv + kvh) * (size_t)a.max_ctx;
  const u32x4* kc = reinterpret_cast<const u32x4*>(reinterpret_cast<const bf16_t*>(a.kc) + rowbase * HD);
  const u32x4* vc = reinterpret_cast<const u32x4*>(reinterpret_cast<const bf16_t*>(a.vc) + rowbase * HD);

  // This thread's pieces of a super tile: piece `piece` of slots sl0 + j * 64 NW / PIECES.  The registers are
  // free again once their contents sit in LDS, so the next tile is requested while the current one is still
  // being worked on; the first one before the queries are converted.
  // (They are requested behind this row's query all the same: loads return in order.)
  // Loads are unconditional: a slot past the chunk's end (only the last chunk of the longest column has any:
  // chunks are multiples of 64 slots) re-reads the last row; its scores are masked below for every query row,
  // so its probabilities are exact zeros.
  const int piece = tid % PIECES, sl0 = tid / PIECES;
  constexpr int SL = 64 * NW / PIECES;  // slots one load of the workgroup covers
  u32x4 kf[NL], vf[NL];
  const char* kb = reinterpret_cast<const char*>(kc);
  const char* vb = reinterpret_cast<const char*>(vc);
  auto request = [&](int base) {
    if (base + 64 <= ws1) {  // uniform: a whole tile lies one constant apart (32-bit offsets: a head's rows are at most 16 MB)
      const uint32_t at = (uint32_t)(base + sl0) * (HD * 2) + piece * 16;
#pragma unroll
      for (int j = 0; j < NL; ++j) kf[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kb + (at + j * (SL * HD * 2))));
#pragma unroll
      for (int j = 0; j < NL; ++j) vf[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vb + (at + j * (SL * HD * 2))));
    } else {
#pragma unroll
      for (int j = 0; j < NL; ++j) kf[j] = __builtin_nontemporal_load(kc + (size_t)min(base + sl0 + j * SL, ws1 - 1) * PIECES + piece);
#pragma unroll
      for (int j = 0; j < NL; ++j) vf[j] = __builtin_nontemporal_load(vc + (size_t)min(base + sl0 + j * SL, ws1 - 1) * PIECES + piece);
    }
  };
  // The query in 16-byte pieces, unconditionally (a padding row takes the group's first; its results are dropped): an element at a
  // time under the row's condition, behind the first tile, a launch took 6.1 us to its first products.  us a call, before and now:
  // prefill of 16 tokens at context 8192 3862 -> 3757, tree levels of 4 and 12 nodes 5595 -> 5537, 4 x 6 tokens at 4096 .. 32768
  // 5219 -> 5157, 16 x 16 tokens 9410 -> 9220.
  f32x4 q_raw[KT][2];
  {
    const float* qp = a.Q + ((size_t)li * kMaxCols + col) * HQ + (kvh * G + g) * HD + q4 * 8;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int h = 0; h < 2; ++h) q_raw[kt][h] = *reinterpret_cast<const f32x4*>(qp + kt * 32 + h * 4);
  }
  asm volatile("" ::: "memory");
  request(ws0);

  // B operands of S^T: this row's query, hi and lo bf16 terms, k-group q4 of every k-tile; a third term where asked for
  constexpr bool Q3 = Src::kQueryTerms == 3;
  bf16x8 qh[KT], ql[KT], qr[Q3 ? KT : 1];
  {
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        x[e] = q_raw[kt][e >> 2][e & 3];
        asm volatile("" : "+v"(x[e]));  // behind the requests, the conversions too
      }
      split_bf16x8(x, qh[kt], ql[kt]);
      if constexpr (Q3) qr[kt] = third_bf16x8(x, qh[kt], ql[kt]);
    }
  }

  f32x4 o[ET];
#pragma unroll
  for (int et = 0; et < ET; ++et) o[et] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;  // m_run: of the unscaled scores; l_run: this lane's 16 slots per super tile only
  const float scale2 = a.scale * 1.44269504088896340736f;  // log2(e)
  auto sees = [&](int slot) {  // this lane's row
    // no short circuit: the shift amount is masked instead of guarded, so that this stays straight-line code
    const bool seen = !TREE || (int)(slot < vbase) | (int)((vmask >> ((slot - vbase) & 63)) & 1ull);
    return (bool)((int)row_ok & (int)(slot < n_slots) & (int)seen);
  };

  for (int base = ws0; base < ws1; base += 64) {
    if (base > ws0) __syncthreads();  // every wave has read the previous tile
    const bool edge = base + 64 > n_all;  // workgroup-uniform: some query row does not see the whole super tile
    // A slot that a row does not see has the probability zero, which leaves the row alone only if V is finite there:
    // infinities and NaNs are taken out of those slots and put back below, for the rows that see theirs.  (Causal columns
    // only: a tree's nodes share their siblings' infinities, in the vector kernel too.  Prefill of 16 tokens at context 8192:
    // attention and merge 13.2 -> 13.3 us a layer.)
    if (!TREE && edge) {
      bool mine = false;  // wave-uniform
#pragma unroll
      for (int j = 0; j < NL; ++j) {
        if (base + (j + 1) * SL <= n_all) continue;  // uniform: slots that every row sees
        if (__builtin_amdgcn_ballot_w64(any_nonfinite(vf[j])) != 0) {
          vf[j] = clear_nonfinite(vf[j]);
          mine = true;
        }
      }
      if (lane == 0) s_odd[wave] = mine;
    }
    // K rows as the four score tiles take them: slot sl is row m = (sl / 16) * 4 + sl % 4 of tile t = (sl / 4) % 4;
    // piece p of row m is stored at p ^ m, so that the 16 rows of one piece hit 16 different banks.
    // V rows in order, the 32-byte blocks of slot s XORed by s % 4: the transposing reads below take the same
    // block of four consecutive slots at once, which then lie in different banks.
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int sl = sl0 + j * SL, t = (sl >> 2) & 3, m = (sl >> 4) * 4 + (sl & 3);
      kt_lds[(t * 16 + m) * PIECES + (piece ^ (m & (PIECES - 1)))] = kf[j];
    }
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int sl = sl0 + j * SL;
      vt[sl * PIECES + (piece ^ ((sl & 3) << 1))] = vf[j];
    }
    __syncthreads();
    if (base + 64 < ws1) request(base + 64);
    if (!active) continue;
    // scores of this lane's row against its 16 slots base + q4*16 + t*4 + i
    f32x4 st[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) st[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < KT; ++kt) {
      u32x4 ka[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) ka[t] = kt_lds[(t * 16 + r) * PIECES + ((kt * 4 + q4) ^ (r & (PIECES - 1)))];
#pragma unroll
      for (int t = 0; t < 4; ++t) st[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[t]), qh[kt], st[t], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < 4; ++t) st[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[t]), ql[kt], st[t], 0, 0, 0);
      if constexpr (Q3) {
#pragma unroll
        for (int t = 0; t < 4; ++t) st[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[t]), qr[kt], st[t], 0, 0, 0);
      }
    }
    // Scores stay unscaled: scale and log2(e) go into the exponential's argument, one fused multiply-add per score
    if (edge) {  // padding rows elsewhere get scores of the group's first query; they are never stored
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) st[t][i] = sees(base + q4 * 16 + t * 4 + i) ? st[t][i] : -INFINITY;
    }
    float bm = -INFINITY;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) bm = fmaxf(bm, st[t][i]);
    bm = fmaxf(bm, __shfl_xor(bm, 16, 64));  // the four quarters of a row must share the reference:
    bm = fmaxf(bm, __shfl_xor(bm, 32, 64));  // their slots are summed by one instruction below
    const float m_new = fmaxf(m_run, bm);
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // nothing visible so far: exponentials give 0
    const float ref2 = m_ref * scale2;
    const float alpha = __builtin_amdgcn_exp2f((m_run - m_ref) * scale2);
    m_run = m_new;
    l_run *= alpha;
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {  // wave-uniform: once the running maxima have settled nothing is rescaled
#pragma unroll
      for (int et = 0; et < ET; ++et) o[et] *= alpha;
    }
    // B operands of P.V: MFMA number h takes slots q4*16 + h*8 .. +8 of this lane = tiles 2h, 2h+1
    // Wide passes, and launches that are here by attn_mfma_rows alone, carry probabilities in three terms, all 24 bits: the vector
    // kernel, whose the shorter contexts among them would otherwise be, keeps probabilities in fp32.
    bf16x8 ph[2], pl[2], pr[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float pv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        pv[j] = __builtin_amdgcn_exp2f(fmaf(st[2 * h + (j >> 2)][j & 3], scale2, -ref2));
        l_run += pv[j];
      }
      split_bf16x8(pv, ph[h], pl[h]);
      if constexpr (Src::kProbTerms == 3) pr[h] = third_bf16x8(pv, ph[h], pl[h]);
    }
    // A operands: V^T row e = et*16 + lane%16, the 8 slots q4*16 + h*8 + j, by the LDS transposing
    // read (ds_read_b64_tr_b16): in a group of 16 lanes, lane i offers the 8 bytes at its address
    // (4 elements of "row" i) and receives element i%4 of rows i/4, i/4 + 4, i/4 + 8, i/4 + 12.
    // With row 4j + c = (slot s0 + j, elements e0 + 4c .. +3), lane i receives V[s0 + j][e0 + i],
    // j = 0..3: four consecutive slots of its own V^T row.  Two reads per 8-slot k-group.
#pragma unroll
    for (int et = 0; et < ET; ++et) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        v4i16 half[2];
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
          const int slot = q4 * 16 + h * 8 + t2 * 4 + (r >> 2);  // this lane's row of the transposed block
          const int vp = (et * 2 + ((r & 3) >> 1)) ^ ((slot & 3) << 1);
          const char* src = reinterpret_cast<const char*>(vt) + slot * (HD * 2) + vp * 16 + (r & 1) * 8;
          half[t2] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(src));
        }
        const v8i16 both = {half[0][0], half[0][1], half[0][2], half[0][3], half[1][0], half[1][1], half[1][2], half[1][3]};
        const bf16x8 va = __builtin_bit_cast(bf16x8, both);
        o[et] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, ph[h], o[et], 0, 0, 0);
        o[et] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pl[h], o[et], 0, 0, 0);
        if constexpr (Src::kProbTerms == 3) o[et] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pr[h], o[et], 0, 0, 0);
      }
    }
    bool odd = false;
    if (!TREE && edge) {
#pragma unroll
      for (int k = 0; k < NW; ++k) odd |= s_odd[k];
    }
    if (!TREE && __builtin_amdgcn_ballot_w64(odd) != 0) {  // an infinity or a NaN times a positive probability is itself; slots past the chunk's end are seen by no row
      const char* v = reinterpret_cast<const char*>(vc) + q4 * 8;
#pragma unroll 1
      for (int slot = base; slot < min(base + 64, ws1); ++slot) {
        if (!sees(slot)) continue;
#pragma unroll
        for (int et = 0; et < ET; ++et) {
          u32x2 x = *reinterpret_cast<const u32x2*>(v + (size_t)slot * (HD * 2) + et * 32);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float f = __uint_as_float(i & 1 ? x[i >> 1] & 0xFFFF0000u : x[i >> 1] << 16);
            if (!(fabsf(f) < INFINITY)) o[et][i] += f;
          }
          __builtin_amdgcn_sched_barrier(0);  // one load at a time: no registers for a path that is hardly ever taken
        }
      }
    }
  }

  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if (!row_ok || ws0 >= n_slots) return;  // padding rows; columns that end before this chunk
  const int head = kvh * G + g;
  if (n_slots <= a.CH) {  // the whole context
#pragma unroll
    for (int et = 0; et < ET; ++et) {
      const int e = et * 16 + q4 * 4;
      bf16_t* dst = reinterpret_cast<bf16_t*>(a.AO);
      size_t part;
      if constexpr (Src::kWide) {
        dst += wide_off(HQ, col, head * HD + e);
        part = kWidePart;
      } else {
        dst += (size_t)li * 2 * kMaxCols * HQ + xoff<bf16_t>(src.c.n, HQ, col, head * HD + e);
        part = (size_t)kMaxCols * HQ;
      }
      store_act4<bf16_t>(dst, part, o[et][0] / l_run, o[et][1] / l_run, o[et][2] / l_run, o[et][3] / l_run);
    }
  } else {
    const size_t prow = ((size_t)li * kMaxCols + col) * a.Hq + head;  // wide passes are one layer: li = 0
    const size_t pitch = Src::kWide ? a.nch_ref : kMaxChunks;
#pragma unroll
    for (int et = 0; et < ET; ++et)
      *reinterpret_cast<f32x4*>(a.PO + (prow * pitch + chunk) * HD + et * 16 + q4 * 4) = o[et];
    if (q4 == 0) {
      a.PM[prow * pitch + chunk] = m_run * a.scale;
      a.PL[prow * pitch + chunk] = l_run;
    }
  }
}

// Merge the chunk partials of one (layer, column, query head), chunks in order.  Runs as its own
// launch: the kernel boundary is what makes the partials written by workgroups on other XCDs
// visible (a device-scope fence inside the attention kernel costs an L2 write-back per workgroup
// and was measured several times slower).  Columns whose context fits one chunk were finished by
// attn_kernel.  A wave per head, HD / 64 adjacent elements per lane, the chunks' weights a lane each and
// handed round by scalar reads: no LDS, no barrier, one memory latency.  W waves to a workgroup: W heads of a
// column, or, in a wide pass, one head of W columns, whose outputs lie side by side in the operand (16 bytes each; with
// eight columns whole lines leave from one workgroup).  grid = (columns, ceil(Hq / W), k), or (ceil(columns / W), Hq).
// us a launch, a workgroup per head (weights through LDS, a barrier) and now: 256 columns of 32 heads 12.9 -> 7.4 (8192 workgroups
// took that long to start); 6 columns 4.65 and 4.65, a launch's floor.  Partials past the first 16 by 24 instead of 8 at
// a time: 24 columns with up to 64 chunks 7.6 -> 6.7.
// Src: MergeCols, or Spans for the columns of a wide pass (chunks of CH slots, partials nch_ref apart, wide operand).
// The columns of a merge launch: those of a pass with their chunk counts, or of a wide pass.
struct MergeCols {
  int32_t n;
  int32_t nch[kMaxCols];
};
template <typename T, int HD, int W, class Src>
__global__ __launch_bounds__(64 * W) void attn_merge_kernel(AttnArgs a, Src c) {
  constexpr bool kWide = std::is_same<Src, Spans>::value;
  constexpr int VE = HD / 64;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = kWide ? blockIdx.x * W + wave : blockIdx.x, head = kWide ? blockIdx.y : blockIdx.y * W + wave, li = blockIdx.z;
  int nch;
  size_t pitch = kMaxChunks;
  if (col >= c.n || head >= a.Hq) return;
  if constexpr (kWide) {
    const int en = span_entry(c, col);
    nch = (c.pos0[en] + (col - c.first[en]) + a.CH) / a.CH;
    pitch = a.nch_ref;
  } else {
    nch = c.nch[col];
  }
  if (nch == 1) return;
  const int HQ = a.Hq * HD, e = lane * VE;
  const size_t row = ((size_t)li * kMaxCols + col) * a.Hq + head;
  // every load is issued up front: the first 16 chunk partials of this lane's output elements (all
  // of them for contexts up to 16 chunks) together with the chunk maxima and sums
  const float* po = a.PO + row * pitch * HD + e;
  auto partial = [&](int u, float (&v)[VE]) {
    const float* p = po + (size_t)u * HD;
    if constexpr (VE == 2) {
      const float2 x = u < nch ? *reinterpret_cast<const float2*>(p) : make_float2(0.f, 0.f);
      v[0] = x.x;
      v[1] = x.y;
    } else {
      v[0] = u < nch ? *p : 0.f;
    }
  };
  const float pm = lane < nch ? a.PM[row * pitch + lane] : -INFINITY;  // one lane per chunk: at most 64
  const float pl = lane < nch ? a.PL[row * pitch + lane] : 0.f;
  float pv[16][VE];
#pragma unroll
  for (int u = 0; u < 16; ++u) partial(u, pv[u]);
  const float wgt = __expf(pm - wave_max(pm)), tot = wave_sum(pl * wgt);
  float o[VE] = {};
  auto add = [&](int u, const float (&v)[VE]) {  // u is uniform; past the last chunk both factors are 0
    const float w = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wgt), u));
#pragma unroll
    for (int i = 0; i < VE; ++i) o[i] += v[i] * w;
  };
#pragma unroll
  for (int u = 0; u < 16; ++u) add(u, pv[u]);
  for (int c0 = 16; c0 < nch; c0 += 24) {
    float pw[24][VE];
#pragma unroll
    for (int u = 0; u < 24; ++u) partial(c0 + u, pw[u]);  // independent loads
#pragma unroll
    for (int u = 0; u < 24; ++u) add(c0 + u, pw[u]);
  }
  T* dst = reinterpret_cast<T*>(a.AO);
  size_t part;
  if constexpr (kWide) {
    dst += wide_off(HQ, col, head * HD + e);
    part = kWidePart;
  } else {
    dst += (size_t)li * Tr<T>::PARTS * kMaxCols * HQ + xoff<T>(c.n, HQ, col, head * HD + e);
    part = (size_t)kMaxCols * HQ;
  }
  if constexpr (VE == 2) store_act2<T>(dst, part, o[0] / tot, o[1] / tot);
  else store_act1<T>(dst, part, o[0] / tot);
}
template <typename T, int HD, bool TREE>
static void launch_attn_g(int G, dim3 grid, int nwv, hipStream_t st, AttnArgs a, const Cols& c, const ChunkMap& map) {
  // partial state of every slot group of the workgroup if that fits the default 64 KB of
  // dynamic LDS, else of every wave
  const int groups = nwv * AttnGeom<T, HD>::SPW;
  a.direct = (size_t)groups * G * (HD + 2) * sizeof(float) <= 65536 ? 1 : 0;
  const int sets = a.direct ? groups : nwv;
  size_t lds = (size_t)sets * G * (HD + 2) * sizeof(float);
  // scores from the matrix cores (four query heads per KV head, bf16 caches): 8 KB per wave for the K tiles
  if (G >= 4 && AttnGeom<T, HD>::LPS == 16 && std::is_same<T, bf16_t>::value)
    lds = std::max(lds, (size_t)nwv * kAttnIT * AttnGeom<T, HD>::SPW * HD * sizeof(T));
  const dim3 blk(64 * nwv);
  switch (G) {
    case 1: ES_LAUNCH((attn_kernel<T, HD, 1, TREE>), grid, blk, lds, st, a, c, map); break;
    case 2: ES_LAUNCH((attn_kernel<T, HD, 2, TREE>), grid, blk, lds, st, a, c, map); break;
    case 4: ES_LAUNCH((attn_kernel<T, HD, 4, TREE>), grid, blk, lds, st, a, c, map); break;
    case 7: ES_LAUNCH((attn_kernel<T, HD, 7, TREE>), grid, blk, lds, st, a, c, map); break;
    case 8: ES_LAUNCH((attn_kernel<T, HD, 8, TREE>), grid, blk, lds, st, a, c, map); break;
    default: break;  // rejected at create
  }
}

// Matrix-core attention or the vector-ALU kernel?  The MFMA kernel reads K and V once per group of columns of a sequence and does
// the per-slot arithmetic on the matrix cores.  It takes bf16 launches that hold several columns of a sequence and
//   * enough (column, layer, slot) work, over several layers or at least five columns (attn_mfma_long), or
//   * heads of 128 elements, four or more per KV head, contexts of more than one piece, and at least 12 query rows of a sequence,
//     three quarters of a tile (attn_mfma_rows): calibrations of three tokens or more (two with seven or eight heads), short ones
//     too.  With four heads such a sequence has to have at least half of the longest context: a tile that a longer, lone column fills
//     by a quarter is the time of the launch then.
// Single columns (plain draft steps) stay on the vector kernel.  EASYSPEC_ATTN_MFMA = 0 / 2 forces never / always (bf16 only).
// The second line was drawn when the kernel had lost 2.7 us of its start; us a call of 12 layers on the vector and the matrix-core kernel with
// three terms to a probability.  8B shape, 3 / 4 / 6 / 8 / 12 tokens at context 300 1022 / 1081 / 1114 / 1126 / 1214 and 1028 / 1079 / 1109 /
// 1127 / 1210, at 2048 1103 / 1109 / 1162 / 1192 / 1315 and 1105 / 1107 / 1145 / 1167 / 1248, at 4096 1139 / 1151 / 1232 / 1274 / 1612 and
// 1137 / 1140 / 1178 / 1192 / 1279; 2 tokens (two terms) at 2048 1095 and 1099, at 8192 1162 and 1181.  Qwen2-7B shape, 3 / 6 / 12 tokens at
// 600 1187 / 1233 / 1394 and 1168 / 1214 / 1389, at 2048 1206 / 1261 / 1444 and 1180 / 1234 / 1408.  Two tree levels of 3 / 6 / 12
// nodes at 600, sets of four, 8B 1880 / 2063 / 2196 and 1869 / 2033 / 2121.  6-token calibration at 2048, 32 layers: 3094 -> 3057.
// Mixed passes, tokens of the sequences at their contexts.  8B: 3 and 1 at 100 and 16 000 1157 and 1197, 3000 and 16 000 1182 and 1257, 1000
// and 6000 1095 and 1115, 600 and 2000 1043 and 1051, 2000 and 2000 1059 and 1061, 2000 and 600 1079 and 1053; 3 and 2 at 1000 and 4000 1117 and
// 1134; 3 and nine times 1 at 700 1211 and 1207, at 1500 1300 and 1276.  Qwen2-7B shape, 3 and 1 at the same: 1211 and 1220, 1247 and 1245, 1174
// and 1172, 1144 and 1113, 1134 and 1121, 1139 and 1120; 2 tokens at 300 / 2048 / 8192 1119 / 1140 / 1202 and 1112 / 1126 / 1190.  Eight
// heads per KV head, 2 tokens at 300 / 2048 / 8192 1057 / 1079 / 1173 and 1012 / 1027 / 1092, 3 and 1 at 100 and 16 000 1192 and 1131.
static bool attn_mfma_long(const Cols& c, int n_set) {
  const long min_work = env_int("EASYSPEC_ATTN_MFMA_MIN", 30000);
  bool shared = false;
  int max_len = 1;
  for (int i = 0; i < c.n; ++i) {
    shared = shared || (i > 0 && c.seq[i] == c.seq[i - 1]);
    max_len = std::max(max_len, c.pos[i] + 1);
  }
  return shared && (long)n_set * c.n * max_len >= min_work && (n_set > 1 || c.n >= 5);
}
static int longest_run(const Cols& c) {
  int longest = 1;
  for (int i = 1, run = 1; i < c.n; ++i) {
    run = c.seq[i] == c.seq[i - 1] ? run + 1 : 1;
    longest = std::max(longest, run);
  }
  return longest;
}
constexpr int kAttnOnePiece = 256;  // contexts up to here are one piece (attn_cut)
static bool attn_mfma_heads(const Shape& s) { return s.hd == 128 && s.Hq / s.Hkv >= 4; }
static bool attn_mfma_rows(const Shape& s, const Cols& c) {
  const int G = s.Hq / s.Hkv;
  int max_len = 1, max_filled = 0;
  for (int i = 0; i < c.n;) {
    int j = i, len = 1;
    for (; j < c.n && c.seq[j] == c.seq[i]; ++j) len = std::max(len, c.pos[j] + 1);
    if (j - i > 1 && (j - i) * G >= 12) max_filled = std::max(max_filled, len);
    max_len = std::max(max_len, len);
    i = j;
  }
  return attn_mfma_heads(s) && max_len > kAttnOnePiece && max_filled > 0 && (G >= 7 || 2 * max_filled >= max_len);
}
static bool attn_use_mfma(const Shape& s, const Cols& c, int n_set) {
  const int mode = env_int("EASYSPEC_ATTN_MFMA", 1);  // read at every call: tests switch it between contexts
  if (mode == 0 || s.dtype != 1) return false;
  return mode == 2 || attn_mfma_long(c, n_set) || attn_mfma_rows(s, c);
}

// Waves per workgroup of the matrix-core kernel = tiles of 16 query rows that share K and V: as many as the
// longest run of columns of one sequence fills (1, 2 or 4).
static int row_tiles(const Cols& c, int G) {
  const int forced = env_int("EASYSPEC_ATTN_ROW_TILES", 0);  // tests: read at every call
  if (forced == 1 || forced == 2 || forced == 4) return forced;
  const int tiles = (longest_run(c) * G + 15) / 16;
  return tiles <= 2 ? tiles : 4;
}

// Runs of consecutive columns of one sequence, cut so that a group's query rows (columns x G
// heads per KV head) fill at most the 16 columns of each of its MFMA tiles.
static void group_columns(const Cols& c, int G, int n_tiles, ColGroups& cg) {
  const int most = std::max(1, 16 * n_tiles / G);
  cg.n = 0;
  for (int i = 0; i < c.n;) {
    int j = i + 1;
    while (j < c.n && c.seq[j] == c.seq[i] && j - i < most) ++j;
    ColGroups::Group& g = cg.g[cg.n++];
    g.first = i; g.count = j - i; g.seq = c.seq[i]; g.n_max = 0; g.n_all = INT_MAX;
    for (; i < j; ++i) {
      g.n_max = std::max(g.n_max, c.pos[i] + 1);
      g.n_all = std::min(g.n_all, std::min(c.pos[i] + 1, c.vis_base[i]));  // causal columns: vis_base = pos + 1
    }
  }
}

AttnCut attn_cut(const Shape& s, const Cols& c, int n_set) {
  AttnCut cut;
  cut.mfma = attn_use_mfma(s, c, n_set);
  cut.three = cut.mfma && attn_mfma_heads(s) && !attn_mfma_long(c, n_set);
  cut.tiles = 1;
  cut.chunk = 0;
  cut.nb_ref = 0;
  int max_len = 1;
  for (int i = 0; i < c.n; ++i) max_len = std::max(max_len, c.pos[i] + 1);
  // Short contexts: one piece of work per (layer, column, KV head) walks the whole context, which
  // saves the merge launch; two dependent launches cost more than the narrower launch loses.
  static const int single_max = env_int("EASYSPEC_ATTN_SINGLE", kAttnOnePiece);
  if (cut.mfma) {
    // one workgroup per (group of columns, chunk, KV head), walking its chunk in super tiles of 64 slots: chunks of a
    // fixed length, grown until their count fits the partial buffers and the launch is not cut finer than max_wg
    ColGroups cg;
    cut.tiles = row_tiles(c, s.Hq / s.Hkv);
    group_columns(c, s.Hq / s.Hkv, cut.tiles, cg);
    const int unit = 64;
    if (max_len <= single_max) {
      cut.chunk = (max_len + unit - 1) / unit * unit;
      cut.n_chunks = 1;
      return cut;
    }
    int ch = unit;
    auto nch = [&](int ch_) { return (max_len + ch_ - 1) / ch_; };
    auto wgs = [&](int ch_) {
      long n = 0;
      for (int i = 0; i < cg.n; ++i) n += (c.pos[cg.g[i].first + cg.g[i].count - 1] + ch_) / ch_;
      return n * s.Hkv * n_set;
    };
    // Waves aimed at: eight per CU (two per SIMD hide each other's chains) while a workgroup still has four super
    // tiles to walk, four per CU below that (a launch of few tiles is all start and end): prefill of 16 tokens at
    // context 8192 4205 us with eight, 4090 us with four; 4 x 6 tokens at contexts 4096 .. 32768 6618 us with four,
    // 6403 us with eight, no better with 12 or 16.
    const long few = (long)cu_count() * 4 / cut.tiles, many = 2 * few;
    const long max_wg = std::max(few, std::min(many, wgs(unit) / 4));
    while (ch < 1024 && (nch(ch) > kMaxChunks || wgs(ch) > max_wg)) ch += unit;
    cut.chunk = ch;
    cut.n_chunks = nch(ch);
    return cut;
  }
  return attn_cut_vector(s, c, n_set);
}

AttnCut attn_cut_vector(const Shape& s, const Cols& c, int n_set) {
  AttnCut cut;
  cut.mfma = false;
  cut.three = false;
  cut.tiles = 1;
  cut.chunk = 0;
  int max_len = 1;
  for (int i = 0; i < c.n; ++i) max_len = std::max(max_len, c.pos[i] + 1);
  static const int single_max = env_int("EASYSPEC_ATTN_SINGLE", kAttnOnePiece);
  // Vector kernel: one workgroup of four waves per (chunk, KV head, layer, column).  Every column's
  // units (the slots of a wave's small step) are dealt evenly to its chunks (chunk_range) and a
  // chunk's units evenly to its waves, which work through them in full batches of four units and
  // up to two small steps.  The chunk count of the longest column is the one that minimises the
  // arithmetic of the busiest SIMD — (workgroups per CU, rounded up) x (cost of the busiest wave
  // of a workgroup) — and among equals the smallest (fewer partials to merge).
  const int lps = s.hd * (s.dtype == 1 ? 2 : 4) / 16;
  const int unit = kAttnSmallIT * (64 / lps);
  const int nb_max = (max_len + unit - 1) / unit;
  cut.nb_ref = nb_max;
  cut.n_chunks = 1;
  if (max_len <= single_max) return cut;
  const int forced = env_int("EASYSPEC_ATTN_NCH", 0);  // tests: a fixed count for the longest column, read at every call
  static const int n_cu = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
    return n;
  }();
  // cost of a wave with u units, in tenths of a full batch: a small step does a quarter of a
  // batch's slots at about a third of its time
  constexpr int per_batch = kAttnIT / kAttnSmallIT;
  auto wave_cost = [](long u) {
    const long full = u / per_batch, rest = u % per_batch;
    return 10 * full + (rest == 0 ? 0 : rest <= 2 ? 3 * rest + 1 : 10);
  };
  long best = -1;
  for (int nch = forced > 0 ? std::min(forced, nb_max) : 2; nch <= std::min(kMaxChunks, nb_max); ++nch) {
    long wgs = 0;
    for (int i = 0; i < c.n; ++i) {
      const int nb = (c.pos[i] + 1 + unit - 1) / unit;
      wgs += std::max(1, std::min(nb, (nb * nch + nb_max / 2) / nb_max));
    }
    wgs *= (long)s.Hkv * n_set;
    const long per_cu = (wgs + n_cu - 1) / n_cu;
    const long per_wave = ((nb_max + nch - 1) / nch + 3) / 4;  // units of the busiest wave
    const long score = per_cu * wave_cost(per_wave);
    if (best < 0 || score < best) {
      best = score;
      cut.n_chunks = nch;
    }
    if (forced > 0) break;
  }
  return cut;
}

// slots of a wave's smallest step
static int attn_unit(const Shape& s) { return kAttnSmallIT * (64 / (s.hd * (s.dtype == 1 ? 2 : 4) / 16)); }

int attn_waves(const AttnCut& cut) { return cut.n_chunks == 1 ? 8 : 4; }

void attn_ranges(const Shape& s, const AttnCut& cut, int n_slots, int chunk, int wave, int* nch, int* w0, int* w1) {
  const int unit = attn_unit(s);
  const ColumnCut cc = column_cut(cut.n_chunks, cut.nb_ref, n_slots, unit);
  *nch = cc.nch;
  if (chunk >= cc.nch) {
    *w0 = *w1 = 0;
    return;
  }
  int s0, s1;
  chunk_range(cc, n_slots, unit, chunk, s0, s1);
  wave_range(s0, s1, unit, wave, attn_waves(cut) == 8 ? 3 : 2, *w0, *w1);
}

void launch_attn(const Shape& s, const Buffers& b, const Cols& c, int layer0, int n_set, const AttnCut& cut, hipStream_t st) {
  const int n_chunks = cut.n_chunks;
  AttnArgs a;
  a.Q = b.Q; a.kc = b.kc; a.vc = b.vc; a.PO = b.PO; a.PM = b.PM; a.PL = b.PL; a.AO = b.AO;
  a.layer0 = layer0; a.Hq = s.Hq; a.Hkv = s.Hkv; a.B = s.B; a.max_ctx = s.max_ctx;
  a.CH = cut.chunk; a.nch_ref = cut.n_chunks;
  a.log2_nwv = attn_waves(cut) == 8 ? 3 : 2;
  a.scale = 1.0f / sqrtf((float)s.hd);
  const int G = s.Hq / s.Hkv;
  MergeCols mc;
  mc.n = c.n;
  // one chunk per context: eight waves share the whole context of a (layer, column, KV head) and
  // no merge launch is needed; several chunks: four waves per chunk
  const int nwv = attn_waves(cut);
  bool tree = false;  // any column that does not see every slot up to its own
  for (int i = 0; i < c.n; ++i) tree = tree || c.vis_base[i] <= c.pos[i];
  if (cut.mfma) {
    ColGroups cg;
    group_columns(c, G, cut.tiles, cg);
    a.n = cg.n;
    a.inv_n = 1.0f / (float)a.n;
    for (int i = 0; i < c.n; ++i) mc.nch[i] = (c.pos[i] + cut.chunk) / cut.chunk;
    const dim3 mg(n_chunks, s.Hkv, n_set * cg.n), blk(64 * cut.tiles);
    auto launch = [&](auto hd, auto is_tree, auto terms) {
      constexpr int HD = decltype(hd)::value;
      constexpr bool TREE = decltype(is_tree)::value;
      typedef PassCols<decltype(terms)::value> Src;
      Src src;
      src.c = c;
      src.cg = cg;
      if (cut.tiles == 4) ES_LAUNCH((attn_mfma_kernel<HD, TREE, 4, Src>), mg, blk, 0, st, a, src, G);
      else if (cut.tiles == 2) ES_LAUNCH((attn_mfma_kernel<HD, TREE, 2, Src>), mg, blk, 0, st, a, src, G);
      else ES_LAUNCH((attn_mfma_kernel<HD, TREE, 1, Src>), mg, blk, 0, st, a, src, G);
    };
    auto go = [&](auto hd, auto is_tree) {
      if constexpr (decltype(hd)::value == 128) {
        if (cut.three) return launch(hd, is_tree, std::integral_constant<int, 3>{});
      }
      launch(hd, is_tree, std::integral_constant<int, 2>{});
    };
    const std::integral_constant<int, 128> h128{};
    const std::integral_constant<int, 64> h64{};
    if (s.hd == 128 && tree) go(h128, std::true_type{});
    else if (s.hd == 128) go(h128, std::false_type{});
    else if (tree) go(h64, std::true_type{});
    else go(h64, std::false_type{});
  } else {
    ChunkMap map;
    int total = 0;
    a.even = 1;
    a.n = c.n;
    a.inv_n = 1.0f / (float)a.n;
    for (int i = 0; i < kMaxCols; ++i) {
      map.first[i] = i < c.n ? total * s.Hkv : INT_MAX;
      if (i >= c.n) continue;
      map.col[i].cut = column_cut(n_chunks, cut.nb_ref, c.pos[i] + 1, attn_unit(s));
      map.col[i].n_slots = c.pos[i] + 1;
      map.col[i].seq = c.seq[i];
      mc.nch[i] = map.col[i].cut.nch;
      total += mc.nch[i];
      if (mc.nch[i] != n_chunks) a.even = 0;
    }
    const dim3 grid = a.even ? dim3(n_chunks, s.Hkv, n_set * c.n) : dim3(total * s.Hkv, n_set);
    DISPATCH_T(s.dtype, {
      if (s.hd == 128 && tree) launch_attn_g<T, 128, true>(G, grid, nwv, st, a, c, map);
      else if (s.hd == 128) launch_attn_g<T, 128, false>(G, grid, nwv, st, a, c, map);
      else if (tree) launch_attn_g<T, 64, true>(G, grid, nwv, st, a, c, map);
      else launch_attn_g<T, 64, false>(G, grid, nwv, st, a, c, map);
    });
  }
  if (n_chunks > 1) {
    const dim3 mgrid(c.n, s.Hq, n_set);  // few: a wave each, so that they spread over the CUs
    DISPATCH_T(s.dtype, {
      if (s.hd == 128) ES_LAUNCH((attn_merge_kernel<T, 128, 1, MergeCols>), mgrid, dim3(64), 0, st, a, mc);
      else ES_LAUNCH((attn_merge_kernel<T, 64, 1, MergeCols>), mgrid, dim3(64), 0, st, a, mc);
    });
  }
}

// Would the vector kernel, with queries in fp32, take any of the passes of at most kMaxCols columns that a wide pass stands
// for?  (It holds them in fp32 with heads of 64 elements, or with one or two query heads per KV head.)  Then the wide launch takes
// queries in three bf16 terms, all 24 bits; otherwise in two, as those passes do.  Median error of a row against 64
// bits, one layer, 2048 wide, heads of 64: 6.8e-6 with two terms, 6.1e-6 with three and in passes of 16 columns.  8B shape
// (two terms on either route), 32 layers, 16 x 16 tokens at contexts 512 .. 1067, 32 draws: 6.4e-5 wide, 6.5e-5 in passes
// of 16 columns.  Where it is not needed the third term is not free: 9810 and 9890 us for that call, 5280 and 5330 us
// for 4 x 6 tokens at contexts 4096 .. 32768.
static bool queries_in_fp32(const Shape& s, const Spans& sp) {
  if (s.hd == 128 && s.Hq / s.Hkv >= 4) return false;
  Cols c;
  c.n = 0;
  for (int e = 0; e < sp.n_seq; ++e) {
    const int n = sp.first[e + 1] - sp.first[e];
    if (c.n + n > kMaxCols) {
      if (!attn_use_mfma(s, c, 1)) return true;
      c.n = 0;
    }
    for (int i = 0; i < n; ++i, ++c.n) c.seq[c.n] = sp.seq[e], c.pos[c.n] = sp.pos0[e] + i;
  }
  return !attn_use_mfma(s, c, 1);
}

// Attention of a wide pass: always the matrix-core kernel, one launch for the columns of every sequence.
template <int QT>
static void launch_wide_attn_terms(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, hipStream_t st) {
  const int G = s.Hq / s.Hkv;
  int longest = 1, max_len = 1;
  for (int e = 0; e < sp.n_seq; ++e) {
    const int n = sp.first[e + 1] - sp.first[e];
    longest = std::max(longest, n);
    max_len = std::max(max_len, sp.pos0[e] + n);
  }
  const int want = (longest * G + 15) / 16, tiles = want <= 2 ? want : 4;
  SpanCols<QT> src;
  src.sp = sp;
  src.most = std::max(1, 16 * tiles / G);
  src.n = 0;
  for (int e = 0; e < kWideSeqs; ++e) {
    src.first_group[e] = e < sp.n_seq ? src.n : INT_MAX;
    if (e < sp.n_seq) src.n += (sp.first[e + 1] - sp.first[e] + src.most - 1) / src.most;
  }
  // the cut of attn_cut's matrix-core kernel; the partials of all columns share the buffer that a set of
  // EASYSPEC_MAX_SET layers of kMaxCols columns has for its own
  const int unit = 64, most_chunks = std::min(kMaxChunks, EASYSPEC_MAX_SET * kMaxCols * kMaxChunks / ((sp.n + 15) / 16 * 16));
  auto nch = [&](int ch) { return (max_len + ch - 1) / ch; };
  auto wgs = [&](int ch) {
    long n = 0;
    for (int e = 0; e < sp.n_seq; ++e) {
      const int cols = sp.first[e + 1] - sp.first[e];
      n += (long)((cols + src.most - 1) / src.most) * ((sp.pos0[e] + cols + ch - 1) / ch);
    }
    return n * s.Hkv;
  };
  const long few = (long)cu_count() * 4 / tiles, many = 2 * few;
  const long max_wg = std::max(few, std::min(many, wgs(unit) / 4));
  int ch = unit;
  while (nch(ch) > most_chunks || (ch < 1024 && wgs(ch) > max_wg)) ch += unit;
  if (max_len <= 256) ch = (max_len + unit - 1) / unit * unit;  // as in attn_cut: no merge launch
  AttnArgs a;
  a.Q = w.Q; a.kc = b.kc; a.vc = b.vc; a.PO = b.PO; a.PM = b.PM; a.PL = b.PL; a.AO = w.AO;
  a.layer0 = layer; a.Hq = s.Hq; a.Hkv = s.Hkv; a.B = s.B; a.max_ctx = s.max_ctx;
  a.CH = ch; a.nch_ref = nch(ch); a.log2_nwv = 0; a.direct = 0; a.even = 0; a.n = src.n; a.inv_n = 0.f;
  a.scale = 1.0f / sqrtf((float)s.hd);
  const dim3 grid(a.nch_ref, s.Hkv, src.n), blk(64 * tiles);
  auto go = [&](auto hd) {
    constexpr int HD = decltype(hd)::value;
    if (tiles == 4) ES_LAUNCH((attn_mfma_kernel<HD, false, 4, SpanCols<QT>>), grid, blk, 0, st, a, src, G);
    else if (tiles == 2) ES_LAUNCH((attn_mfma_kernel<HD, false, 2, SpanCols<QT>>), grid, blk, 0, st, a, src, G);
    else ES_LAUNCH((attn_mfma_kernel<HD, false, 1, SpanCols<QT>>), grid, blk, 0, st, a, src, G);
    if (a.nch_ref > 1) ES_LAUNCH((attn_merge_kernel<bf16_t, HD, 8, Spans>), dim3(ceil_div(sp.n, 8), s.Hq), dim3(512), 0, st, a, sp);
  };
  if (s.hd == 128) go(std::integral_constant<int, 128>{});
  else go(std::integral_constant<int, 64>{});
}

void launch_wide_attn(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, hipStream_t st) {
  if (queries_in_fp32(s, sp)) launch_wide_attn_terms<3>(s, b, w, sp, layer, st);
  else launch_wide_attn_terms<2>(s, b, w, sp, layer, st);
}

}  // namespace es
