// Small kernels around the hot path (gfx950): weight repacking at load, greedy acceptance, KV cache
// import / export, the streaming-read probe; and their launch wrappers.
#include "launch_common.hpp"

#include <algorithm>

namespace es {

// ------------------------------------------------------------------------------------------
// Small utilities.
// ------------------------------------------------------------------------------------------

// Row-major [.][K] -> tiles of R <= 16 rows, per k-tile a fragment of [k-group 4][R rows] 16-byte
// pieces (1 KB for R = 16: piece i is lane i's share of an MFMA A operand); rows padded with zeros
// up to a multiple of R.  Packed row r is source row r (half = 0), or, for the rotary halves of
// stacked heads (half > 0), source row (r / half) * 2 * half + r % half + row_add: the first
// (row_add = 0) or second (row_add = half) half of head r / half.
template <typename T>
__global__ void repack_kernel(const T* __restrict__ src, u32x4* __restrict__ dst, int rows, int K, int R, int half, int row_add,
                              size_t n_frag) {
  constexpr int EPL = Tr<T>::EPL, KT = Tr<T>::KT;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_frag) return;
  const int nkt = K / KT;
  const int piece = (int)(i % (4 * R));
  const size_t tile = i / (4 * R);
  const int kt = (int)(tile % nkt);
  const size_t rt = tile / nkt;
  const size_t row = rt * R + piece % R;
  u32x4 v = {0u, 0u, 0u, 0u};
  if (row < (size_t)rows) {
    const size_t srow = half > 0 ? (row / half) * 2 * half + row % half + row_add : row;
    v = *reinterpret_cast<const u32x4*>(src + srow * K + (size_t)kt * KT + (piece / R) * EPL);
  }
  dst[i] = v;
}

__global__ void accept_kernel(const int32_t* draft, const int32_t* target, int batch, int gamma, int32_t* accept_len,
                              int32_t* bonus) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= batch) return;
  int m = 0;
  while (m < gamma && draft[b * gamma + m] == target[b * (gamma + 1) + m]) ++m;
  accept_len[b] = m;
  bonus[b] = target[b * (gamma + 1) + m];
}

// user [L][Hkv][n][hd] <-> cache [L][B][Hkv][max_ctx][hd], K and V in one launch.  The slots of a (layer, KV head)
// are one contiguous run on both sides, so a workgroup moves a piece of one run: no division per element, and
// kKvPieces 16-byte loads per thread are in flight before the first store.  Bound by memory (every byte read once
// and written once): an import or export of 2048 slots of the 8B shape (268 MB each way, 537 MB of traffic).  Ordinary loads,
// non-temporal stores, two pieces a thread.  us a call with its wait on arrays not used just before, 8 pieces with both
// non-temporal and this: 136 .. 141 -> 102 .. 104 (5.2 TB/s; the kernel alone 94.5, 5.7 TB/s), 512 slots 47 -> 37, 8192 slots
// 505 -> 378, 16 slots 15 -> 14.  One import again and again on the same arrays, which the caches then serve in part: 8 pieces
// 136 (both non-temporal), 4 pieces 97 (both), 112 (neither), 79 (loads only), 74 .. 84 (stores only), 2 pieces 73 (stores
// only), 1 piece 74 .. 80.
// grid = (pieces of a run, layer x KV head, K / V).
constexpr int kKvThreads = 256, kKvPieces = 2;
__global__ __launch_bounds__(kKvThreads) void kv_copy_kernel(u32x4* kc, u32x4* vc, u32x4* k_user, u32x4* v_user, size_t layer_pitch,
                                                             size_t head_pitch, size_t seq_off, int Hkv, size_t run, int to_cache) {
  const int lh = blockIdx.y, l = lh / Hkv, h = lh % Hkv;
  u32x4* cache = (blockIdx.z ? vc : kc) + l * layer_pitch + seq_off + h * head_pitch;
  u32x4* user = (blockIdx.z ? v_user : k_user) + (size_t)lh * run;
  const u32x4* src = to_cache ? user : cache;
  u32x4* dst = to_cache ? cache : user;
  const size_t i0 = (size_t)blockIdx.x * (kKvThreads * kKvPieces) + threadIdx.x;
  u32x4 v[kKvPieces];
#pragma unroll
  for (int j = 0; j < kKvPieces; ++j) {
    const size_t i = i0 + (size_t)j * kKvThreads;
    if (i < run) v[j] = src[i];
  }
#pragma unroll
  for (int j = 0; j < kKvPieces; ++j) {
    const size_t i = i0 + (size_t)j * kKvThreads;
    if (i < run) __builtin_nontemporal_store(v[j], dst + i);
  }
}

void launch_repack(int dtype, const void* src, void* dst, int rows, int K, int R, int half, int row_add, hipStream_t st) {
  const size_t n_frag = tile_stride(rows, K, dtype, R);
  const unsigned grid = (unsigned)((n_frag + 255) / 256);
  DISPATCH_T(dtype, hipLaunchKernelGGL(repack_kernel<T>, dim3(grid), dim3(256), 0, st, (const T*)src, (u32x4*)dst, rows, K, R, half,
                                       row_add, n_frag));
}
// Streaming-read probe: the same non-temporal 16-byte loads as the weight stream, 8 in flight per
// lane, summed so that nothing is optimised away.  sink: one float per workgroup.
constexpr int kProbeBlocks = 4096, kProbeThreads = 256;
__global__ __launch_bounds__(kProbeThreads) void stream_read_kernel(const u32x4* __restrict__ p, size_t n16, float* sink) {
  // a workgroup reads 8 consecutive 4 KB pieces (32 KB contiguous) per round, as the waves of a
  // weight-streaming workgroup do
  const size_t stride = (size_t)gridDim.x * blockDim.x * 8;
  size_t i = (size_t)blockIdx.x * blockDim.x * 8 + threadIdx.x;
  uint32_t acc = 0;
  for (; i + 7 * (size_t)blockDim.x < n16; i += stride) {
    u32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = __builtin_nontemporal_load(p + i + (size_t)u * blockDim.x);
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  for (int u = 0; u < 8; ++u) {  // ragged end: the last, partial round
    const size_t j = i + (size_t)u * blockDim.x;
    if (j < n16) {
      const u32x4 v = __builtin_nontemporal_load(p + j);
      acc += v.x ^ v.y ^ v.z ^ v.w;
    }
  }
  __shared__ uint32_t sh[kProbeThreads / 64];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) sink[blockIdx.x] = (float)(sh[0] + sh[1] + sh[2] + sh[3]);
}

void launch_stream_read(const void* buf, size_t bytes, float* sink, hipStream_t st) {
  hipLaunchKernelGGL(stream_read_kernel, dim3(kProbeBlocks), dim3(kProbeThreads), 0, st, (const u32x4*)buf, bytes / 16, sink);
}
int stream_read_sink_floats() { return kProbeBlocks; }

void launch_accept(const int32_t* draft, const int32_t* target, int batch, int gamma, int32_t* accept_len, int32_t* bonus,
                   hipStream_t st) {
  hipLaunchKernelGGL(accept_kernel, dim3((batch + 63) / 64), dim3(64), 0, st, draft, target, batch, gamma, accept_len, bonus);
}

void launch_kv_copy(const Shape& s, const Buffers& b, int seq, void* k_user, void* v_user, int n_slots, int to_cache,
                    hipStream_t st) {
  const int fpr = s.hd * (s.dtype == 1 ? 2 : 4) / 16;
  const size_t run = (size_t)n_slots * fpr, head_pitch = (size_t)s.max_ctx * fpr, seq_pitch = s.Hkv * head_pitch;
  if (run == 0) return;
  constexpr size_t per_wg = kKvThreads * kKvPieces;
  // the grid's second extent is limited: whole layers at a time
  const int layers_at_once = std::max(1, 65535 / s.Hkv);
  for (int l0 = 0; l0 < s.L; l0 += layers_at_once) {
    const int nl = std::min(layers_at_once, s.L - l0);
    const size_t c0 = (size_t)l0 * s.B * seq_pitch, u0 = (size_t)l0 * s.Hkv * run;
    hipLaunchKernelGGL(kv_copy_kernel, dim3((unsigned)((run + per_wg - 1) / per_wg), nl * s.Hkv, 2), dim3(kKvThreads), 0, st,
                       (u32x4*)b.kc + c0, (u32x4*)b.vc + c0, (u32x4*)k_user + u0, (u32x4*)v_user + u0, s.B * seq_pitch, head_pitch,
                       seq * seq_pitch, s.Hkv, run, to_cache);
  }
}

}  // namespace es
