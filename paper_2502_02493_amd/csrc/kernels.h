// Internal interface between the host state machine (easyspec.cpp) and the gfx950 kernels
// (gemv.hip, attention.hip, wide.hip, resident.hip, util.hip, accept.hip).  Plain structs and launch functions; no device code in this header.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace es {

constexpr int kMaxCols = 16;  // token columns of one forward pass (= one MFMA N tile)
constexpr int kMaxChunks = 64;  // split-KV chunks per (column, head)

// Which (sequence, position, token) each column of a forward pass stands for.
struct Cols {
  int32_t n;
  int32_t seq[kMaxCols];
  int32_t pos[kMaxCols];        // slot the column writes; the highest slot it attends to
  int32_t rope_pos[kMaxCols];   // its rotary position (= pos except for the nodes of a token tree)
  // Visibility of slots 0..pos: every slot below vis_base, and slot vis_base + i iff bit i of
  // vis_mask (pos < vis_base + 64).  Causal columns: vis_base = pos + 1.
  int32_t vis_base[kMaxCols];
  unsigned long long vis_mask[kMaxCols];
  int32_t tok_idx[kMaxCols];    // index into the caller's token array
  int32_t logit_row[kMaxCols];  // row of logits_out to write, or -1
  int32_t out_idx[kMaxCols];    // index of tokens_out to write, or -1
};

// The columns of a wide pass: a calibration of more than kMaxCols columns in one pass.  Entry e is a sequence with
// columns first[e] .. first[e + 1] - 1, its tokens in order from position pos0[e] on (causal).
constexpr int kWideCols = 256;  // 16 sequences of 16 tokens
constexpr int kWideSeqs = 16;
struct Spans {
  int32_t n, n_seq;
  int32_t tok_pitch;  // the token of column i of entry e: tokens[seq[e] * tok_pitch + i - first[e]]
  int32_t first[kWideSeqs + 1];
  int32_t seq[kWideSeqs], pos0[kWideSeqs];
};

struct Shape {
  int32_t dtype;  // 0 fp32, 1 bf16
  int32_t L, d, Hq, Hkv, hd, F, V;
  int32_t HQ;     // Hq*hd
  int32_t RQKV;   // (Hq + 2 Hkv) * hd
  int32_t B, max_ctx;
  float eps;
  int32_t has_bias;
  int32_t R_ffn;  // rows per weight tile of the gate and up matrices (tile_rows(F))
  int32_t R_qkv;  // rotation pairs per tile of the QKV matrices (qkv_tile_rows); every other matrix: tiles of 16 rows
};

// Device buffers of a context.  "T" = storage dtype.  Activation arrays in T hold two parts
// [hi | lo] per slot when T is bf16 (the value is hi + lo), one part when T is fp32.  Packed matrices are arrays of 1 KB tiles
// (16 rows x 16 bytes per lane-group, see device_common.hpp) ordered [layer][row tile][k tile].
struct Buffers {
  // weights
  void *wqkv, *wo, *wg, *wu, *wd, *wlm;  // packed tiles
  void *embed;                           // plain [V][d] T
  float *bqkv;                           // [L][RQKV] or null
  float *g_attn, *g_mlp, *g_final;       // [L][d], [L][d], [d]
  float2 *rope;                          // [max_ctx][hd/2] (cos, sin)
  // cache
  void *kc, *vc;  // [L][B][Hkv][max_ctx][hd] T
  // workspaces (per forward pass).  fp32 arrays are [.][kMaxCols][width].  Arrays in T are operands of
  // the next weight contraction: per part either plain rows [column][width] (passes of one or two
  // columns) or 1 KB tiles of KT consecutive k holding [k-group][column][EPL elements], the order of
  // a wave's B fragments (see xoff() in device_common.hpp); a slot of XA / AO is PARTS * 16 * width elements.
  float *H;     // [16][d]      residual stream
  float *ssp;   // [16][d/16]   per-row-tile partial sums of squares of the vector to be normed next
  float *ssp_set;  // [MAX_SET][16][d/16]  the same per layer of a set (full-layer mode: one MLP input per layer)
  void *XA;     // [MAX_SET] x (16 x d) T   H * g_attn(layer) for the layers of the coming set (or g_final)
  void *XM;     // [MAX_SET] x (16 x d) T   H' * g_mlp(layer); one slot outside full-layer mode
  float *Q;     // [MAX_SET][16][HQ]    rotated queries
  void *AO;     // [MAX_SET] x (16 x HQ) T  attention output (rounded to T)
  float *A;     // [MAX_SET][16][d]     Attnoutput_i
  void *ACT;    // [MAX_SET] x (16 x F) T   SiLU(gate)*up; one slot outside full-layer mode
  float *PO;    // [MAX_SET*16*Hq][kMaxChunks][hd]  split-KV partial outputs
  float *PM, *PL;  // [MAX_SET*16*Hq][kMaxChunks]   partial max / sum
  float *amax_val; // [16][n_head_blocks]
  int32_t *amax_idx;
};

// Workspaces of a wide pass (bf16 models; operands in the layout of wide_off, tile_index.hpp).
struct WideBuffers {
  int32_t cols;  // columns there is room for: a multiple of 16, 0 = no wide passes
  float* H;      // [cols][d]  residual stream
  float* rs;     // [cols]     rsqrt(mean square + eps) of the residual row that the operand X was made of
  void* X;       // operand of width d: H * gain
  float* Q;      // [cols][HQ] rotated queries
  void* AO;      // operand of width HQ: attention output
  void* ACT;     // operand of width F: SiLU(gate) * up
  float* P;      // split-K partial sums [split][cols][rows]
};
constexpr int kWideSplitCols = 2048;  // columns x splits the partial sums have room for

// Resident passes of small models (resident.hip): counters, the places of a pass's tagged values, and a host word that a
// pass sets if it gave up waiting.
struct ResidentCtl {
  uint32_t ticket, pad0[31];
  uint32_t done, pad1[31];
  uint32_t epoch, pad2[31];
};
struct Resident {
  ResidentCtl* ctl;  // null: the model's passes are separate launches
  void* granules;
  uint32_t* failed;  // pinned host memory
  int32_t hasty;     // 1: passes give up at the first value that is not there yet (tests)
};
constexpr int kResMaxLayers = 64;
constexpr int kResMaxVocab = 16384;

// Per-launch timing (easyspec_profile_*): while a timer is installed for the calling thread, every kernel
// launch of the forward pass binds the next start / stop event pair to its own dispatch, so that the pair's
// elapsed time is the kernel's begin-to-end time as a kernel trace reports it (no stream markers between).
struct LaunchTimer {
  hipEvent_t* ev;   // start / stop pairs
  int8_t* op;       // kernel class of the launch that took pair i (EASYSPEC_OP_*), one entry per pair
  size_t cap, used;
  int cur_op;       // class of the launches made right now
};
extern thread_local LaunchTimer* g_launch_timer;

// How one launch of a weight-streaming kernel class (EASYSPEC_OP_QKV, _OPROJ, _GATEUP, _DOWN, _HEAD) cuts its
// packed matrices: decided in one place (stream_plan) for the launch wrappers and for stream_walk.
struct StreamPlan {
  int op;
  int n_mat;        // packed matrices a unit reads side by side: QKV 2 (first and second rotary halves), gate/up 2, else 1
  int split_array;  // 1: the n_mat matrices are separate arrays of the same tiling (gate, up); 0: one array, one after the other
  int units;        // units per layer: row tiles, or tiles of rotation pairs
  int TP;           // units per workgroup
  int R;            // rows per tile
  int K, nkt;       // contraction length, k-tiles
  int nw;           // waves per workgroup
  int NB;           // activation fragments per k-tile
  int n_layers;     // layers the grid spans
  int grid;
  size_t mat_pieces;    // 16-byte pieces of one packed matrix of one layer
  size_t layer_pieces;  // pieces from one layer to the next inside an array
};
// twin: of a launch that serves two passes
StreamPlan stream_plan(const Shape& s, int op, int ncols, int n_layers, bool full_layer, bool twin = false);
// What a host walk of the launch found: the highest piece index against the pieces the launch's layers
// hold, the highest activation element against an operand slot, k-tiles never read, read twice (apart
// from the deliberate re-reads of a missing last unit), and fragment pieces no lane takes.
struct StreamWalk {
  long long w_max, w_pieces, w_out_of_range;
  long long x_max, x_slot_elems, x_out_of_range;
  long long tiles, missed_tiles, repeated_tiles, reread_tiles, uncovered_pieces;
};
int stream_walk(const Shape& s, const StreamPlan& p, int ncols, StreamWalk* r);
// ... and of a product of a wide pass of n_cols columns: its cut, and what its workgroups load, multiply and store.
struct WideWalk {
  long long RW, CT, KS, col_blocks, row_blocks, splits, per_split, grid, kernel;
  long long w_max, w_pieces, w_out_of_range, x_max, x_pieces, x_out_of_range;
  long long products, missed, repeated, misplaced, empty_splits, out_max, out_room;
};
int wide_walk(const Shape& s, int op, int n_cols, WideWalk* r);

// Launch wrappers (all asynchronous on `st`).
// Packed matrices: row tiles of R <= 16 rows (see repack_kernel).
int tile_rows(int rows);
int qkv_tile_rows(int n_pairs);
size_t packed_bytes(int dtype, int rows, int K, int R);
// half = 0: packed row r is source row r; half > 0: source row (r / half) * 2 * half + r % half + row_add
void launch_repack(int dtype, const void* src, void* dst, int rows, int K, int R, int half, int row_add, hipStream_t st);
void launch_embed(const Shape& s, const Buffers& b, const Cols& c, const int32_t* tokens, int layer0, int n_set,
                  hipStream_t st);
// The weight kernels take an optional second pass (b2, c2: its workspaces and columns, c2->n == c.n): one launch then
// serves both passes, every wave using each weight fragment it loads for both passes' columns
// (twin_passes_fit(): whether the launch shapes of passes of n_cols columns allow it).
bool twin_passes_fit(const Shape& s, int n_cols);
// Once per context of a bf16 model, before its first launch.
hipError_t weight_kernels_prepare();
void launch_qkv(const Shape& s, const Buffers& b, const Cols& c, int layer0, int n_set, hipStream_t st,
                const Buffers* b2 = nullptr, const Cols* c2 = nullptr);
// How an attention launch over n_set layers cuts the contexts of these columns into split-KV chunks.
struct AttnCut {
  bool mfma;     // the matrix-core kernel takes the launch (groups of columns of one sequence)
  bool three;    // matrix-core kernel: probabilities in three bf16 terms (what the vector kernel would have held in fp32)
  int tiles;     // matrix-core kernel: tiles of 16 query rows per workgroup, one per wave (1, 2 or 4)
  int n_chunks;  // chunks of the longest column = grid extent; 1: every context in one piece, no merge launch
  int chunk;     // matrix-core kernel: slots per chunk (fixed length)
  int nb_ref;    // vector kernel: batches of the longest column; shorter columns get proportionally fewer chunks
};
AttnCut attn_cut(const Shape& s, const Cols& c, int n_set);
AttnCut attn_cut_vector(const Shape& s, const Cols& c, int n_set);  // the cut the vector kernel would get
// Host evaluation of the kernels' own index arithmetic for a vector-kernel cut: the chunk count of a
// column of n_slots slots and the slots [w0, w1) that wave `wave` of chunk `chunk` works through
// (empty beyond the column's chunks); attn_waves: waves per workgroup of the launch.
int attn_waves(const AttnCut& cut);
void attn_ranges(const Shape& s, const AttnCut& cut, int n_slots, int chunk, int wave, int* nch, int* w0, int* w1);
void launch_attn(const Shape& s, const Buffers& b, const Cols& c, int layer0, int n_set, const AttnCut& cut, hipStream_t st);
// O projection of the set's layers; the first layer's result goes straight into the residual.
void launch_oproj(const Shape& s, const Buffers& b, const Cols& c, int layer0, int n_set, hipStream_t st,
                  const Buffers* b2 = nullptr, const Cols* c2 = nullptr);
// Gate/up of n_layers consecutive layers, layer i on operand slot i of XM with partial sums slot i
// of ssp ([n_layers][16][d/16]) into operand slot i of ACT.  n_layers = 1 outside full-layer mode.
void launch_gateup(const Shape& s, const Buffers& b, const Cols& c, int layer, int n_layers, const float* ssp, hipStream_t st,
                   const Buffers* b2 = nullptr, const Cols* c2 = nullptr, const float* ssp2 = nullptr);
// Full-layer-parallel mode (App. B ablation), per set: the O projections (every layer parks its
// Attnoutput and writes its own MLP's input into XM / ssp_set) and the down projections (summed
// over the set's layers and added to the residual together with the Attnoutputs).
void launch_oproj_full(const Shape& s, const Buffers& b, const Cols& c, int layer0, int n_set, hipStream_t st);
void launch_down_full(const Shape& s, const Buffers& b, const Cols& c, int layer0, int n_set, const float* gain, int n_gain,
                      void* xout, hipStream_t st);
// Down projection + residual.  a_next: Attnoutput of the next layer of the same set to add, or
// -1.  The normed-input vectors for what comes next are written with gains
// gain[0..n_gain) (stride d) into xout (stride 16*d elements of T).
void launch_down(const Shape& s, const Buffers& b, const Cols& c, int layer, int a_next, const float* gain,
                 int n_gain, void* xout, hipStream_t st, const Buffers* b2 = nullptr, const Cols* c2 = nullptr,
                 void* xout2 = nullptr);
void launch_head(const Shape& s, const Buffers& b, const Cols& c, float* logits_out, int32_t* tokens_out,
                 hipStream_t st, const Buffers* b2 = nullptr, const Cols* c2 = nullptr);
// Wide passes.  The QKV, O and down products leave fp32 partial sums per split of K, which the launch after each adds in
// split order and does what follows (bias, rotary, cache write; residual, norm operand); gate/up and the head are not split
// and write activations and logits themselves.
size_t wide_operand_bytes(int cols, int K);
size_t wide_partial_bytes(const Shape& s);
void launch_wide_embed(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, const int32_t* tokens, hipStream_t st);
void launch_wide_qkv(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, hipStream_t st);
void launch_wide_attn(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, hipStream_t st);
// H += (O or down projection); operand X = H * gain, rs.  last: the last layer's down projection, which also leaves the
// rows whose tokens are asked for (the last column of every entry) as the operand of the 16-column head launch in b.
void launch_wide_proj(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, bool down, const float* gain,
                      bool last, hipStream_t st);
void launch_wide_gateup(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, int layer, hipStream_t st);
// logits of every column into logits[seq * tok_pitch + i][V], and the argmax of every entry's last column
void launch_wide_head(const Shape& s, const Buffers& b, const WideBuffers& w, const Spans& sp, float* logits, int32_t* tokens_out,
                      hipStream_t st);
// A whole pass of a small model in one launch: which models, which passes, what it needs.
bool resident_model(const Shape& s);
bool resident_pass(const Shape& s, const Cols& c, const int32_t* bounds, int n_sets);
size_t resident_granule_bytes(const Shape& s);
hipError_t resident_prepare(const Shape& s);
bool resident_hasty_model(const Shape& s);  // is there a kernel for Resident::hasty?
void launch_resident(const Shape& s, const Buffers& b, const Resident& r, const Cols& c, const int32_t* tokens, const int32_t* bounds, int n_sets,
                     float* logits, int32_t* tokens_out, hipStream_t st);
void launch_accept(const int32_t* draft, const int32_t* target, int batch, int gamma, int32_t* accept_len,
                   int32_t* bonus, hipStream_t st);
// Acceptance by speculative sampling; ws: sample_accept_workspace_bytes() of scratch.  give_up: at the first value that is not there yet.
size_t sample_accept_workspace_bytes(int batch, int gamma, int V);
void launch_sample_accept(const int32_t* draft, const float* draft_logits, const float* target_logits, const float* r,
                          const float* u, int batch, int gamma, int V, double T, double* ws, int32_t* accept_len,
                          int32_t* bonus, bool give_up, hipStream_t st);
// The library's own workspace for launch_sample_accept (a static device array, one copy per GPU): its
// address on the current device (resolved at the first call there) and its size.  Allocates nothing.
hipError_t sample_accept_static_workspace(double** out);
size_t sample_accept_static_capacity_bytes();
// Reads `bytes` (multiple of 16) of buf once; sink: stream_read_sink_floats() floats.
void launch_stream_read(const void* buf, size_t bytes, float* sink, hipStream_t st);
int stream_read_sink_floats();
void launch_kv_copy(const Shape& s, const Buffers& b, int seq, void* k_user, void* v_user, int n_slots,
                    int to_cache, hipStream_t st);

}  // namespace es
