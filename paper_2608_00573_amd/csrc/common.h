// Internal definitions shared by the HIP kernels and the host launcher of
// libtrimmoe (adaptive-depth MoE step, gfx950).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "trimmoe.h"

namespace trimmoe {

typedef uint16_t bf16_t;

// ---------------------------------------------------------------- tiling --
// tokens handled by one block of the route and permute kernels (at most; small
// batches use fewer per block: route_block_tokens)
constexpr int kRouteTokens = 32;
// route blocks the look-ahead aims for: one per CU
constexpr int kLookaheadBlocks = 256;
// route blocks a batch without look-ahead is dealt to at most (while that
// leaves kRouteTokens or fewer a block)
constexpr int kRouteBlocks = 128;
// bounds of the scan inside the bucket kernel: block histogram entries (route
// blocks x experts) and route blocks a bucket block holds in LDS
constexpr int kFusedScanEntries = 4096;
constexpr int kFusedScanBlocks = 1024;

// tokens per route block for a batch of T tokens: the power of two that gives
// about a block per CU, at most kRouteTokens.  Without look-ahead at least
// kRouteTokensMin: every block reads the router weights and the Sim table
// again, and its top-k takes kRouteTokensMin tokens (one a wavefront) at once
constexpr int kRouteTokensMin = 8;
inline int route_block_tokens(int T, bool lookahead, int E) {
  int rb = lookahead ? 1 : kRouteTokensMin;
  if (lookahead) {
    while (rb < kRouteTokens && 2 * rb * kLookaheadBlocks <= T) rb *= 2;
  } else {
    // ... and no more blocks than keep the scan in the bucket kernel
    while (rb < kRouteTokens &&
           (rb * kRouteBlocks < T || (long long)((T + rb - 1) / rb) * E > kFusedScanEntries))
      rb *= 2;
  }
  return rb;
}
// route blocks the workspace provides for batches of up to T tokens
inline int route_blocks_max(int T) {
  const int full = (T + kRouteTokens - 1) / kRouteTokens;
  const int la = T < 2 * kLookaheadBlocks ? T : 2 * kLookaheadBlocks;
  return full > la ? full : la;
}
// rows of an expert group covered by one grouped-GEMM tile: kGemmBM, or
// kBigBM for the large-group core (bf16 batches with at least
// kBigRowsPerExpert rows per expert on average)
constexpr int kGemmBM = 128;
constexpr int kBigBM = 256;
constexpr int kBigRowsPerExpert = 1024;
// the large-group down GEMM cuts the tiles of its last round into at most
// kSkPieces runs of K slices, with at most kSkSlots 256 x 256 extra partials
constexpr int kSkPieces = 8;
constexpr int kSkSlots = 256;
// the dense shared-expert GEMMs use the large-group core from this many tokens:
// below, its 256-row tiles leave most CUs idle (Qwen shapes, layer step on it
// and on the 128-row tiles: 2048 tokens 968 and 931 us, 3000 1279 and 1219, 4099
// 1571 and 1567)
constexpr int kBigDenseTokens = 4096;
// the large-group core addresses its operands with 32-bit byte offsets
inline bool big_offsets_fit(long long rows, long long cols) {
  return rows * cols * 2 < (1ll << 31);
}
inline int expert_tile_rows(bool bf16, int T, int k, int E, int d, int F) {
  const long long R = (long long)T * k;
  return bf16 && R >= (long long)kBigRowsPerExpert * E && big_offsets_fit(T, d) &&
                 big_offsets_fit(R, F)
             ? kBigBM
             : kGemmBM;
}
inline bool big_dense(bool bf16, int T, int d, int Fs) {
  return bf16 && T >= kBigDenseTokens && big_offsets_fit(T, d) && big_offsets_fit(T, Fs);
}
// the exit head uses the large-group core for wide models and large batches
// (its 256-row vocabulary tiles match kExitTileBF16)
constexpr int kBigExitTokens = 1024;
constexpr int kBigExitDModel = 2048;
inline bool big_exit(bool bf16, int T, int V, int d) {
  return bf16 && T >= kBigExitTokens && d >= kBigExitDModel && big_offsets_fit(V, d) &&
         big_offsets_fit(T, d);
}
// batches of this many tokens or more use the 256-token exit-head tile
constexpr int kWideTokens = 4096;
// ... and output heads over n_rows rows where its tiles come in no more rounds
// of the grid than they are worth: a 256 x 256 tile takes nearly twice as long as
// a 256 x 128 one, so against one round of those, or three against its two, it
// loses (argmax kernel in 256 x 128 tiles and on the large-group core, d = 2048,
// us: V = 4000, 1500 rows, 192 tiles against 96: 35 and 62; V = 6000, 1500 rows, 288
// against 144: 66 and 61; 3000 rows, 576 against 288: 102 and 121; V = 16000, 2048
// rows, 1008 against 504: 146 and 116).  From kWideTokens rows the other tile is
// 256 x 256 too, and better at short K and few vocabulary tiles (d = 2048, 6000
// rows: V = 6000 176 and 186, V = 8000 190 and 180; d = 4096, V = 6000: 317 and 299)
inline bool big_argmax(int n_rows, int V, int d, int n_cu) {
  if (!big_exit(true, n_rows, V, d)) return false;
  const int vt = (V + kBigBM - 1) / kBigBM;
  if (n_rows >= kWideTokens) return d >= 2 * kBigExitDModel || vt >= 32;
  const int tiles = vt * ((n_rows + 127) / 128), big_tiles = vt * ((n_rows + 255) / 256);
  return tiles > 3 * n_cu || (tiles > n_cu && big_tiles <= n_cu);
}
constexpr int kGemmBN = 128;
constexpr int kGemmBK = 64;
// K splits of the routed down GEMM (128-row tiles), from the live tile and row
// counts: the row tiles of an uneven batch are fewer than the bound the host
// knows (one per expert more than the rows need), and too few tiles leave CUs
// idle.  The fewest K slices on the busiest of n_cu CUs, 1, 2, 4 or 8 splits
// of at least 8 slices whose partial rows the workspace holds; a split has to
// save an eighth (its partials are written, and read by the combine, once
// more).  The GEMM and the combine evaluate the same rule.  Mixtral shapes, 333
// tokens (7 row tiles where the bound is 14): down 225 -> 140 us.
__host__ __device__ inline int live_down_splits(int n_mt, int rows, int N, int K, long long cap_rows,
                                                int n_cu) {
  const int tiles = n_mt * ((N + 255) / 256), nk = K / kGemmBK;
  int best = 1;
  long long best_cost = (long long)((tiles + n_cu - 1) / n_cu) * nk;
  for (int s = 2; s <= 8; s *= 2) {
    if (nk % s != 0 || nk / s < 8 || (long long)rows * s > cap_rows) break;
    const long long cost = (long long)((tiles * s + n_cu - 1) / n_cu) * (nk / s);
    if (8 * cost <= 7 * best_cost) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}
// bf16 batches of up to this many tokens run the weight-streaming kernels
// (skinny.hip) for every GEMM
constexpr int kSkinnyTokens = 64;
// ... and the shared expert, one pass over its weights (which then stay in the
// last-level cache) per kSkinnyTokens executed tokens, up to this many: two
// passes (Qwen shapes, layer step: 65 tokens 376 -> 317 us, 150 tokens of which
// 85 execute 389 -> 340; a third pass costs more than the 128-row tiles)
constexpr int kSkinnyDenseTokens = 128;
// vocabulary rows per exit partial (bf16 MFMA tiles / fp32 path).  The
// weight-streaming exit head writes one partial per block; its workspace is
// sized for blocks of at least kExitTileBF16Small rows
constexpr int kExitTileBF16 = 256;
constexpr int kExitTileBF16Small = 128;
constexpr int kExitTileF32 = 16;
constexpr int kExitTileF32Mma = 128;

// fp32 rows of K floats that are whole 128-byte K slices run in fp32 MFMAs
inline bool f32_slices(int K) { return K % 32 == 0; }
// ... and so do the operands of a head_argmax call, which asks no alignment
inline bool f32_mma(const void* W, const void* H, int K) {
  return f32_slices(K) &&
         ((reinterpret_cast<uintptr_t>(W) | reinterpret_cast<uintptr_t>(H)) & 15) == 0;
}

// Operand order of the activations those kernels read: a tile of n <= 16 rows
// is kept as [k-step of 32][4 groups of 8][n rows][8 elements], so that the
// operand of a k-step is one contiguous run; element offset of (k-step, group,
// row) within the tile
__host__ __device__ inline int frag_order(int kstep, int group, int row, int n) {
  return ((kstep * 4 + group) * n + row) * 8;
}

inline int exit_tile_rows(bool bf16, int T) {
  return bf16 ? (T <= kSkinnyTokens ? kExitTileBF16Small : kExitTileBF16) : kExitTileF32;
}
// bf16 exit heads of up to kSkinnyTokens tokens that stream W (skinny.hip); the
// others run 128 x 32 tiles (gemm.hip).  A wavefront of the streaming kernel
// takes a quarter of K and every 16 rows of W end in a sum through LDS, so it
// pays where rows are long; a block of it takes 128 rows of W or more, so
// beyond 16 tokens it needs enough of them for three quarters of the CUs (below,
// the tile's chain of K slices is shorter).  Kernel times on an MI355X, tiles and
// streaming, W not in the cache (us): d = 768, V = 32000: 12.0 and 13.5 at 16
// tokens, 16.8 and 20.0 at 64; d = 2048, V = 16000: 20.8 and 19.7 at 16, 22.8 and
// 29.2 at 64; V = 32000: 32.6 and 24.9, 42.6 and 33.8; d = 4096, V = 4000: 32.8
// and 29.8, 32.6 and 44.7; V = 32000: 59.6 and 42.5, 75.2 and 53.7.  Heads past the
// last-level cache stream with shorter rows too (d = 1024, V = 150000: 55.0 and
// 50.1, 90.2 and 84.9), but not at 17 to 32 tokens, one column of tiles (55.8 and
// 68.8); there an argmax, which gathers a caller's rows, never does (d = 2048,
// V = 32000: 33.8 and 35.5).  A head of one group of 16 rows is one short unit
// (sigmoid, d = 768, 16 tokens: 9.3 and 6.1).
constexpr int kStreamExitDModel = 2048;
constexpr int kStreamExitVocab = 24576;
inline bool exit_streams(bool bf16, bool argmax, int T, int V, int d) {
  if (!bf16 || T > kSkinnyTokens) return false;
  const bool wide = d >= kStreamExitDModel, huge = (long long)V * d >= 1ll << 27;
  if (T <= 16) return V <= 16 || wide || huge;
  if (V <= 16) return T <= 32 || wide;
  if (T <= 32) return !argmax && wide && V >= kStreamExitVocab;
  return (wide && V >= kStreamExitVocab) || huge;
}
// exit partials per token of a launch on n_cu compute units (never more than
// the exit_tile_rows tiles the workspace is sized for); mma_f32: an fp32 head
// in fp32 MFMAs; streams: one partial per block (exit_streams)
inline int exit_vtiles(bool bf16, bool mma_f32, bool streams, int T, int V, int n_cu) {
  const int rows = !bf16 && mma_f32 ? kExitTileF32Mma : exit_tile_rows(bf16, T);
  const int n = (V + rows - 1) / rows;
  return streams && n > n_cu ? n_cu : n;
}
// fp32 GEMM tile
constexpr int kF32Tile = 16;
// exit-head training: the one-pass descent step takes heads of up to
// kTrainMaxCols columns and at most kTrainBlocks blocks of partial sums
constexpr int kTrainMaxCols = 4096;
constexpr int kTrainBlocks = 256;
// per-layer trace counters (row stride of trimmoe_trace.counters)
constexpr int kCounters = 16;
// look-ahead: later layers a decision looks at, and first-level branches
// (candidate action, next-layer target tuple) per token
constexpr int kMaxLookahead = TRIMMOE_MAX_HORIZON - 1;
constexpr int kMaxBranches = 1024;

// slots of the small device counter block in the workspace
enum CountSlot {
  kCntRows = 0,   // merged (token, expert) rows of this layer
  kCntTiles = 1,  // grouped-GEMM row tiles
  kCntExec = 2,   // executed tokens
  kCntSlots = 8
};

// --------------------------------------------------------------- numbers --
__device__ __forceinline__ float bf2f(bf16_t v) {
  return __uint_as_float(static_cast<uint32_t>(v) << 16);
}

// fp32 -> bf16, round to nearest, ties to even (NaN stays NaN)
__device__ __forceinline__ bf16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<bf16_t>((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<bf16_t>(u >> 16);
}

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) { return bf2f(v); }

template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return f2bf(v); }

// --------------------------------------------------- per-layer arguments --
// Everything one layer's kernels need, passed by value.
struct LayerParams {
  // model
  int N, d, E, k, F, Fs, V, act, conf_mode, normalize, layer;
  // layer tensors
  const void* w_router;
  const float* b_router;
  const void* w_up;
  const void* w_gate;
  const void* w_down;
  const void* ws_up;
  const void* ws_gate;
  const void* ws_down;
  const void* w_exit;
  const float* b_exit;
  const uint8_t* local_mask;
  const float* sim;
  float theta, skip_slope;
  // policy
  float p_exit, budget, omega_t, t_local, t_remote, phi_scale, sim_min;
  const float* p_exit_tok;
  const float* budget_tok;
  // look-ahead (Eq. (39)): la_*[j - 1] describe layer + j for j = 1 ..
  // horizon - 1; la_tto/la_tp[j] the transitions from layer + j to the next
  int horizon;  // effective horizon: min(policy horizon, N - layer)
  int la_subs;  // look-ahead: local substitute candidates per remote slot (1 at H = 1)
  int trans_b;
  int rb;       // tokens per route block (route, scan and bucket agree on it)
  int bm;       // rows per expert tile of the grouped GEMMs (kGemmBM or kBigBM)
  const uint8_t* la_mask[kMaxLookahead];
  const float* la_sim[kMaxLookahead];
  float la_theta[kMaxLookahead], la_slope[kMaxLookahead];
  const int16_t* la_tto[kMaxLookahead];
  const float* la_tp[kMaxLookahead];
  // state
  int T;
  void* h;
  float* d_acc;
  int32_t* active_idx;
  int32_t* n_active;
  int32_t* exit_layer;
  float* xi;
  // trace (already offset to this layer's rows; all NULL when no trace)
  int8_t* tr_action;
  int16_t* tr_target;
  int16_t* tr_exec;
  int8_t* tr_kind;
  float* tr_gate;
  float* tr_importance;
  float* tr_xi;
  float* tr_d_acc;
  int32_t* tr_counters;
  // workspace
  int32_t* tok_exec;   // [T*k] merged rows per active position, -1 padded
  float* tok_w;        // [T*k]
  int32_t* tok_row;    // [T*k] permuted row of each merged row
  int32_t* tok_action; // [T]   ACT_EXEC / ACT_SKIP per active position
  int32_t* tok_keep;   // [T]   1 = still active after this layer
  int32_t* exec_list;  // [T]   token id of each executed token (active order)
  int32_t* exec_pos;   // [T]   active position of each executed token
  int32_t* blk_cnt;    // [nblk*E]
  int32_t* blk_off;    // [nblk*E]
  int32_t* blk_xcnt;   // [nblk]
  int32_t* blk_xoff;   // [nblk]
  int32_t* exp_off;    // [E+1]
  int32_t* counts;     // [kCntSlots]
  int4* tiles;         // [max_tiles] (expert, row begin, row end, 0)
  int32_t* exp_toff;   // [E]   first tile of each expert in `tiles`
  int32_t* sk_flag;    // [max_tiles * cdiv(d, 256)] large-group down GEMM: per tile,
                       // 0 (whole) or (first compact partial << 4 | pieces) when
                       // its K slices were cut; NULL when the layer's down GEMM
                       // is not on that core
  float* sk_part;      // [kSkSlots][256][256] compact partials of later pieces
  int32_t* row_src;    // [T*k] token whose h row feeds each permuted row
  void* act_buf;       // [T*k, F]
  float* y_buf;        // [splits][rows, d] partial down-projection slices
  long long y_cap_rows;  // rows y_buf holds when the down GEMM splits K
                         // (live_down_splits), or 0: one slice
  void* act_s;         // [T, Fs]
  float* y_s;          // [T, d]
  void* hx;            // [T, d]    updated rows of executed tokens (exit input;
                       // in operand order for the weight-streaming exit head)
  float2* partials;    // [T, n_vtiles] (max, sum exp) per vocabulary tile
  int n_vtiles;
  bool exit_stream;    // the exit head streams W (exit_streams)
  int max_tiles;
  int n_cu;            // compute units of the device (persistent grids)
  // engine-clock record (measurement): [class][2] sums of core cycles and
  // 100 MHz ticks per GEMM block, or NULL
  unsigned long long* clk;
};

// observations of one stack pass for the runtime feedback rules
struct WindowArgs {
  int T, N, k;
  const int32_t* exit_layer;  // [T]
  const float* xi;            // [T]
  const float* d_acc;         // [T]
  const float* budget_tok;    // [T] or NULL
  float budget, t_local, t_remote;
  const int32_t* counters;    // trace counters [N, kCounters]
  double* stats;              // [6], accumulated
};

// launchers (decide.hip)
hipError_t launch_state_reset(const trimmoe_model* m, const trimmoe_state* s,
                              hipStream_t st);
// inactive defaults of the trace rows of n_layers consecutive layers, from
// the layer p's trace pointers point at
hipError_t launch_trace_fill(const LayerParams& p, int n_layers, hipStream_t st);
hipError_t launch_route(const LayerParams& p, bool bf16, hipStream_t st);
hipError_t launch_scan(const LayerParams& p, hipStream_t st);
hipError_t launch_bucket(const LayerParams& p, hipStream_t st);
hipError_t launch_combine(const LayerParams& p, bool bf16, hipStream_t st);
hipError_t launch_exit_reduce(const LayerParams& p, hipStream_t st);
hipError_t launch_compact(const LayerParams& p, hipStream_t st);
// exit-head training (Sec. IV-A): per-tile (max logit, row) partials of an
// output head over rows of hidden states (head.hip reduces them to argmax)
hipError_t launch_head_argmax_partials(bool bf16, const void* W, const float* bias, const void* H,
                                       const int* n_rows_dev, int n_rows, int V, int K,
                                       int n_vtiles, float2* partials, int n_cu, hipStream_t st);
hipError_t launch_argmax_reduce(const float2* partials, int n_vtiles, int n_rows, int32_t* out,
                                hipStream_t st);
hipError_t launch_consistency(const int32_t* pred, const int32_t* ref, int n_rows,
                              uint8_t* labels, hipStream_t st);
// *p = v on the stream (a kernel, so that the call can be captured)
hipError_t launch_set_int(int32_t* p, int v, hipStream_t st);
// one full-batch descent step of the sigmoid exit head on BCE (Eq. (23)):
// residuals r = sigmoid(w . h + c) - y and per-row losses, then the update
hipError_t launch_bce_step(bool bf16, const void* H, const uint8_t* y, int n_rows, int d,
                           float lr, float* w, float* c, float* r, double* row_loss,
                           float* loss_out, hipStream_t st);
// the same step with the rows read once (d <= kTrainMaxCols): part holds nb
// rows of bce_slots partial column sums (the columns padded to what the
// kernel's lanes cover), part_rl nb partial (residual, loss) sums
int bce_slots(bool bf16, const void* H, int d, int* vec);
hipError_t launch_bce_rows_step(bool bf16, const void* H, const uint8_t* y, int n_rows, int d,
                                float lr, float* w, float* c, double* part, double2* part_rl,
                                int nb, float* loss_out, hipStream_t st);
hipError_t launch_window_stats(const WindowArgs& w, hipStream_t st);

// launchers (gemm.hip)
hipError_t launch_expert_up(const LayerParams& p, bool bf16, hipStream_t st);
hipError_t launch_expert_down(const LayerParams& p, bool bf16, hipStream_t st);
hipError_t launch_shared_expert(const LayerParams& p, bool bf16, hipStream_t st);
hipError_t launch_exit_head(const LayerParams& p, bool bf16, hipStream_t st);
int down_splits(int max_tiles, int N, int K);
// dynamic LDS of a route block (logits, and the look-ahead tables at H > 1)
size_t route_lds_bytes(bool bf16, int E, int d, int horizon, int trans_b, int k, int la_subs);
// dynamic LDS a route block may take next to its static arrays (about 10 KB;
// gfx950: 160 KB per workgroup)
constexpr size_t kRouteLdsMax = 148 * 1024;

}  // namespace trimmoe
