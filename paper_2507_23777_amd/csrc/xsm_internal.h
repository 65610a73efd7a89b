// Host-side internals of libxsm: context, buffer layouts, kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "../../include/xsm.h"

namespace xsm {

constexpr int kPrefillChunk = 16;   // prefix rows per sequence per backbone pass (general kernels)
constexpr int kFastPassRows = 8192; // rows of one backbone pass the MFMA path's workspace always holds (prefill chunks)
constexpr int kMaxRows = 16;        // rows per sequence per pass (K+1 <= 16)

// Element offsets of the canonical weight tensors (same order as the weight file).
struct LayerOff {
  size_t g1, Wqkv, Wo, gc, Wcq, Wckv, Wco, g2, W1, W2;
};
struct WeightOff {
  size_t E, gf, WU, total;
  std::vector<LayerOff> layer;
  std::vector<size_t> hW, hb;                 // MLP heads
  std::vector<size_t> hq, hkv, ho, hU;        // cross-attention heads
};

// Byte offsets inside the caller's workspace buffer.
struct WorkOff {
  size_t X, Xn, QKV, Qr, AO, U, Z0, G, Hh, Rk, Zh;
  size_t eff_len, slot, acc, y0, wflags, rowidx, arrived, eff2, slot2;   // int32 arrays
  size_t part, tickets, gpart, gtickets;                                  // split-key attention partials
  size_t ll, ctrl, head_all, tlog;                       // single-launch step: exchange buffers
  size_t lctrl, lssq;                                    // persistent layers kernel: queues and partition, square sums
  size_t gpart_floats;                                   // size of gpart
  size_t total;
};

// Byte offsets of the fragment-ordered (tiled) bf16 matrices inside the weights buffer.
struct TiledLayer { size_t Wqkv, Wo, Wcq, Wckv, Wco, W1, W2; };
struct TiledOff {
  std::vector<TiledLayer> layer;
  size_t WU, Wh, hb;       // unembedding, stacked head matrices [K*d][d] (MLP: W_k, CA: Wq_k), stacked head biases [K][d]
  std::vector<size_t> Who, WhU, Whkv;   // cross-attention heads: output projections, unembeddings, key/value projections
  bool wu_ok;              // vocabulary is a multiple of 16
};

// Output of a residual-add projection that is still in split-contraction partial blocks
// [N/64][kspl][M][64]; the next RMSNorm pass over Y (or flush_pending_add) adds it in.
struct PendingAdd {
  bool active = false;
  const float* part = nullptr;
  int kspl = 0, M = 0, N = 0;
  float* Y = nullptr;
  int ldy = 0;
};
void flush_pending_add(PendingAdd* p, hipStream_t s);

// Per-layer pointers of the persistent layers kernel and of the single-launch step (uploaded to the
// device at load time).
struct LayerWts {
  const uint4 *Wqkv, *Wo, *Wcq, *Wco, *W1, *W2;       // fragment-ordered weights
  const uint16_t *gc, *g2, *g_next;                   // gains; g_next: the following layer's first norm (the last layer's: the final norm)
  uint16_t *Kc, *Vt;                                  // key and value cache (fragment order)
  const uint16_t *Kx, *Vx;                            // cross-attention keys / values
};
struct LayerTab {
  const uint4 *Wqkv, *Wo, *W1, *W2;     // fragment-ordered weights
  const uint16_t *g1, *g2;              // RMSNorm gains (bf16)
  uint16_t *Kc, *Vt;                    // this layer's key and value cache (fragment order)
};

}  // namespace xsm

struct xsm_ctx {
  xsm_config cfg;
  xsm::WeightOff woff;
  xsm::WorkOff ws;
  size_t esz;              // bytes per storage element
  size_t w_canon_bytes;    // canonical weights
  size_t rope_off;         // byte offset of the rotary table in the weights buffer
  size_t weights_bytes, kv_bytes;
  size_t kv_self_elems;    // elements of the self-attention cache (cross cache follows)
  size_t kv_cross_elems;   // elements of the layers' cross cache (the heads' condition cache follows)
  bool fast = false;       // bf16 MFMA path (head_dim 64, cache in fragment order)
  bool small_ok = false;   // single-launch step available for this model shape
  bool use_small = true;   // xsm_set_option(XSM_OPT_SINGLE_LAUNCH)
  bool small_dev = false;  // the bound device can hold the single launch's 256 workgroups at once
  bool small_failed = false;   // xsm_check_device found a timed-out wait: per-stage kernels until weights are loaded again
  bool gemm_unmatched = false; // a projection found no kernel for its (prologue, epilogue) pair: the step reports it
  bool layers_failed = false;  // xsm_check_device found a timed-out wait of it: per-stage kernels until weights are loaded again
  bool tile_ok = false;    // row- and column-blocked projections of large passes available for this model shape
  bool layers_ok = false;  // persistent layers kernel available for this model shape
  size_t layer_wts_off = 0;              // byte offset of the LayerWts array in the weights buffer
  size_t layers_err_off = 0;             // and of the layers kernel's error word (it outlives the workspace's contents)
  std::vector<xsm::LayerWts> layer_wts;  // host copy (source of the upload)
  bool timeline = false;   // xsm_set_option(XSM_OPT_TIMELINE)
  int force_splits = 0;    // xsm_set_option(XSM_OPT_ATTN_SPLITS): key-range slices per (sequence, head), 0 = automatic
  int prefill_rows = 0;              // XSM_OPT_PREFILL_ROWS: rows per prefill pass, 0 = what the workspace holds
  size_t layer_tab_off = 0;              // byte offset of the LayerTab array in the weights buffer
  std::vector<xsm::LayerTab> layer_tab;  // host copy (source of the upload)
  xsm::TiledOff toff;
  int cap_self = 0, cap_cross = 0;   // cache capacities in positions, padded to 64
  xsm::PendingAdd pend;              // see PendingAdd
  size_t part_entries = 0;           // (sequence, head, query tile, split) partial slots in the workspace
  size_t rows_max = 0;               // rows of one backbone pass the workspace holds
  // layout of the static scratch array (decoding steps only) for xsm_spec_step_static
  xsm::WorkOff ws_static;
  size_t part_entries_static = 0, rows_max_static = 0, n_tickets_static = 0;
  int dev = -1;                      // device the buffers were bound on
  char* d_static = nullptr;          // that device's address of the static scratch array
  char* d_w = nullptr;
  char* d_kv = nullptr;
  char* d_ws = nullptr;
  bool loaded = false;
  std::string err;
};

namespace xsm {

// Optional per-kernel timing with HIP events on the launch stream (off by default; used by
// the benchmark to attribute step time to kernels).  A scope brackets one launch.
// A kernel's dynamic-LDS limit above 64 KB is a property of (kernel, device): raised once for
// each pair, and again if a later launch of the kernel needs more.
inline void allow_dynamic_lds(const void* kfn, size_t bytes) {
  if (bytes <= 64 * 1024) return;
  static std::mutex mu;
  static std::map<std::pair<const void*, int>, size_t> granted;
  int dev = 0;
  (void)hipGetDevice(&dev);
  std::lock_guard<std::mutex> lock(mu);
  size_t& have = granted[{kfn, dev}];
  if (bytes > have) {
    (void)hipFuncSetAttribute(kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    have = bytes;
  }
}

struct TraceScope {
  TraceScope(const char* name, hipStream_t s);
  ~TraceScope();
  hipStream_t s_;
  int idx_;
};

// ---- launchers (xsm_kernels_basic.hip) -------------------------------------
// dtype: XSM_F32 or XSM_BF16 selects the storage type of weights / cache / embeddings.
void launch_rope_table(float2* tab, int max_ctx, int head_dim, float theta, hipStream_t s);

// Validate one step's inputs: eff_len[b] = kv_len[b] or -1 (sequence skipped), slot copy,
// flag bits.
void launch_prepare(const int32_t* kv_len, const int32_t* slot, const int32_t* block, int n_seq,
                    int R, int vocab, int max_batch, int max_ctx, int kv_len_bound,
                    const uint32_t* err, int32_t* eff_len, int32_t* slot_out, uint32_t* wflags, uint32_t* arrived, hipStream_t s);
void launch_fill_i32(int32_t* p, int n, int32_t v, hipStream_t s);

void launch_embed(int dtype, const void* E, const int32_t* block, const int32_t* eff_len, float* X,
                  int n_seq, int R, int d, hipStream_t s);
// X[b*C + j] = emb[b][row0 + j] for j < C
// bf16 rows -> one fragment-ordered operand plane [n_seq*C][d] (d % 32 == 0)
void launch_load_rows_plane(const void* emb, void* plane, int n_seq, int C, int row0, int rows_per_seq, int d,
                            hipStream_t s);
void launch_load_rows(int dtype, const void* emb, float* X, int n_seq, int C, int row0,
                      int rows_per_seq, int d, hipStream_t s);
void launch_rmsnorm(int dtype, const float* X, const void* gain, float* Y, int M, int d, float eps,
                    hipStream_t s);
enum { EPI_STORE = 0, EPI_ADD = 1, EPI_GELU = 2 };
// Y[m][n] (op)= sum_k A[m][k] * W[n][k]
void launch_gemm(int dtype, int epi, const float* A, int lda, const void* W, float* Y, int ldy,
                 int M, int N, int K, hipStream_t s);
// rotate q,k of QKV[M][3d], write q to Qr[M][d], k/v into the cache at eff_len[b] + j
void launch_rope_kv(int dtype, const float* QKV, const float2* rope, const int32_t* eff_len,
                    const int32_t* slot, float* Qr, void* Kc, void* Vc, int n_seq, int R, int H,
                    int hd, int max_ctx, hipStream_t s);
// cond K/V rows of one chunk into the cross cache: KV[M][2d] -> caches at rows row0..row0+C-1
void launch_store_cond(int dtype, const float* KV, const int32_t* slot, void* Kc, void* Vc,
                       int n_seq, int C, int row0, int H, int hd, int cap, int frag_order,
                       hipStream_t s);
// attention of row m = b*R + j over cache positions < (fixed_limit > 0 ? fixed_limit
// : eff_len[b] + j + 1)
void launch_attention(int dtype, const float* Q, const void* Kc, const void* Vc,
                      const int32_t* eff_len, const int32_t* slot, float* O, int n_seq, int R,
                      int H, int hd, int cap, int fixed_limit, hipStream_t s);

// ---- MFMA path (xsm_gemm_mfma.hip, xsm_attn_mfma.hip) ----------------------------
enum { PRO_NORM = 0, PRO_F32 = 1, PRO_PLANES = 2 };   // PRO_PLANES: X holds fragment-ordered bf16 hi/lo planes (M > 256 only)
enum { FEPI_STORE = 0, FEPI_ADD = 1, FEPI_GELU = 2, FEPI_QKV = 3, FEPI_HEAD = 4 };
struct FastGemm {
  const uint4* Wt;             // fragment-ordered weights [N/16][K/32][64 lanes][8]
  int N, K, M, KC;
  const float* X; int ldx;     // fp32 input rows (PRO_PLANES: the planes, ldx unused)
  int x_single;                // PRO_PLANES: the input is exact in bf16, only the hi plane exists (FEPI_STORE only)
  const uint16_t* gain;        // bf16 RMSNorm gain [K] (PRO_NORM)
  float eps;
  const int32_t* row_index;    // optional gather: input row of output row m
  float* Y; int ldy;           // fp32 output (for FEPI_QKV: the rotated queries [M][d])
  int y_planes;                // FEPI_GELU in the row-blocked kernel: write Y as operand planes [M][N] instead
  const uint16_t* bias;        // FEPI_HEAD: stacked biases [N]
  float* nscratch;             // [M][K] fp32: normalised rows for the kernels that do not fuse the norm
  int ksplit;                  // row-blocked kernel, FEPI_ADD: slices of the contraction index (set by the launcher)
  float* ws_part; uint32_t* ws_tickets;   // split-contraction partial products and arrival counters
  PendingAdd* pend;            // host-side: where a residual-add projection may leave its sum pending
  // FEPI_QKV
  const float2* rope; const int32_t* eff_len; const int32_t* slot;
  int R, H, hd, cap;
  uint16_t* Kc; uint16_t* Vc;
};
bool fgemm_supported(int N, int K);
// true when a projection of these sizes can take its input as operand planes (PRO_PLANES)
bool fgemm_planes_ok(int M, int N, int K);
// slices of the contraction index the row-blocked kernel takes for a residual-add projection
// from operand planes (1 = whole contraction per workgroup), and the partial-product floats
// such projections need for up to Mmax rows
int blk_add_split(int M, int N, int K);
size_t blk_add_part_floats(int Mmax, int N, int K);
constexpr size_t kWsTickets = 4096;      // arrival counters of the split-contraction GEMM
bool ws_gemm_shape_ok(int M, int N, int K);
size_t ws_gemm_part_floats(int M, int N, int K);
// false: no kernel takes this (prologue, epilogue) pair at this shape; nothing was enqueued
bool launch_fgemm(int pro, int epi, const FastGemm& g, hipStream_t s);
void launch_tile_weights(const void* W, void* out, int N, int K, int rope_d, int rope_hd, hipStream_t s);
void launch_copy_u16(const void* src, void* dst, int n, hipStream_t s);

struct FastAttn {
  const float* Q; int ldq;            // fp32 rotated queries [M][d]
  const uint16_t* Kc;                 // layer's keys and values [slot][H][cap * 64], fragment order
  const uint16_t* Vt;
  const int32_t* eff_len; const int32_t* slot;
  float* O; int ldo;                  // fp32 output [M][d]
  int o_planes, o_rows;               // o_planes: write O as operand planes [o_rows][ldo] instead (o_rows = M)
  float* part; uint32_t* tickets;     // split-key partials and arrival counters
  int R, H, cap, S, fixed_limit;
  float scale_log2;                   // log2(e) / sqrt(head_dim)
};
void launch_fattn(const FastAttn& a, int n_seq, hipStream_t s);
size_t fattn_part_bytes(size_t entries);
void launch_head_ca_prep(const float* G, float* Rk, const int32_t* eff, const int32_t* slot, int32_t* eff2,
                         int32_t* slot2, int n_seq, int K, int d, int max_batch, hipStream_t s);
// out[m][:] = RMSNorm(X[row_index ? row_index[m] : m][:]) * gain (fp32 in and out, bf16 gain)
void launch_norm_rows(const float* X, int ldx, const int32_t* row_index, const uint16_t* gain, float eps, float* out,
                      int M, int K, hipStream_t s);

// ---- all layers of a pass in one persistent kernel (xsm_layers.hip) ------------------
constexpr int kLayersMaxRows = 1280;    // rows of a pass it takes (17 ..)
enum { kStQkv = 0, kStAtt, kStO, kStCq, kStCatt, kStCo, kStUp, kStDown };
constexpr int kMaxLayerStages = 8;
struct LayerStage { int kind, NT, MT, KS, NG, MG, MC, base, count, adds_before; };   // base: first task number inside a layer
struct LayersBegin {
  const uint16_t* E; const int32_t* block; const int32_t* kv_len; const int32_t* slot;   // decoding: tokens and sequences
  const uint16_t* rows; int rows_per_seq, row0;                                          // prefill: bf16 rows [n_seq][rows_per_seq][d]
  const uint16_t* gain;                 // first norm
  int n_seq, R, d, H, vocab, max_batch, max_ctx, bound;
  int32_t* eff_len; int32_t* slot_out; uint32_t* wflags;
  const uint32_t* err;                  // not 0: an earlier pass of the layers kernel gave up, every sequence is skipped (may be null)
  uint32_t* arrived;                    // decoding: counters of the step's tail, one per sequence, cleared
  int partition;                        // 1: also attention's shares and cleared queues (xsm_layers.hip)
  float* x; void* planes; float* ssq; uint32_t* ctrl; int32_t* unit_pre;                 // (set by launch_layers)
};
struct LayersArgs {
  const LayerWts* wts; int L;
  int kv_only;                          // the cache is all that is wanted: the last layer ends with its QKV stage
  float* x[2]; void* P[2]; float* ssq[2];   // residual tiles, operand planes, square sums: each stage that adds writes the other one
  float* q; void* AO; void* U; float* part; uint32_t* tickets; float* gpart; uint32_t* gtickets;
  float* x_out;                         // final residual rows [M][d]
  const int32_t* eff_len; int32_t* eff_len_w; const int32_t* slot; uint32_t* wflags; uint32_t* err;
  uint32_t* err_small;                  // the single-launch step's error word (may be null)
  const float2* rope; uint32_t* ctrl; const int32_t* unit_pre;
  float eps, scale_log2;
  int cap, cap_cross, n_cond;
  // set by launch_layers
  int M, mtiles, n_seq, R, n_stages, per_layer, adds;
  LayerStage stage[kMaxLayerStages];
};
bool layers_supported(int D, int F, int L);
bool layers_usable(int n_seq, int R);
size_t layers_ctrl_bytes();
size_t layers_part_bytes();
void launch_layers(LayersBegin b, LayersArgs a, int D, hipStream_t s);
void launch_layers_begin(const LayersBegin& b, hipStream_t s);

// ---- projections of large passes (xsm_gemm_tile.hip) ------------------------------------
enum { kTileQkv = 0, kTileStore, kTileGelu, kTileAdd };
struct TileGemm {
  const uint4* W;              // fragment-ordered weights [N/16][K/32][64]
  const void* A;               // bf16 hi / lo operand planes [M][K]
  int M, N, K, kind;
  const float* ssq_in; float eps;        // square sums [M][K/16] of the rows the planes come from: scale by 1 / rms (nullptr: don't)
  float* Y;                    // kTileQkv: rotated queries [M][K]; kTileStore: rows [M][N]; kTileGelu: operand planes [M][N]
  // kTileAdd: residual in tile order (updated), planes of (residual x gain), their square sums; x_out: fp32 rows instead
  float* x; float* x_out; const uint16_t* gain; void* P; float* ssq_out;
  // kTileQkv
  const float2* rope; const int32_t* eff_len; const int32_t* slot; uint16_t* Kc; uint16_t* Vc;
  int R, H, cap;
  // slices of the contraction (set by the launcher)
  int KS; float* part; uint32_t* tickets;
};
bool tile_supported(int d, int F, int H);
void launch_gemm_tile(TileGemm g, size_t part_floats, hipStream_t s);

// ---- single-launch step for <= 16 block rows (xsm_step_small.hip) -------------------
struct SmallArgs {
  const LayerTab* layers; int L;
  const uint16_t* E; const uint16_t* gf; const uint16_t* hb;
  const uint4* WU; const uint4* Wh;
  const float2* rope;
  uint32_t* ll; size_t ll_layer_stride;  // tagged-word exchange buffers (4-byte words), words per layer
  size_t ll_words;                       // words of the whole exchange region
  uint32_t* ctrl;                        // [0] step epoch, [1] error word, [64..319] the workgroups' barrier words
  const int32_t* slot; int32_t* kv_len; int32_t* block; int32_t* out_tokens; int32_t* n_accepted;
  uint32_t* flags;
  float* logits_dbg; float* head_logits_dbg; float* head_all_dbg; int32_t* acc_out;
  uint64_t* tlog;                        // optional stage timeline [256][L*16 + 8] clock stamps
  int n_seq, R, S, V, max_batch, max_ctx, bound, cap;   // S: key slices per (sequence, head), or their upper limit
  int s_auto;                            // 1: the kernel picks the slice count <= S from the cache lengths it reads
  int full_verify;                       // 0: greedy verification with argmax draws from the per-tile top-2 statistics;
                                         // 1: the last stage reads the full logits rows (logits_dbg / head_all_dbg must
                                         // be set) and applies the criterion and sampling rule of vp
  xsm_verify_params vp;
  float eps, scale_log2;
};
constexpr int kSmallMaxRows = 144;     // backbone rows + head rows (M + M K) of one single-launch step
bool small_supported(int D, int F);
size_t small_ll_words(int n_layers, int D, int F, int K);     // 4-byte words
size_t small_ll_layer_stride(int D, int F);
constexpr size_t kSmallCtrlBytes = 2048;
void launch_step_small(const SmallArgs& a, int D, int F, hipStream_t s);
void launch_fill_u64(uint64_t* p, size_t n, uint64_t v, hipStream_t s);
// head_logits_dbg[b][k][:] = head_all[(b*R + acc[b])*K + k][:]
void launch_gather_head_dbg(const float* head_all, const int32_t* acc, float* out, int n_seq, int R,
                            int K, int V, hipStream_t s);

// ---- launchers (xsm_kernels_verify.hip) --------------------------------------
constexpr int kTailWords = 128;      // scratch words of a sequence (words: [n_seq][kTailWords]); tickets: [n_seq] zeros, zero again
                                     // after each kernel
void launch_verify(const float* Z0, const float* Hf, const int32_t* block, const int32_t* eff_len,
                   const int32_t* slot, const xsm_verify_params& vp, int32_t* acc, int32_t* y0,
                   uint32_t* wflags, int32_t* row_index /*optional: b*R + accepted*/, int32_t* words, uint32_t* tickets, float* G,
                   int n_seq, int R, int V, int d, hipStream_t s);
void launch_head_act(int dtype, const float* G, const float* Hh, const void* const* bias_ptrs,
                     float* Rk, int n_seq, int K, int d, hipStream_t s);
void launch_emit(const float* Zh, const xsm_verify_params& vp, const int32_t* eff_len,
                 const int32_t* slot, const int32_t* acc, const int32_t* y0,
                 const uint32_t* wflags, int32_t* words, uint32_t* tickets, int32_t* block, int32_t* kv_len,
                 int32_t* out_tokens, int32_t* n_accepted, uint32_t* flags, int n_seq, int R, int K, int V,
                 hipStream_t s);
void launch_copy_f32(const float* src, float* dst, size_t n, hipStream_t s);
// cache of one slot <-> float staging [H][n_pos][hd]; layout: 0 rows [pos][hd], 1 keys / 2 values in
// fragment order
void launch_kv_convert(int dtype, void* slot_base, float* staging, int H, int pos0, int n_pos,
                       int hd, int cap, int layout, int to_cache, hipStream_t s);

}  // namespace xsm
