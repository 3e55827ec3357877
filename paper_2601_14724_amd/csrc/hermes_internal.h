// Internal declarations shared by the host entry points (hermes_api.cpp) and
// the gfx950 kernels (*.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hermes.h"

namespace hermes {

constexpr int kMaxLayers = HERMES_MAX_LAYERS;
constexpr int kMaxHalfDim = 64;   // frequency pairs of the largest head size (128)
// Summary metadata per layer: insert index, stream position, RoPE position
// (t with M-RoPE), evicted count, then h and w with M-RoPE.
constexpr int kSumMeta = 8;
// 3D re-indexing ranks an axis's coordinates through an LDS bitmap over a
// window of this many consecutive values, one window after another.
constexpr int kMropeWindow = 262144;

// Static per-layer description, uploaded once into the workspace.
struct LayerTable {
  uint16_t *k[2];
  uint16_t *v[2];
  int32_t *pos[2];
  int32_t *rpos[2];         // RoPE positions of the stored keys (null when not kept); t with M-RoPE
  int32_t *rpos_h[2];       // M-RoPE h and w coordinates (null unless three axes)
  int32_t *rpos_w[2];
  float *w;
  float *s_dbg;
  int32_t *kept_dbg;
  int32_t cap;
  int32_t budget;
  int32_t cls;
  int32_t pad_;
  double lambda;
  double omega;
};

// What an attention launch needs of one entry (layer), in one piece: the
// launch's first loads are then one 32-byte read of its arguments, with no
// read of the layer table behind it (a one-token query took 14.7 us a layer
// with an array for each field and the pointers in the layer table, 13.4 so).
struct AttnEntry {
  uint16_t *k, *v;          // the current buffer of the layer's cache
  int32_t T0;               // its cached rows
  int32_t st_off, st_tiles; // stream and split mode, see AttnArgs
  int8_t layer, slot, cur;  // slot: index of the layer's inputs in the stacked tensors
  int8_t pad_;
};

// Chunk (or query) attention: entry e[j] reads the T0 cached rows of its layer
// and new rows from the stacked inputs at its slot (stride *_lstride elements),
// writes out (if non-null) and lse (if non-null).
struct AttnArgs {
  const LayerTable *tab;
  const uint16_t *q, *kn, *vn;
  uint16_t *out;
  float *lse;               // [n_layers][Hkv][C*G] log2-domain row LSE, or null
  // Appends (pos non-null): the launch also copies the new rows and their
  // positions into rows [T0, T0 + C) of the current buffer.
  const int32_t *pos;
  const int32_t *rope_pos;  // RoPE positions of the new rows (null: = pos); t with M-RoPE
  const int32_t *rope_h, *rope_w;   // M-RoPE h and w of the new rows (null unless three axes)
  int64_t q_lstride, kv_lstride, lse_lstride;
  int32_t Hq, Hkv, C;
  float scale_log2;         // sm_scale * log2(e)
  // Stream mode: the key tiles of every (entry, KV head) pair, concatenated in
  // pair order (entry j's Hkv pairs of e[j].st_tiles tiles each start at tile
  // e[j].st_off; st_total tiles in all), are cut into st_units equal ranges of
  // nqt workgroups each.  Unit u writes the unnormalised O, running maximum
  // and row sum (fp32) of each pair k it touches to opart / mlpart block u + k
  // of part_groups 32-row groups; a combine kernel merges each pair's blocks.
  // Split mode (`split`): pair k's steps are cut into e[j].st_tiles ranges of
  // st_units steps, entry j's ranges from e[j].st_off; range x writes block x.
  // split 1: up to kSplitRows packed rows, workgroups of four waves, steps of
  // 128 keys (64 with more than 32 rows); split 2: key_groups key groups, steps
  // of 128 keys (256 with 8 groups).
  // st_units = 0: the plain kernel, one workgroup per (entry, KV head, query
  // tile).
  int32_t split;
  int32_t st_units, st_total, st_entries, part_groups;   // (st_entries: the launch's entries, in every mode)
  int32_t key_groups;       // 1, 2, 4 or 8 groups of waves that share the keys (256 / key_groups rows a workgroup)
  float *opart;             // [..][part_groups][d / 8][64 lanes][4 channels] fp32 (unnormalised; scale in mlpart)
  float *mlpart;            // [..][part_groups * 32][2] fp32 (max, sum)
  AttnEntry e[kMaxLayers + 1];   // (the last one used has only st_off)
};

// What a mass sweep needs of one entry, in one piece as in AttnEntry.
struct MassEntry {
  const uint16_t *k;        // the current buffer of the layer's cache
  float *w;                 // the layer's mass
  int32_t T0, ncand;
  int8_t layer, slot;
  int8_t alpha_mode;        // weighting of the normaliser partials (0 per observer, 1 plain)
  int8_t pad_;
};

// Attention-mass sweep: W_i for the candidates i < ncand of each entry's layer
// (ncand = T0 + C for the chunk's own mass, T0 for a guidance prompt, whose
// rows are not candidates).  Each KV head's share, cut into
// `splits` ranges of its query rows, goes to wpart[layer - layer0][kv * splits +
// split][i] (fp64, rows of wpart_hstride), then is summed into the layer's w
// buffer in that order.
struct ColsumArgs {
  const uint16_t *q, *kn;
  const float *lse;
  double *wpart;
  double *normpart;         // [n_layers][normpart_lstride] fp64 partials of sum_i alpha_i W_i
  int64_t q_lstride, kv_lstride, lse_lstride, wpart_lstride, wpart_hstride, normpart_lstride;
  int32_t Hq, Hkv, C;
  int32_t splits;           // workgroups that share a block's query rows (1: none)
  int32_t layer0;           // the layer whose partials wpart starts with
  float scale_log2;
  MassEntry e[kMaxLayers];
};

// Scoring, smoothing and selection; one workgroup per listed layer.  len and
// cur are indexed by LAYER (the smoothing reads layer l+1).
struct SelectArgs {
  const LayerTable *tab;
  uint32_t *keys;           // [n_layers][max_cap]
  int32_t *kept;            // [n_layers][max_budget]
  const double *normpart;   // normaliser partials written with W (kNormBlock candidates each)
  int64_t keys_lstride, kept_lstride, normpart_lstride;
  double forget_rate;
  int32_t n_layers, C, alpha_mode, align_mode;
  int32_t n_list;           // layers over budget, in layer_id
  int32_t len[kMaxLayers];
  int32_t guide_rows[kMaxLayers];   // by layer: > 0 = W came from that many prompt rows
  double inv_z[kMaxLayers];   // by layer: 1 / Z, Z = sum_{i<len} e^{-k i} = (1 - e^{-k len}) / (1 - e^{-k})
  double ek;                  // e^{k}
  double inv_c;               // 1 / C
  int8_t cur[kMaxLayers];
  int8_t layer_id[kMaxLayers];
};

// Order-preserving gather of kept rows into the other buffer of each pair,
// optionally with a summary row inserted and with RoPE re-indexing.
// mode[j] 0: rows [0, row_start[j+1] - row_start[j]) of the other buffer
// from the kept list (and the summary row when has_sum[j]); mode 1: the
// layer did not evict, re-index its current buffer in place.
struct GatherArgs {
  const LayerTable *tab;
  const int32_t *kept;
  int64_t kept_lstride;
  int32_t row_elems;        // Hkv * d
  int32_t head_dim;
  int32_t n_list;
  int32_t reindex;          // 0 never, 1 always, 2 when *flag != 0
  int32_t rope_offset;
  double inv_freq[kMaxHalfDim];   // RoPE frequencies theta_j = base^(-2j/d), host-computed
  const int32_t *flag;      // lazy re-indexing decision (device)
  const uint16_t *sum_k, *sum_v;   // [n_layers][row_elems] staged summary rows
  const int32_t *sum_meta;  // [n_layers][kSumMeta]
  int32_t axes;             // 1, or 3 for M-RoPE (t, h, w)
  int32_t section[3];       // M-RoPE: frequency pairs of the t, h, w sections
  const int32_t *newc;      // M-RoPE: [n_layers][3][newc_lstride] re-indexed coordinates by output row
  int64_t newc_lstride;
  int32_t row_start[kMaxLayers + 1];   // prefix of output rows over the list
  int8_t layer_id[kMaxLayers];
  int8_t cur[kMaxLayers];
  int8_t mode[kMaxLayers];
  int8_t has_sum[kMaxLayers];
};

// Summary token of every listed (deep, evicting) layer: fp64 partial sums of
// the evicted rows per block of kSummaryRows candidates, then the mean.
struct SummaryArgs {
  const LayerTable *tab;
  const int32_t *kept;
  int64_t kept_lstride;
  double *part;             // [n_layers][blocks][2 * row_elems]
  int64_t part_lstride;
  uint16_t *sum_k, *sum_v;  // [n_layers][row_elems]
  int32_t *sum_meta;        // [n_layers][kSumMeta]
  int32_t row_elems, head_dim, n_list;
  int32_t axes;             // 3: keys aligned to the target's (t, h, w) section by section
  int32_t section[3];
  double inv_freq[kMaxHalfDim];   // RoPE frequencies theta_j = base^(-2j/d), host-computed
  int32_t len[kMaxLayers];      // by entry: candidates T
  int32_t budget[kMaxLayers];   // by entry: kept M
  int8_t layer_id[kMaxLayers];
  int8_t cur[kMaxLayers];
};

// Lazy re-indexing decision: the largest RoPE position each layer retains
// after this compression, against limit - headroom.
struct DecideArgs {
  const LayerTable *tab;
  const int32_t *kept;
  int64_t kept_lstride;
  const int32_t *sum_meta;
  int32_t *flag;
  int32_t n_layers, limit, headroom;
  int32_t axes;             // 3: the largest of the t, h and w coordinates
  int32_t len[kMaxLayers];      // by layer: T before compression
  int32_t budget[kMaxLayers];
  int8_t cur[kMaxLayers];
  int8_t evicts[kMaxLayers];
  int8_t has_sum[kMaxLayers];
};

// M-RoPE ranks (appendix, 3D re-indexing): for list entry j and axis a, the
// coordinate of every output row (mode 0: kept row kept[r] of the current
// buffer; mode 1: row r in place) becomes offset + the number of distinct
// retained coordinates below it, written to newc[layer][a][r].
struct RankArgs {
  const LayerTable *tab;
  const int32_t *kept;
  int64_t kept_lstride;
  const int32_t *sum_meta;  // summary rows (has_sum): insert index and (t, h, w)
  int32_t *newc;
  int64_t newc_lstride;
  const int32_t *flag;      // lazy decision (device)
  int32_t reindex;          // 0 never, 1 always, 2 when *flag != 0
  int32_t offset;
  int32_t n_list;
  int32_t row_start[kMaxLayers + 1];
  int8_t layer_id[kMaxLayers];
  int8_t cur[kMaxLayers];
  int8_t mode[kMaxLayers];
  int8_t has_sum[kMaxLayers];
};

// Device scratch of the no-allocation context entry point (scratch.hip):
// kStaticWorkspaceBytes per GPU.  acquire looks up the array's address on the
// current device (once per device) and marks it owned: HERMES_ESTATE while
// another context owns it, HERMES_ENOTSUP beyond kMaxDevices GPUs.
constexpr size_t kStaticWorkspaceBytes = (size_t)HERMES_STATIC_WORKSPACE_BYTES;
constexpr int kMaxDevices = 64;
int static_workspace_acquire(void **ptr, int *device);
void static_workspace_release(int device);

// Launchers (return the hipError_t of the launch).
hipError_t launch_attention(const AttnArgs &a, int n_list, int head_dim, hipStream_t s);
hipError_t launch_attention_parted(const AttnArgs &a, int n_list, int head_dim, hipStream_t s);
hipError_t launch_colsum(const ColsumArgs &a, int n_list, int max_T, int head_dim,
                         hipStream_t s);
hipError_t launch_select(const SelectArgs &a, hipStream_t s);
// Precondition checks (device side): q, k, v bf16 with nq / nkv elements
// (multiples of 8, 16-byte aligned), the chunk positions pos[0..n_new) (or
// null) against the last cached position of each listed layer; violations
// are ORed into *flag.
struct CheckArgs {
  const LayerTable *tab;
  const uint16_t *q, *k, *v;
  int64_t nq, nkv;
  const int32_t *pos;
  int32_t n_new;
  int32_t n_list;
  int32_t len[kMaxLayers];
  int8_t layer_id[kMaxLayers];
  int8_t cur[kMaxLayers];
  int32_t *flag;
};

hipError_t launch_check(const CheckArgs &a, hipStream_t s);
hipError_t launch_gather(const GatherArgs &a, hipStream_t s);
hipError_t launch_topk(const float *keys, int n, int k, int32_t *out, hipStream_t s);
hipError_t launch_summary(const SummaryArgs &a, int max_T, hipStream_t s);
hipError_t launch_decide(const DecideArgs &a, hipStream_t s);
hipError_t launch_gather_rope(const GatherArgs &a, hipStream_t s);
hipError_t launch_mrope_rank(const RankArgs &a, hipStream_t s);

// Geometry shared by host sizing and kernels.
constexpr int kAttnRowsPerBlock = 256;   // packed (row, head) pairs per attention workgroup
constexpr int kColsumKeysPerBlock = 256; // candidates per workgroup of the sweep
constexpr int kMassSplitMax = 32;       // ranges a sweep's query rows are cut into at most
constexpr int kSummaryRows = 128;        // candidates per workgroup of the summary sums
constexpr int kSplitMaxTokens = 64;      // rows of a query or prompt that may share a room of partial rows
constexpr int64_t kRoomRows = 131072;    // partial rows of a stream's longer passes at most (68 MB at head size 128)
constexpr int kStreamRooms = 3;          // streams with a room of their own
constexpr int kStreamSlots = 256;        // resident attention workgroups (one per CU)
constexpr int kSplitRows = 128;          // packed rows of a split-mode workgroup at most
constexpr int kNormBlock = 256;         // candidates per fp64 partial of the score normaliser

// How a context cuts calls, worked out on the host alone (no device, no
// launches): for tests.  limit: bytes of workspace (0: what the configuration
// asks for).  The calls are taken in order, as one context would see them.
enum { PLAN_APPEND = 0, PLAN_QUERY = 1, PLAN_PROMPT = 2 };
struct PlanCall {
  int32_t kind, n_rows, layer, captured;
  uint64_t stream;          // the stream's handle (0: the null stream)
  const int32_t *len;       // [n_layers] cached rows of every layer
};
struct PlanInfo {
  int32_t key_groups, mode, four_waves, units;   // mode 0 plain, 1 stream, 2 split
  int32_t splits, pad_;     // of the sweep (0: none)
  int64_t rows;             // partial rows the pass may write
  int64_t o_lo, o_hi, ml_lo, ml_hi;   // and where, as bytes of the workspace
  int64_t sweep_lo, sweep_hi;         // and the sweep's partials
  int64_t total;            // bytes of the layout
};
extern "C" int hermes_plan_probe(const hermes_config *cfg, size_t limit, const PlanCall *calls, int n_calls,
                                 PlanInfo *out);

}  // namespace hermes
