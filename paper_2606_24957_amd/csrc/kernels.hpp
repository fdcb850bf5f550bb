// kernels.hpp -- argument blocks and launchers of the libdustin kernels (internal).
#pragma once

#include "common.hpp"

namespace dustin {

// ---- verification attention (attn.hip) ----
constexpr int kAttnMaxSplits = 32;  // token splits per (b, g)

struct AttnArgs {
  const uint16_t* q;
  int64_t q_sb, q_st, q_sh;
  uint16_t* out;
  int64_t o_sb, o_st, o_sh;
  KvView k, v;          // paged K and V share one page table and page size
  SeqDims dims;
  const int32_t* idx;   // NULL: dense (every committed position)
  int64_t idx_sb, idx_sg;
  const int32_t* count;
  int32_t groups;
  int32_t num_kv_heads, group_size;
  int32_t pairs;        // B * num_kv_heads
  float scale_log2;
  int32_t splits;           // splits of each pair when all are equally long
  int32_t units;            // unit slots of the launch, at least pairs * splits
  int32_t split_steps;      // 32-token steps per split when every pair is as long as the longest
  int32_t min_split_steps;  // smallest split the kernel's balancing may choose
  int32_t rows_pad;
  float* part_acc;          // [units, rows_pad, 128], by unit  (units > pairs only)
  float* part_ml;           // [units, rows_pad, 2]
  int32_t* counters;        // one per kAttnCounterStride, marks from kAttnMaskOffset on; zero between calls
  int32_t merge_spins;      // polls after which a split leaves its share of the merge to the last
};

// Row tiles (16 query rows each) up to which the attention kernel gives the verification
// window's tokens a step of their own; beyond that they share the last step with the
// selected (or committed) positions.
constexpr int kAttnSepMaxRT = 3;

// Splits of a pair up to which the last to finish merges alone (16 sequences, 8 KV heads, 2048
// tokens, two splits: 35.1 us, shared 37.5).
constexpr int kAttnMergeAlone = 3;

// Looks at the arrival counter after which a split waits no longer: about a millisecond, which bounds
// what splits lose that hold CUs while another launch holds those of the splits they wait for.  Alone,
// 16 sequences, dense, one of 65536 tokens and 15 of 4096, need the most: 99 us with 256 looks, 116
// with 64, 130 with one (8 KV heads of 2048 tokens: 14.6 us with 16 looks, 50 with one).  Two streams
// of such launches in turn take no longer a pair than two launches on one.
constexpr int kAttnMergeSpins = 1 << 10;

// Pairs the attention kernel's split balancing handles (four per lane of one wave); with
// more pairs there is one workgroup per pair.
constexpr int kAttnBalancePairs = 256;  // (and one round of its workgroups)

// int32 between the arrival counters of two pairs (each in a cache line and a memory channel of
// its own: 256 workgroups poll and count at once), and from a counter to the pair's marks of
// slices left undone.
constexpr int kAttnCounterStride = 64, kAttnMaskOffset = kAttnBalancePairs * kAttnCounterStride;

hipError_t launch_verify_attn(const AttnArgs& a, int rt, bool sparse, bool paged, hipStream_t stream);

// ---- scoring-head importance (score.hip) ----
constexpr int kScoreWaves = 4;
constexpr int kScoreChunk = 1024;        // positions per pass-1 workgroup
constexpr int kScorePageChunk = 256;     // pages per pass-1 workgroup in page mode (or twice as many)
constexpr int kScoreFinishChunk = 1024;  // positions per pass-2 workgroup (4 per thread)
constexpr int kScoreFinishPages = 64;    // pages per pass-2 workgroup in page mode
constexpr int kScoreMaxHeads = 64;
constexpr int kScoreMaxEntries = 64;     // pass-1 column tiles: (KV head, up to 16 pairs)
constexpr int kScoreGroupTiles = 3;      // column tiles of one KV head per pass-1 workgroup
constexpr int kScoreMaxLayers = 32;
constexpr int kScoreMaxPairs = 1024;     // (layer, head, query) rows one output sums
// Single-pass form (score_sync.hip): the workspace starts with kScoreSyncBytes of
// per-sequence counters (zero between calls) and a timeout flag; every form of the score
// keeps its logits and statistics after them.
constexpr int kSyncWaves = 16;             // waves per single-pass workgroup
constexpr int kScoreSyncMaxBatch = 2048;   // sequences the counters cover
constexpr int kScoreSyncMaxChunks = 128;   // chunks of one sequence (far below the chip's CUs)
constexpr int64_t kScoreSyncPositions = INT64_C(192) * 2048;  // positions from which chunks of 2048 fill the chip
constexpr int kScoreSyncCUs = 256;         // MI355X compute units: one single-pass workgroup each
constexpr size_t kScoreSyncBytes = 16896;  // 2 * kScoreSyncMaxBatch counters + the flag, 256-aligned
static_assert(kScoreSyncBytes >= (2 * kScoreSyncMaxBatch + 1) * 4 && kScoreSyncBytes % 256 == 0, "sync region");
static_assert(kScoreSyncBytes == DUSTIN_SCORE_SYNC_BYTES && 2 * kScoreSyncMaxBatch * 4 == DUSTIN_SCORE_SYNC_FLAG_OFFSET,
              "the workspace layout the header documents");

// Eq. 5 over the positions of a cache, or (page mode) over the pages of a page-statistics
// array, whose rows [max | min] of length 2d meet the sign-split query [q+ | q-].
struct ScoreArgs {
  const uint16_t* q_layers[kScoreMaxLayers];  // queries of each scored layer (same strides)
  int64_t q_sb, q_sj, q_sh;
  KvView k;                                  // K view shared by the layers, but for its data
  const uint16_t* k_layers[kScoreMaxLayers];
  int32_t n_layers, batch;
  SeqDims dims;
  int32_t page_mode;   // 0: rows of k are positions; 1: rows are pages of page statistics
  int32_t page_shift;  // page mode: log2 of the page size (0 otherwise)
  int32_t chunk;       // rows per pass-1 workgroup
  int32_t heads[kScoreMaxHeads];
  int32_t n_heads;
  int32_t used_kv[kScoreMaxEntries];       // KV head of each pass-1 column tile
  int32_t pairs_per_kv[kScoreMaxEntries];  // (head, query) pairs of that tile
  uint8_t tile_first[kScoreMaxEntries];    // pass-1 workgroup x: its first tile
  uint8_t tile_count[kScoreMaxEntries];    // and its tile count (same KV head)
  uint8_t pair_head[kScoreMaxEntries * 16];   // head slot of pair i of tile u
  uint8_t pair_query[kScoreMaxEntries * 16];  // query of that pair
  int32_t group_size, groups;
  float scale_log2;
  const float* init;
  int64_t init_sb, init_sg;
  float* out;
  int64_t out_sb, out_sg;
  int32_t per_layer;  // 1: layer l writes out + l * out_sl (no init); 0: layers summed
  int64_t out_sl;
  float* logits;  // [n_layers, B, n_heads, nq_max, ld]  scaled logits, log2 domain
  float* stats;   // [n_layers, B, n_heads, nq_max, n_chunks, 2]  (max, sum of exp2) per chunk
  int64_t ld;
  int32_t nq_max, n_chunks;
  // optional: one count per written position added to hist[(b groups + go) kDigitBins +
  // order_key(out) >> 20] (summed outputs only)
  uint32_t* hist;
};
static_assert(sizeof(ScoreArgs) <= 4096, "kernel arguments stay within 4 KiB");

// n_groups pass-1 workgroups along x (tile_first / tile_count), max_group the largest
// tile count; row_dim: length of a K row (head_dim, or 2 * head_dim for page statistics)
hipError_t launch_score(const ScoreArgs& a, int B, int n_groups, int max_group, int row_dim, hipStream_t stream);

// One call of the single-pass form (score_sync.hip): columns 0 .. np - 1 are (query head
// col_head, query col_query) pairs on used KV head kv[col_u]; chunks of 256 tw positions,
// `chunks` per sequence, a sequence's chunks on one XCD when `local`.
struct SyncCall {
  const uint16_t* q_layers[kScoreMaxLayers];
  const uint16_t* k_layers[kScoreMaxLayers];
  int64_t q_sb, q_sj, q_sh;
  KvView k;
  SeqDims dims;
  const float* init;
  int64_t init_sb;
  float* out;
  int64_t out_sb;
  float* stats;   // [n_layers, batch, chunks, 16] (max, sum of exp2) per chunk and column
  int32_t* sync;  // the workspace's counter region (zero between calls) and timeout flag
  float scale_log2;
  int32_t batch, n_layers, head_dim, nu, tw, np, chunks, local;
  int32_t extent;  // bytes of K rows one buffer resource covers (a sequence, or the page pool)
  int32_t kv[4];
  int32_t col_head[16];
  uint8_t col_query[16], col_u[16];
  uint32_t* hist;  // optional: as ScoreArgs::hist (one output row per sequence)
};

struct SyncArgs {
  SyncCall call[2];
  int32_t blocks0;  // blocks of call 0 (set by the launcher)
};
static_assert(sizeof(SyncArgs) <= 4096, "kernel arguments stay within 4 KiB");

// the single-pass form of one call; and of two calls in one launch, for the pairs of
// shapes score_sync_pair_supported accepts
hipError_t launch_score_sync(const SyncArgs& a, hipStream_t stream);
bool score_sync_pair_supported(const SyncCall& c0, const SyncCall& c1);
hipError_t launch_score_sync_pair(const SyncArgs& a, hipStream_t stream);

// ---- score calls by chunks of four-wave workgroups (score_once.hpp, score_reread.hip) ----
constexpr int kChunkWaves = 4;
constexpr int kChunkMaxTW = 16;            // most 16-position tiles per wave
constexpr int64_t kChunkMaxBlocks = (INT64_C(1) << 32) / (kChunkWaves * kWave) - 1;  // a grid has less than 2^32 threads
constexpr int kChunkMaxOnce = 256;         // most chunks of a sequence in score_once.hpp
// Most int32 between the counters of two units: as far apart as the region allows, so that the
// polls and counts of one unit's workgroups do not queue behind another's in a cache line and memory
// channel (per-layer calls of 16 units of 8192 positions, 28 pairs: adjacent 26.3 us, apart 14.7;
// score_reread.hip, 24 layers of 16 x 16384, 56 pairs: 866 us, 640).
constexpr int kChunkSyncStride = 64;
// Looks at a counter (each a memory round trip) before a wait ends: some milliseconds, where calls that
// share the chip with nobody need up to 512 (24 pairs, three layers of 16 x up to 32768, several rounds
// of workgroups: 77 us, with 128 looks 1041).
constexpr int kChunkPolls = 1 << 12;
constexpr int kChunkMaxTiles = 4;          // most column tiles of 16 pairs
constexpr int kChunkMaxQ = 12;             // most column tiles times layers that one output sums (score_reread.hip)

// One call: column i < cols[t] of column tile t is the pair (query head col_head, query
// col_query)[16 t + i] on used KV head kv[col_u]; nt = 0: one tile for the pairs of all nu KV
// heads, else tiles u nt .. u nt + nt - 1 belong to KV head kv[u].  A sequence has at most
// `chunks` chunks of 64 tw positions.
struct ChunkCall {
  const uint16_t* q_layers[kScoreMaxLayers];
  const uint16_t* k_layers[kScoreMaxLayers];
  int64_t q_sb, q_sj, q_sh;
  KvView k;
  SeqDims dims;
  const float* init;
  int64_t init_sb;
  float* out;
  int64_t out_sb, out_sl;
  float* stats;   // (max, sum of exp2) of every chunk and column
  int32_t* sync;  // the workspace's counter region (zero between calls)
  int32_t polls;  // looks at a counter after which a workgroup waits for the others no longer
  float scale_log2;
  int32_t batch, n_layers, per_layer, head_dim, nu, nt, tw, chunks;
  int32_t sync_stride;  // the launcher's: int32 between two units' counters
  int32_t share_merge;  // score_once.hpp: every workgroup of the call gets a slot at once
  int32_t extent;  // bytes of K rows one buffer resource covers (a sequence, or the page pool)
  int32_t kv[4];
  int32_t cols[kChunkMaxTiles];
  int32_t col_head[16 * kChunkMaxTiles];
  uint8_t col_query[16 * kChunkMaxTiles], col_u[16 * kChunkMaxTiles];
  uint32_t* hist;  // optional: as ScoreArgs::hist (one output row per sequence)
};

struct ChunkArgs {
  ChunkCall call[2];
  int32_t units, lag;  // the launcher's: score_once.hpp, score_reread.hip
};
static_assert(sizeof(ChunkArgs) <= 4096, "kernel arguments stay within 4 KiB");

// small calls in one pass (score_once.hpp): one call, or two in one launch
bool score_once_supported(const ChunkCall& c);
bool score_once_pair_supported(const ChunkCall& c0, const ChunkCall& c1);
hipError_t launch_score_once(const ChunkArgs& a, int n_calls, hipStream_t stream);

// calls that read K twice (score_reread.hip)
bool score_reread_supported(const ChunkCall& c);
hipError_t launch_score_reread(const ChunkArgs& a, hipStream_t stream);

// ---- attention recovery rate (arr.hip) ----
struct ArrArgs {
  const float* s;  // Eq. 5 score over the served heads and the window's queries
  int64_t s_sb, s_sg;
  const int32_t* idx;
  int64_t idx_sb, idx_sg;
  const int32_t* count;
  SeqDims dims;    // seq_lens (N_b), n_query (w_b), k_max
  int32_t groups, heads_per_group;
  double* arr;     // [B, groups]
};

hipError_t launch_arr(const ArrArgs& a, int B, hipStream_t stream);

// ---- page statistics for the page estimator (page.hip) ----
constexpr int kMaxPageSize = 4096;
struct PageMetaArgs {
  KvView k;
  SeqDims dims;
  const int32_t* from;  // device [B]: first position that changed, or NULL (= 0)
  uint16_t* meta;       // [B, pages, Hkv, 2 d]: per page, channel max then min
  int64_t m_sb, m_sp;
  int32_t num_kv_heads, page_shift, span_pages;
};

hipError_t launch_page_meta(const PageMetaArgs& a, int B, int head_dim, hipStream_t stream);

// ---- tiered selection (topk.hip) ----
struct TopkArgs {
  const float* s_draft;
  int64_t d_sb, d_sg;
  const float* s_target;
  int64_t t_sb, t_sg;
  SeqDims dims;
  int32_t groups, n_sink, n_window;
  int32_t* idx;
  int64_t idx_sb, idx_sg;
  int32_t* count;
  // hand-off between the two tiers of a row (both score arrays given): per (b, go) an
  // arrival counter (zero between calls) and two chosen-set bitmaps of `words` words
  uint32_t* counters;  // [B * groups]
  uint32_t* bitmaps;   // [B * groups][2][words]
  int32_t words;
  // optional (groups = 1): per sequence the top-digit histogram of the whole row of S_D /
  // S_T, which replaces the tier's first pass and is returned to zero
  uint32_t* hist_d;
  uint32_t* hist_t;
};

hipError_t launch_topk(const TopkArgs& a, int B, hipStream_t stream);

// ---- verification window K/V into the caches, and the commit of accepted tokens (kv.hip) ----
struct KvAppendArgs {
  const uint16_t* k_new;
  int64_t k_sb, k_st, k_sh;
  const uint16_t* v_new;
  int64_t v_sb, v_st, v_sh;
  KvView k, v;   // the caches (written)
  SeqDims dims;  // seq_lens (N_b), n_query (T_b), max_len, nq_max
  int32_t batch, num_kv_heads, head_dim;
};

hipError_t launch_kv_append(const KvAppendArgs& a, hipStream_t stream);
hipError_t launch_kv_commit(int32_t* seq_lens, const int32_t* accepted, const int32_t* n_query, int nq_max,
                            int batch, hipStream_t stream);

}  // namespace dustin
