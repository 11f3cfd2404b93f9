// Host-side launchers for the libmemattn kernels and the selection plan.
// Internal to the library: the public interface is include/memattn.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace memattn {

// How one retrieval/relation call is split over the GPU.
struct Plan {
  bool mfma;              // fused bf16 matrix-core path (else the general score and select path)
  int qw;                 // matrix-core workgroup shape: 64 * qw queries (1, 2 or 4)
  int tile_rows;          // bank rows per matrix-core tile (512 for qw = 1, else 256)
  int tile_queries;       // queries per matrix-core workgroup
  int kcap;               // partial list length per split (power of two >= k)
  int n_splits;           // bank splits per query row
  int n_parts;            // partial (list, max, sum) entries per query row seen by the merge
  int part_stride;        // ... at every part_stride-th workspace slot
  int64_t rows_per_split; // bank rows per split (multiple of the row tile)
  int q_tiles;            // query tiles (MFMA path)
  int tiles_per_split;    // bank tiles per split (MFMA path)
  size_t ws_part_keys;    // byte offsets into the workspace
  size_t ws_part_ms;
  size_t ws_lse2;
  int ns;                 // sampled tiles per sampled split (0 = no threshold sample)
  int samp_stride;        // every samp_stride-th split is sampled
  int n_samp_splits;      // sampled splits
  int64_t n_samp;         // sample scores per query (n_samp_splits * ns * tile)
  size_t ws_samp;         // 16-bit sample order keys [m, n_samp]
  size_t ws_t0;           // sampled k-th-best lower bound per query [m]
  size_t ws_thr;          // per-query score bound shared by its partials [m] (order keys)
  int ph_split;           // matrix-core full pass in two launches split at this tile of each split (0: one)
  size_t ws_lane_ms;      // per-slot softmax state between the two launches [m, slots] (float2)
  int order;              // room for the clustered query order (used by relation builds with a sample)
  size_t ws_near;         // best sampled position, then order label, per query [m] (int32)
  size_t ws_perm;         // clustered position -> query [m] (int32)
  size_t ws_olab;         // label of each sampled position [kOrderMaxSample] (int32)
  size_t ws_ocnt;         // queries per label, then each label's first position [kOrderMaxSample] (int32)
  size_t ws_orank;        // each query's rank among its label's queries [m] (int32)
  size_t ws_stop;         // each query's sampled keys at or above its k-th, with positions [m, 64] (uint32)
  size_t ws_qbuf;         // the queries in clustered order [m, d] (bf16)
  int64_t blk_queries;    // general path: queries and bank rows scored at a time
  int64_t blk_rows;
  size_t ws_part_lo;      // low words of the partial softmax sums [m, n_splits] (float); with one split,
                          // all partials are those of a block's queries
  size_t ws_scores;       // the block's scores [blk_queries, blk_rows] (float)
  size_t ws_bytes;        // total workspace bytes
};

constexpr int kMfmaTile = 256;   // bank rows and query rows per workgroup tile
constexpr int kMfmaMaxK = 32;    // largest k served by the matrix-core path
// Clustered query order: from this many queries on (a wave's 64 lanes can
// then share a region of the bank), while the reordered copy of the queries
// stays within 1 GiB, and for samples of at most 32,768 positions (the order
// kernel's labels live in LDS).
constexpr int64_t kOrderMinQueries = 4096;
constexpr size_t kOrderMaxQueryBytes = size_t{1} << 30;
constexpr int64_t kOrderMaxSample = 32768;
constexpr int64_t kOrderSampleFloor = 1024;  // fewest sampled rows of a relation build in that order
// Matrix-core workgroup shapes by query count: 64 x 512-row tiles (<= 64
// queries), 128 x 256 (<= 128), else 256 x 256; every wave owns 128 rows of
// a tile, so a split keeps tile_rows / 128 partials while the kernel runs.
constexpr int kSelectRows = 4096;  // scores per step of the general path's select kernel
constexpr int64_t kSelectOneSplit = 16384;  // banks of at most so many rows take one split per query there
constexpr size_t kScoreBlock = size_t{96} << 20;  // most bytes of scores it holds at a time
constexpr int kMaxK = 64;
constexpr int kMaxD = 8192;

// Namespace scope of a selection (both NULL = the whole bank): row j is a
// candidate of query i only if row_ns[j] >= 0 and row_ns[j] == key_ns[i].
struct Scope {
  const int32_t* row_ns;  // device [n]; negative = tombstoned row
  const int32_t* key_ns;  // device [m]; negative = no candidates
};

// mfma_ok: caller allows the matrix-core path (bf16, d % 32 == 0, k <= 32,
// no full probability output).  relation: the queries are the bank's own
// rows, scoped: it takes namespaces (the sample size and the path, and with
// the path the plan's ws_bytes, depend on them; mem_workspace_bytes covers
// every path).
Plan make_plan(int64_t m, int64_t n, int32_t d, int32_t k, int32_t dtype, bool mfma_ok, bool relation, bool scoped);
// Grouped selection over per-namespace chunk tables: the narrow matrix-core
// shape, S splits per namespace (S from the mean table size), no sample.
Plan make_grouped_plan(int64_t m, int32_t n_ns, int64_t n_entries, int32_t k);
// The same over tables that the device collects (room for kScopeMaxSplits).
Plan make_scope_plan(int64_t m, int64_t n, int32_t k);

// General path: scores block by block, each block followed by its selection.
// `self_base` >= 0 removes bank row self_base + i from query i's candidates.
// With one split per query (p.n_splits == 1) the results are final, the full
// probability rows included; else the partials are left for the merge.  All
// launches go to `stream`.
hipError_t launch_topk_score(const Plan& p, const void* bank, int64_t bank_stride, int64_t n, const void* queries,
                             int64_t q_stride, int64_t m, int32_t d, int32_t dtype, float c2, int64_t self_base,
                             int32_t k, const Scope& scope, void* ws, float* full_scores, int32_t* idx, float* score,
                             float* prob, float* lse, hipStream_t stream);
// With p.ns > 0 a sample pass over the first ns tiles of every split first
// bounds each query's k-th best score from below; the full pass starts its
// thresholds there.
// `relation`: query i is bank row i (a relation build); the full pass may
// then take the queries in clustered order (p.order).  gate (scoped calls):
// where *gate != 0 on the device, nothing is done.
hipError_t launch_topk_mfma(const Plan& p, const uint16_t* bank, int64_t bank_stride, int64_t n,
                            const uint16_t* queries, int64_t q_stride, int64_t m, int32_t d, float c2,
                            int64_t self_base, int32_t k, const Scope& scope, bool relation, void* ws,
                            hipStream_t stream, const int32_t* gate);
// Grouped selection over per-namespace chunk tables: workspace regions after
// the plan's (from byte `base` on) and the launch (preparation + matrix-core
// pass; the merge follows with launch_topk_merge).  The plan must be the
// narrow matrix-core shape with n_splits = S splits per namespace.
struct GroupLayout {
  size_t q_cnt, fill, q_off, item_off, bsum, perm, qbuf, q_pos, flag, tile_off, score_off, scores;
  size_t bytes;  // what a call of these sizes uses
  size_t room;   // and what callers are asked for: no less, and never less for larger tables
  bool tables;  // few enough queries and namespaces for launch_topk_tables to be tried
};
GroupLayout group_layout(int64_t m, int32_t n_ns, int64_t n_entries, int32_t d, size_t base);
hipError_t launch_topk_grouped(const Plan& p, const GroupLayout& G, const uint16_t* bank, int64_t bank_stride,
                               int64_t n, const uint16_t* queries, int64_t q_stride, int64_t m, int32_t d, float c2,
                               int32_t k, const int32_t* ns_off, const int32_t* rows, int32_t n_ns,
                               int64_t n_entries, const int32_t* key_ns, int32_t* idx, float* score,
                               float* prob, float* lse, void* ws, hipStream_t stream);
// Chunk tables for a scoped selection (scope.hip), all device memory but the
// numbers.  A query's partials have room for max_splits splits, of which
// flags[1] are used.
constexpr int64_t kScopeMaxQueries = 4096;
constexpr int kScopeRows = 4096;     // bank rows per workgroup (four 1,024-row blocks)
constexpr int kScopeMaxSplits = 16;  // splits of a table
struct ScopeArgs {
  const int32_t* row_ns;    // [n]
  const int32_t* query_ns;  // [m]
  int64_t n, m;
  int bits;                 // log2 of the hash table's slots, at least twice m
  int64_t n_blocks;         // 1,024-row blocks, rounded up to a multiple of 4
  int32_t* key;             // [slots] namespace ids, -1 = free
  int32_t* num;             // [slots] and their numbers
  int32_t* flags;           // tables used, splits per table, namespaces, entries
  int32_t* table;           // [m, 2] first and past-the-last entry of each namespace's table
  int32_t* counts;          // [m, n_blocks]
  int32_t* chunks;          // [n] the tables' entries
  int64_t* q_off;           // [m + 1] as the grouped pass takes them
  int64_t* item_off;        // [m + 1]
  int32_t* perm;            // [m]
  int32_t* q_pos;           // [m] grouped position of each query, -1 = none
  uint32_t* thr;            // [m] shared bounds, cleared here
  uint64_t* part_keys;      // partials of queries without a namespace, emptied here
  float2* part_ms;
  int max_splits, part_stride, kcap;
  const void* queries;      // [m] rows of d bf16, q_stride elements apart, copied to qbuf in grouped order
  int64_t q_stride;
  int32_t d;
  void* qbuf;               // [m, d]
};
hipError_t launch_scope_tables(const ScopeArgs& a, hipStream_t stream);
// Workspace of that selection (p is its grouped plan).  Its regions share
// memory with the whole-bank pass's, which runs only where they are not used
// and initialises what it reads; the flags that tell stand behind both.
struct ScopeLayout {
  Plan p;
  size_t key, num, flags, table, counts, chunks, q_off, item_off, perm, qbuf, q_pos, table_flag, tile_off, score_off,
      scores, end;
  int bits;
  int64_t n_blocks;
};
// The most bank rows that m queries' tables take (16 MiB each of entries and
// of counts).
inline int64_t scope_max_rows(int64_t m) {
  const int64_t by_counts = (int64_t{1} << 22) / m * 1024, by_entries = int64_t{1} << 22;
  return by_counts < by_entries ? by_counts : by_entries;
}
// Whether a scoped call of these sizes tries the tables at all.
bool scope_tables_fit(int64_t m, int64_t n, int32_t d, int32_t k);
ScopeLayout scope_layout(int64_t m, int64_t n, int32_t d, int32_t k, size_t whole_bank_bytes);
// The tables and the grouped pass over them, up to its partials (none of it
// does anything past the plan where flags[0] comes out 0).
hipError_t launch_topk_scope_grouped(const ScopeLayout& L, const uint16_t* bank, int64_t bank_stride, int64_t n,
                                     const uint16_t* queries, int64_t q_stride, int64_t m, int32_t d, float c2,
                                     int32_t k, const Scope& scope, int32_t* idx, float* score, float* prob, float* lse,
                                     void* ws, hipStream_t stream);

// Scores and selection over chunk tables (topk_score.hip): bf16 rows, device
// memory but the numbers.
constexpr int64_t kTableMaxNs = 4096;               // namespaces
constexpr int kTableMaxRows = 32768;                // rows of a table
constexpr int64_t kTableScores = int64_t{12} << 20; // most scores held (48 MiB)
struct TableArgs {
  const uint16_t* bank;
  int64_t bank_stride, n;
  const uint16_t* queries;  // in their own order
  int64_t q_stride, m;
  int32_t d;
  float c2;
  int32_t k;
  const int32_t* ns_off;    // tables: CSR (off_step 1) or first and past-the-last entries (2)
  int off_step;
  const int32_t* chunks;
  int64_t n_entries;
  int n_ns;
  const int64_t* q_off;     // [n_ns + 1] grouped positions of each namespace's queries
  int64_t* item_off;        // [n_ns + 1] the fused pass's work items, taken away where this side runs
  const int32_t* perm;      // grouped position -> query
  const int32_t* q_pos;     // query -> grouped position, -1 = no namespace
  int32_t* flag;            // [0] set where this side runs, [1] where the fused grouped pass does
  int32_t* tile_off;        // [n_ns + 1]
  int64_t* score_off;       // [n_ns]
  float* scores;
  int64_t max_scores;
  const int32_t* gate;      // NULL, or 0: there are no tables
  int32_t* idx;
  float* score;
  float* prob;
  float* lse;
};
hipError_t launch_topk_tables(const TableArgs& a, hipStream_t stream);

// Launches that run only where *flag == go (flag NULL: always).
struct Gate {
  const int32_t* flag = nullptr;
  int go = 0;
};
// Another set of partials that a merge takes where *flag != 0: lists of
// consecutive keys kcap apart, with room for n_parts of which *parts are used.
struct MergeAlt {
  const int32_t* flag = nullptr;
  const int32_t* parts = nullptr;
  const uint64_t* keys = nullptr;
  const float2* ms = nullptr;
  int n_parts = 0;
  int kcap = 0;
  const int32_t* done = nullptr;  // nothing is left to merge where *done != 0 (NULL: never)
};
// Optional full probability output: full[i, j] holds the raw score s_ij on
// entry and p_ij on exit (0 for the excluded row self_base + i).
struct FullProb {
  float* full = nullptr;   // device [m, n] or NULL
  int64_t n = 0;
  int64_t self_base = -1;
};
// Merge split partials into the final top-k, probabilities and lse, and
// finish the full probability rows if requested (launch_full_prob).
hipError_t launch_topk_merge(const Plan& p, int64_t m, int32_t k, float c2, int32_t* idx, float* score, float* prob,
                             float* lse, void* ws, hipStream_t stream, const FullProb& fp = FullProb{},
                             const MergeAlt& alt = MergeAlt{});
// full[i, j] <- exp2(full[i, j] * c2 - lse2[i]) (0 for the excluded row).
hipError_t launch_full_prob(const Plan& p, int64_t m, int64_t n, float c2, int64_t self_base, float* full, void* ws,
                            hipStream_t stream);

hipError_t launch_gather(const void* pool, int64_t n_pages, int64_t page_bytes, const int32_t* table,
                         int64_t n_chunks, int32_t ppc, const int32_t* ids, int64_t count, int32_t order,
                         int32_t group, void* out, hipStream_t stream);

// Budget-aware, time-ordered materialisation of rank-ordered ids [m, k]
// into [m, budget, row_bytes] token rows.
hipError_t launch_gather_budget(const void* pool, int64_t n_pages, int64_t page_bytes, const int32_t* table,
                                int64_t n_chunks, int32_t ppc, const int32_t* tok_len, int32_t row_bytes,
                                const int32_t* ids, int64_t m, int32_t k, int32_t budget, void* out,
                                int32_t* out_tokens, int32_t* out_ids, hipStream_t stream);

// Background block compaction: workspace layout (byte offsets) and the two
// launch phases.  The plan phase leaves {moving pages, fresh pages,
// compacted blocks, malformed-table flag} in totals_host[0..3] and
// synchronises `stream`; the move phase copies the pages and updates the
// directory.
struct CompactLayout {
  int64_t n_blocks;
  size_t live, cand, pos, bsum, ns_base, moves, counter, flags, totals, bytes;
};
CompactLayout compact_layout(int64_t next_free, int32_t P, int64_t n_entries, int32_t ppc, int32_t n_ns);
hipError_t launch_compact_plan(const CompactLayout& L, const int32_t* table, int64_t n_chunks, int32_t ppc,
                               const int32_t* offsets, const int32_t* chunks, int32_t n_ns, int64_t n_entries,
                               int32_t P, int64_t next_free, double theta, float* phi_out, uint8_t* released,
                               void* ws, int64_t* totals_host, hipStream_t stream);
hipError_t launch_compact_move(const CompactLayout& L, void* pool, int64_t page_bytes, int32_t* table,
                               int64_t n_chunks, int32_t ppc, const int32_t* offsets, const int32_t* chunks,
                               int32_t n_ns, int64_t n_entries, int32_t P, int64_t next_free, int64_t first_new,
                               int64_t moved, void* ws, hipStream_t stream);

// Association-aware relocation: workspace layout and the two launch
// phases (the plan leaves {moved chunks, groups} in totals_host and
// synchronises `stream`).
struct ColocLayout {
  size_t owner, klist, cnt, kbase, bsum, counter, totals, bytes;
};
ColocLayout coloc_layout(int64_t m, int32_t k, int64_t n_chunks);
hipError_t launch_coloc_plan(const ColocLayout& L, const int32_t* ids, const float* scores, int64_t m, int32_t k,
                             double tau, int32_t min_group, int64_t n_chunks, void* ws, int64_t* totals_host,
                             hipStream_t stream);
hipError_t launch_coloc_move(const ColocLayout& L, void* pool, int64_t n_pages, int64_t page_bytes, int32_t* table,
                             int32_t ppc, int64_t m, int32_t k, int64_t next_free, int64_t moved, void* ws,
                             hipStream_t stream);

hipError_t launch_append(void* bank, int64_t bank_stride, int64_t n0, const void* new_emb, int64_t new_stride,
                         int64_t m, int32_t d, int32_t elem_bytes, int32_t* table, int32_t ppc, int64_t first_page,
                         hipStream_t stream);

}  // namespace memattn
