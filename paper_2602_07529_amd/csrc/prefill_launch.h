// Kernel argument block shared by the prefill kernels (internal).
#pragma once
#include "common.h"

constexpr int DAG_SCHED_INTS = 128;  // [0..63] item counters, [64] finished workgroups

// Query chunks (k_node_rows): tables of the chunks of DAG_CHUNK_ROWS[i] rows.  A slot may hold a chunk;
// the group of siblings that starts with node v (of the batch) and token t owns the slots from
// t / rows + v on.
constexpr int DAG_CHUNK_SIZES = 3;
constexpr int DAG_CHUNK_ROWS[DAG_CHUNK_SIZES] = {64, 128, 256};  // (each twice the one in front)
// A fourth size belongs to the head counts that pack all heads of a group into an item (pack_heads_of): as many rows as 32 NW
// (row, head) pairs have, at least PACK_MIN_ROWS.
constexpr int DAG_CHUNK_PACK = DAG_CHUNK_SIZES, PACK_MIN_ROWS = 16;
struct ChunkTables {
  int32_t* count;  // [3] number of chunks; (packed heads) the rows that the table was built for, 0: not built; see k_pack_tables
  int32_t* cnt;    // [slots] key tiles of the chunk, -1: no chunk here
  int32_t* pre;    // [slots][8] its descriptor
  int32_t* desc;   // [slots][8] descriptors in launch order
};
inline int64_t chunk_slots(int64_t total_tokens, int64_t total_nodes, int rows) { return total_tokens / rows + total_nodes; }

struct PrefillArgs {
  const void* q;
  const void* k;
  const void* v;
  void* out;
  float* lse;
  void* vt;  // workspace: key-tile-wise transposed V in the LDS tile order (bf16 path)
  int32_t* sched;  // workspace: work-distribution counters of the bf16 kernel, DAG_SCHED_INTS ints, zero between launches
  const int32_t* cu_seqlens;
  const int32_t* node_start;
  const int32_t* tok_node;
  const uint64_t* node_vis;
  const int32_t* qtile_start;
  const int32_t* ktile_start;
  const int32_t* rowptr;
  const int32_t* col;
  const uint8_t* flag;
  const int32_t* nfull;
  const int32_t* qtile_order;
  const int32_t* qtile_desc;  // [total_qtiles][8], see dag_meta_t
  const int64_t* block_map_off;
  const uint8_t* block_map;
  int n_seqs, W, hq, hkv;
  int64_t total_qtiles, total_ktiles;
  float scale;
  // bf16 path: the query heads of every KV head that one launch covers (set per launch)
  int head0, heads;
  const int32_t* n_tiles_dev;  // null, or where the launch reads its number of query tiles
  // bf16 path, workspace: the 256-row query tiles derived from the block map (see k_wide_rows)
  int32_t* wide_count;  // [1] number of 256-row tiles
  int32_t* wide_cnt;    // [total_qtiles] tiles in the row starting at this 64-row tile, -1: none starts here
  int32_t* wide_pre;    // [total_qtiles][8] descriptor of that row
  int32_t* wide_desc;   // [total_qtiles][8] descriptors in launch order (wide_count of them)
  int32_t* wide_col;    // [csr_capacity] key tiles of the rows, row of tile qt at rowptr[qt]
  // bf16 path, workspace: what every node sees, as runs of consecutive tokens (see k_node_rows)
  const int32_t* node_tok_start;
  int64_t total_tokens, total_nodes;
  int32_t* node_runs;  // [total_nodes][64][2], null when the workspace has no room for them
  int32_t* tok_depth;  // [total_tokens] tokens of its own node in front of every token
  ChunkTables chunk[DAG_CHUNK_SIZES + 1];
  int pack_heads, pack_rows;  // packed heads: heads of a KV head in an item and rows of a chunk; 0: not these head counts
  float* part;  // paged prefill: partial results of the pieces of its rows of tiles, null: no room for them
};

// The node tables hold 64 runs per node, the most that 128 nodes can have.  They take the place of the
// transposed V, which is not needed with them: 784 bytes a node and 10.1 a token against at least 128 a
// token, so that they fit wherever a node has seven tokens on average.
inline size_t prefill_node_table_bytes(int64_t total_tokens, int64_t total_nodes) {
  size_t n = (size_t)total_nodes * 128 * 4 + (size_t)total_tokens * 4;
  for (int i = 0; i < DAG_CHUNK_SIZES; ++i) n += (size_t)(62 + 17 * chunk_slots(total_tokens, total_nodes, DAG_CHUNK_ROWS[i])) * 4;
  return n + (size_t)(62 + 17 * chunk_slots(total_tokens, total_nodes, PACK_MIN_ROWS) + 1) * 4;
}

// Points the node tables of `a` into the memory at t (8-byte aligned, prefill_node_table_bytes of it).
inline void prefill_node_tables(PrefillArgs& a, int32_t* t) {
  a.node_runs = t;
  t += a.total_nodes * 128;
  for (int i = 0; i < DAG_CHUNK_SIZES; ++i) {
    const int64_t n = chunk_slots(a.total_tokens, a.total_nodes, DAG_CHUNK_ROWS[i]);
    a.chunk[i] = {t, t + 62, t + 62 + n, t + 62 + 9 * n};
    t += 62 + 17 * n;
  }
  a.tok_depth = t;
  t += a.total_tokens + (a.total_tokens & 1);
  const int64_t n = chunk_slots(a.total_tokens, a.total_nodes, a.pack_rows > 0 ? a.pack_rows : 256);  // (where it lies does not depend on the head count)
  a.chunk[DAG_CHUNK_PACK] = {t, t + 62, t + 62 + n, t + 62 + 9 * n};
}

constexpr int PACK_WAVES(int head_dim) { return head_dim == 128 ? 8 : 4; }  // of an item
// Query heads of a KV head that are neither one, two nor four go into an item together: the 32 NW (row, head) pairs of an item
// are row-major, every lane of a wave with a row and a head of its own, all on the same K / V tiles.  More than eight heads are
// divided evenly.  Five heads were an item of four on 64 rows and, in a launch behind it, one on 256, which random DAGs leave
// half empty: 60 nodes, 40 / 8 heads 154 -> 113 us, 5 x 53 nodes 704 -> 634, a fork-join of 17,000 tokens 7748 -> 7526; eight
// heads on 32 rows instead of twice four on 64: 921 -> 864; 56 batches of 3, 5, 6, 7 and 8 heads 1.24 times as fast.  Where all
// siblings together are a multiple of 256 tokens the rows of four heads, of pairs and of one had no chunk partly empty and these
// have: 16 x 4608 tokens, 24 / 8 heads 1860 -> 1918 us, 16 x 5120 of 48 / 8 heads 2743 -> 2849, with any other lengths 1.02 to
// 1.2 times as fast (the lengths are not known to the host).  At head dimension 64 four heads, too: four waves on 32 rows instead of eight
// on 64 leave room for two workgroups on a compute unit, 2 x 4500 tokens, 8 / 2 heads 90 -> 79 us (but see long_contexts).
inline int pack_heads_of(int g, int head_dim) {
  if (g == 1 || g == 2 || (g == 4 && head_dim == 128)) return 0;
  const int groups = (g + 7) / 8;
  return (g + groups - 1) / groups;
}

// Workspace of the bf16 path behind the transposed V: counters, then the tables above.
inline size_t prefill_bf16_table_bytes(int64_t total_qtiles, int64_t csr_capacity) {
  return (size_t)(DAG_SCHED_INTS + 64 + 17 * total_qtiles + csr_capacity) * 4;
}

// Paged prefill: the kernel argument block (q, k = K pool, vt = V pool, out, lse, sched, hq, hkv,
// scale, head0 / heads, and the five table pointers, of which wide_col holds the tile entries)
// plus what the table kernel reads.
constexpr int PAGED_MAX_ITEMS = 256;  // at most this many items (of one KV head and HG heads) are pieces
constexpr int PAGED_MAX_CUTS = 32;    // of one row of tiles
constexpr int PAGED_CUT_TILES = 24;   // shorter rows of tiles are not cut: the partial results of a full device are 34 MB, 15 us written and read
// (a piece has 256 rows of sums, with two words a row; items are at least as many as rows of tiles)
inline size_t paged_piece_bytes(int64_t slots, int64_t nt_max) {
  return slots > PAGED_MAX_ITEMS / 2 || nt_max < PAGED_CUT_TILES ? 0 : (size_t)PAGED_MAX_ITEMS * (17 * 4 + 8 * (32 * 128 + 64) * 4) + 256;
}
struct PagedPrefillArgs {
  PrefillArgs a;
  int n_nodes, max_new, nt_max, n_pages;
  int32_t* piece_tables;  // room for the count and the two descriptors of PAGED_MAX_ITEMS items, where a.part is not null
  const int32_t *q_off, *ctx_page_off, *ctx_pages, *ctx_page_len, *own_page, *own_len;
};
int launch_prefill_paged(const PagedPrefillArgs& pa, int head_dim, hipStream_t stream);

bool prefill_on_chunks(const PrefillArgs& a, int head_dim);  // bf16: query chunks or the block map's tiles
int launch_prefill_f32(const PrefillArgs& a, int head_dim, hipStream_t stream);
int launch_prefill_bf16_prepare_v(const PrefillArgs& a, int head_dim, hipStream_t stream);  // V -> workspace copy
int launch_prefill_pack_tables(const PrefillArgs& a, int head_dim, hipStream_t stream);     // for a workspace prepared for any head count
int launch_prefill_bf16(const PrefillArgs& a, int head_dim, hipStream_t stream);            // needs the copy
