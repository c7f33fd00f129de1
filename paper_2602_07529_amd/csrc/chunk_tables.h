// Device code of the tables of query chunks, for the kernels that build them in front of the forward and the backward (internal).
#pragma once
#include "prefill_launch.h"

namespace {

constexpr int CHUNK_KEYS = 64;  // keys of a tile

// Launch order of the 256-row tiles: by descending tile count (ties: ascending index), as for the
// 64-row ones; also counts them.  One wave per 64-row tile.
__device__ __forceinline__ void wide_order(int qt, int total_qtiles, const int32_t* wide_cnt, const int32_t* wide_pre,
                                           int32_t* wide_desc, int32_t* wide_count) {
  const int lane = threadIdx.x & 63;
  const int mine = wide_cnt[qt];
  if (mine < 0 && qt != 0) return;
  int oi = 0, n = 0;
  for (int j = lane; j < total_qtiles; j += 64) {
    const int o = wide_cnt[j];
    oi += (o > mine) || (o == mine && j < qt);
    n += o >= 0;
  }
  oi = dag_wave_sum(oi);
  n = dag_wave_sum(n);
  if (mine >= 0 && lane < 8) wide_desc[(int64_t)oi * 8 + lane] = wide_pre[(int64_t)qt * 8 + lane];
  if (qt == 0 && lane == 0) *wide_count = n;
}

// Query chunks.  Consecutive nodes with the same ancestors (the siblings of a fork; most often a single
// node) form a group, and the query rows are cut at the borders of the groups instead of every 64
// tokens.  All rows of a chunk then see the same tokens in front of the group, the ancestors', and
// of the group itself every row the tokens of its own node up to itself.  So with the visible keys in
// one list -- the ancestors' tokens, then the tokens from the start of the chunk's first node u on --
// row i (counted from u's first token) sees the positions < A (A: tokens of the ancestors) and A + (its
// node's first row) .. A + i.  The keys of a chunk stream in that order, whatever tiles of the sequence
// they lie in: every key tile is full, only the last one or two take a mask, and nothing
// invisible is computed but there.  The list is a few runs of consecutive tokens (neighbouring visible
// nodes are one run), kept per node u as {first position, token - position}.
// One wave per node (at most 128 per sequence, so at most 64 runs): its runs, and for the first node of a
// group the descriptors of its chunks.
template <int W>
__device__ __forceinline__ void node_rows(int gv, int n_seqs, int total_nodes, int rows, int64_t n_slots,
                                          const int32_t* __restrict__ node_start,
                                          const int32_t* __restrict__ cu_seqlens,
                                          const int32_t* __restrict__ tok_node,
                                          const int32_t* __restrict__ node_tok_start,
                                          const uint64_t* __restrict__ node_vis,
                                          int32_t* __restrict__ runs, const ChunkTables& t) {
  const int lane = threadIdx.x & 63;
  const int b = dag_find_segment(node_start, n_seqs, gv);
  const int n0 = node_start[b], n = node_start[b + 1] - n0, v = gv - n0;
  const int cu = cu_seqlens[b], T = cu_seqlens[b + 1] - cu;
  const uint64_t below = (1ull << lane) - 1;
  uint64_t mine[W], sees[W], same[W];  // the node's ancestors; with the node itself; nodes with the same ancestors
#pragma unroll
  for (int y = 0; y < W; ++y) {
    const int bit = v - 64 * y;
    mine[y] = node_vis[(int64_t)gv * W + y] & (bit >= 64 ? ~0ull : bit <= 0 ? 0ull : (1ull << bit) - 1);
    sees[y] = mine[y] | (bit >= 0 && bit < 64 ? 1ull << bit : 0ull);
  }
  int2* const out = (int2*)runs + (int64_t)gv * 64;
  int before = 0, n_runs = 0, anc = 0;  // tokens and runs of the words in front; tokens of the ancestors
#pragma unroll
  for (int x = 0; x < W; ++x) {
    const int u = 64 * x + lane;
    const int first = u < n ? node_tok_start[n0 + u] : T, len = (u + 1 < n ? node_tok_start[n0 + u + 1] : T) - first;
    const int seen = (sees[x] >> lane) & 1 ? len : 0;
    const int incl = dag_wave_scan(seen);
    const int pos = before + incl - seen;
    before += __builtin_amdgcn_readlane(incl, 63);
    if (v / 64 == x) anc = __builtin_amdgcn_readlane(pos, v % 64);
    const uint64_t starts = sees[x] & ~(sees[x] << 1 | (x > 0 ? sees[x > 0 ? x - 1 : 0] >> 63 : 0));  // a run starts where the node in front is not visible
    if (runs && (starts >> lane) & 1) out[n_runs + __popcll(starts & below)] = int2{pos, cu + first - pos};
    n_runs += __popcll(starts);
    bool eq = u < n;
#pragma unroll
    for (int y = 0; y < W; ++y) {
      const uint64_t theirs = u < n ? node_vis[(int64_t)(n0 + u) * W + y] & (y < x ? ~0ull : y == x ? below : 0ull) : 0;
      eq = eq && theirs == mine[y];
    }
    same[x] = __ballot(eq);
  }
  if (runs && lane >= n_runs) out[lane] = int2{INT32_MAX, 0};
  auto is_same = [&](int u) { return ((W > 1 && u >= 64 ? same[W - 1] : same[0]) >> (u & 63)) & 1; };
  if (v > 0 && is_same(v - 1)) return;  // the first node of the group writes its chunks
  int end = v + 1;                      // first node behind the group
  while (end < n && is_same(end)) ++end;
  const int g0 = node_tok_start[gv], g1 = end < n ? node_tok_start[n0 + end] : T;
  const int64_t slot0 = (cu + g0) / rows + gv, gend = n0 + end;
  const int64_t slot1 = gend < total_nodes ? (int64_t)(cu + g1) / rows + gend : n_slots;
  for (int c = lane; slot0 + c < slot1; c += 64) {
    if (c * rows >= g1 - g0) {
      t.cnt[slot0 + c] = -1;
      continue;
    }
    const int u = tok_node[cu + g0 + c * rows];  // node of the chunk's first row
    const int u0 = node_tok_start[n0 + u], u1 = u + 1 < n ? node_tok_start[n0 + u + 1] : T;
    const int row0 = g0 + c * rows - u0, row_end = min(row0 + rows, g1 - u0);  // counted from u's first token
    int32_t* d = t.pre + (slot0 + c) * 8;
    t.cnt[slot0 + c] = (anc + row_end + CHUNK_KEYS - 1) / CHUNK_KEYS;
    d[0] = cu + u0;
    d[1] = g1 - u0;
    d[2] = row0;
    d[3] = (n0 + u) * 64;
    d[4] = (anc + row_end + CHUNK_KEYS - 1) / CHUNK_KEYS;
    d[5] = (row_end <= u1 - u0 ? anc + row0 + 1 : anc) / CHUNK_KEYS;  // tiles whose 64 positions every row sees
    d[6] = anc;
    d[7] = 0;
  }
}

// Tokens of its own node in front of a token, for as many tokens as the block has threads, from t0 on (not from the position ids: those
// are the caller's to shift).
__device__ __forceinline__ void token_depths(const PrefillArgs& a, int64_t t0) {
  const int64_t t = t0 + threadIdx.x;
  if (t < a.total_tokens) {
    const int b = dag_find_segment(a.cu_seqlens, a.n_seqs, (int)t);
    a.tok_depth[t] = (int)t - a.cu_seqlens[b] - a.node_tok_start[a.node_start[b] + a.tok_node[t]];
  }
}

// The tables of several chunk sizes are built together (bit i of `sizes`: those of DAG_CHUNK_ROWS[i] rows, the last bit those of pack_rows;
// blockIdx.y, in the small form blockIdx.x, counts the set bits).  The prefill builds all of them whatever the
// launch behind it takes: the head counts of a call may differ from those that its workspace was prepared for.
// What the sizes share by the blocks of the first one: the runs, the work counters of the attention kernel,
// the depths.
__device__ __forceinline__ int nth_size(int sizes, int n) {
  for (; n > 0; --n) sizes &= sizes - 1;
  return __builtin_ctz(sizes);
}
__device__ __forceinline__ ChunkTables tables_of(const PrefillArgs& a, int i) { return i == 0 ? a.chunk[0] : i == 1 ? a.chunk[1] : i == 2 ? a.chunk[2] : a.chunk[3]; }
__device__ __forceinline__ int rows_of(const PrefillArgs& a, int i) { return i == DAG_CHUNK_PACK ? a.pack_rows : DAG_CHUNK_ROWS[0] << i; }
__device__ __forceinline__ int slots_of(const PrefillArgs& a, int i) {  // = chunk_slots
  return (i == DAG_CHUNK_PACK ? (int)a.total_tokens / a.pack_rows : (int)(a.total_tokens >> (__builtin_ctz(DAG_CHUNK_ROWS[0]) + i))) + (int)a.total_nodes;
}

}  // namespace
