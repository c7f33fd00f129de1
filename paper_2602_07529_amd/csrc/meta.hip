// dag_meta_sizes / dag_build_meta: node table + ancestor bitsets -> per-token node ids, adaptive
// position ids (paper section 4.2), per-node visibility sets (Eq. 3 in ancestor-closure form),
// tile-level block map (dense + CSR), launch order, visible-pair counts.  Integer work only.
#include <string.h>

#include <type_traits>
#include <vector>

#include "common.h"

namespace {

struct SeqDims {
  int64_t tokens, qtiles, ktiles;
};

// Host: sums and validation of the counts.  Returns DAG_OK or an error.
int host_dims(const dag_desc_t* d, std::vector<SeqDims>* per_seq, dag_meta_sizes_t* out) {
  if (!d || !out) return DAG_ERR_NULL;
  if (d->n_seqs < 0) return DAG_ERR_BAD_LEN;
  if (d->tile_m < 1 || d->tile_n < 1 || d->tile_m > 1024 || d->tile_n > 1024) return DAG_ERR_UNSUPPORTED;
  if (d->words_per_node < 1) return DAG_ERR_BAD_LEN;
  dag_meta_sizes_t s = {};
  if (d->n_seqs > 0 && (!d->node_offsets || !d->node_len || !d->anc_bits)) return DAG_ERR_NULL;
  if (d->n_seqs > 0 && d->node_offsets[0] != 0) return DAG_ERR_BAD_LEN;
  int64_t max_nodes = 0;
  for (int b = 0; b < d->n_seqs; ++b) {
    int64_t n0 = d->node_offsets[b], n1 = d->node_offsets[b + 1];
    if (n1 < n0) return DAG_ERR_BAD_LEN;
    if (n1 - n0 > max_nodes) max_nodes = n1 - n0;
    int64_t T = 0;
    for (int64_t v = n0; v < n1; ++v) {
      if (d->node_len[v] < 1) return DAG_ERR_BAD_LEN;
      T += d->node_len[v];
    }
    if (T > INT32_MAX) return DAG_ERR_POS_OVERFLOW;
    SeqDims sd;
    sd.tokens = T;
    sd.qtiles = dag_ceil_div(T, d->tile_m);
    sd.ktiles = dag_ceil_div(T, d->tile_n);
    if (per_seq) per_seq->push_back(sd);
    s.total_tokens += T;
    s.total_qtiles += sd.qtiles;
    s.total_ktiles += sd.ktiles;
    s.total_tiles += sd.qtiles * sd.ktiles;
    for (int64_t a = 0; a < sd.qtiles; ++a) {
      int64_t last_row = (a + 1) * d->tile_m < T ? (a + 1) * d->tile_m : T;
      s.csr_capacity += (last_row - 1) / d->tile_n + 1;  // key tiles that start at or before the last row
    }
  }
  s.csr_capacity += 8;  // spare entries: the prefill kernel reads the column list eight entries at a time
  if (s.total_tokens > INT32_MAX || s.total_qtiles > INT32_MAX || s.csr_capacity > INT32_MAX)
    return DAG_ERR_POS_OVERFLOW;
  if (d->n_seqs > 0) s.total_nodes = d->node_offsets[d->n_seqs];
  if (max_nodes > (int64_t)d->words_per_node * 64) return DAG_ERR_BAD_LEN;
  if (max_nodes > 16384) return DAG_ERR_UNSUPPORTED;  // per-sequence node table is kept in LDS
  size_t ws = 0;
  ws += dag_align_up((size_t)(d->n_seqs + 1) * 4, 16);
  ws += dag_align_up((size_t)s.total_nodes * 4, 16);
  ws += dag_align_up((size_t)s.total_nodes * d->words_per_node * 8, 16);
  ws += dag_align_up((size_t)(s.total_qtiles + 1) * 4, 16);
  s.workspace_bytes = (int64_t)ws + 16;
  *out = s;
  return DAG_OK;
}

int host_validate_bits(const dag_desc_t* d) {
  const int W = d->words_per_node;
  for (int b = 0; b < d->n_seqs; ++b) {
    const int64_t n0 = d->node_offsets[b];
    const int n = d->node_offsets[b + 1] - d->node_offsets[b];
    for (int v = 0; v < n; ++v) {
      const uint64_t* row = d->anc_bits + (n0 + v) * W;
      // bits above v must be clear; the self bit is ignored
      for (int w = 0; w < W; ++w) {
        uint64_t allowed;
        int lo = w * 64;
        if (v < lo) allowed = 0;
        else if (v >= lo + 63) allowed = ~0ull;
        else allowed = (2ull << (v - lo)) - 1;  // bits 0..v-lo (includes the self bit)
        if (row[w] & ~allowed) return DAG_ERR_NOT_TOPOLOGICAL;
      }
      if (d->flags & DAG_STRICT_CLOSURE) {
        for (int u = 0; u < v; ++u) {
          if (!((row[u >> 6] >> (u & 63)) & 1)) continue;
          const uint64_t* ru = d->anc_bits + (n0 + u) * W;
          for (int w = 0; w < W; ++w) {
            uint64_t need = ru[w];
            if ((u >> 6) == w) need &= ~(1ull << (u & 63));  // u's own self bit does not count
            if (need & ~row[w]) return DAG_ERR_NOT_CLOSED;
          }
        }
      }
    }
  }
  return DAG_OK;
}

// ------------------------------------------------------------------------------------ kernels
// A node table of at most kArgWords words travels as a kernel argument: three copies from pageable memory
// cost 3 to 5 us of the stream each, an argument nothing.  (The limit keeps the arguments under 4 KB.)
// Words: node_offsets [n_seqs + 1], padded to an even count, then ancestor bitsets, then lengths.
constexpr int kArgWords = 896;
struct NodeTable {
  uint32_t w[kArgWords];
};
struct NoTable {};

struct MetaOut {  // what the kernels write, see dag_meta_t
  int32_t *cu_seqlens, *node_start, *qtile_start, *ktile_start;
  int64_t* block_map_off;
  int32_t *tok_node, *pos_ids, *node_tok_start, *node_pos_start;
  uint64_t* node_vis;
  uint8_t* block_map;
  int32_t *rowptr, *col;
  uint8_t* flag;
  int32_t *nfull, *order, *desc;
  int64_t* useful_pairs;
};

// Whole block: per-sequence token counts and the prefix sums over sequences, a wave per sequence, then a scan
// over 64 sequences at a time.
__device__ __forceinline__ void seq_sums(int n_seqs, const int32_t* node_off, const int32_t* node_len, int tile_m, int tile_n,
                                         int32_t* cu_seqlens, int32_t* qtile_start, int64_t* block_map_off,
                                         int32_t* node_start, int32_t* ktile_start) {
  const int lane = threadIdx.x & 63;
  for (int b = threadIdx.x; b <= n_seqs; b += blockDim.x) node_start[b] = node_off[b];
  for (int b = threadIdx.x >> 6; b < n_seqs; b += blockDim.x >> 6) {
    int t = 0;
    for (int v = node_off[b] + lane; v < node_off[b + 1]; v += 64) t += node_len[v];
    t = dag_wave_sum(t);
    if (lane == 0) cu_seqlens[b + 1] = t;  // turned into a prefix sum below
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  int cu = 0, qs = 0, ks = 0;
  int64_t mo = 0;
  if (lane == 0) {
    cu_seqlens[0] = 0;
    qtile_start[0] = 0;
    ktile_start[0] = 0;
    block_map_off[0] = 0;
  }
  for (int b0 = 0; b0 < n_seqs; b0 += 64) {
    const int b = b0 + lane;
    int t = b < n_seqs ? cu_seqlens[b + 1] : 0;
    int qt = (t + tile_m - 1) / tile_m, kt = (t + tile_n - 1) / tile_n;
    int64_t m = (int64_t)qt * kt;
    t = dag_wave_scan(t);
    qt = dag_wave_scan(qt);
    kt = dag_wave_scan(kt);
    m = dag_wave_scan(m);
    if (b < n_seqs) {
      cu_seqlens[b + 1] = cu + t;
      qtile_start[b + 1] = qs + qt;
      ktile_start[b + 1] = ks + kt;
      block_map_off[b + 1] = mo + m;
    }
    cu += __builtin_amdgcn_readlane(t, 63);
    qs += __builtin_amdgcn_readlane(qt, 63);
    ks += __builtin_amdgcn_readlane(kt, 63);
    mo += dag_readlane(m, 63);
  }
}

// Adaptive positions of one sequence (section 4.2: 0 without ancestors, else one past the largest ancestor
// position), token starts of its nodes and the number of visible pairs; one wave.  A lane holds node c + lane
// and what its ancestors in front have told it so far; the 64 nodes of a step are settled in order, each
// passing its last position and length on to the lanes that have it as an ancestor.  (Gathering at
// every node with a reduction over the lanes took 0.6 us a node: k_seq_node 41 us for 8 sequences of 64
// nodes, 9 us this way.)
__device__ __forceinline__ int64_t node_walk(int n, int W, const int32_t* len, const uint64_t* anc, int32_t* pos_end,
                                             int32_t* tok_start, int32_t* pos_start) {
  const int lane = threadIdx.x & 63;
  int run = 0;
  int64_t pairs = 0;
  for (int c = 0; c < n; c += 64) {
    const int v = c + lane;
    const int x = v < n ? len[v] : 0;
    const int incl = dag_wave_scan(x);
    if (v < n) tok_start[v] = run + incl - x;
    run += __builtin_amdgcn_readlane(incl, 63);
    int best = -1;  // largest ancestor end position seen so far
    long long tokens = 0;
    for (int w = 0; w < c / 64; ++w) {
      const uint64_t bits = v < n ? anc[(size_t)v * W + w] : 0;
      for (int j = 0; j < 64; ++j) {
        const int e = pos_end[w * 64 + j], l = len[w * 64 + j];
        const bool yes = (bits >> j) & 1;
        best = yes && e > best ? e : best;
        tokens += yes ? l : 0;
      }
    }
    const uint64_t own = v < n ? anc[(size_t)v * W + c / 64] & ((1ull << lane) - 1) : 0;
    const int m = min(64, n - c);
    for (int j = 0; j < m; ++j) {
      const int l = __builtin_amdgcn_readlane(x, j), e = __builtin_amdgcn_readlane(best, j) + l;
      const bool yes = (own >> j) & 1;
      best = yes && e > best ? e : best;
      tokens += yes ? l : 0;
    }
    if (v < n) {
      pos_start[v] = best + 1;
      pos_end[v] = best + x;
      pairs += (int64_t)x * tokens + (int64_t)x * (x + 1) / 2;
    }
    __threadfence_block();
  }
  return dag_wave_sum(pairs);
}

// Visible pairs among the rows i0 .. i1 - 1 and keys j0 .. j1 - 1 of a sequence => SKIP / PARTIAL / FULL.
// The pairs of nodes are shared by `lanes` (a power of two) neighbouring lanes, of which this is number sub.
__device__ __forceinline__ uint8_t tile_state(int T, int n, const int32_t* tok_start, const uint64_t* vis, int W, int i0,
                                              int i1, int j0, int j1, int sub = 0, int lanes = 1) {
  if (j0 > i1 - 1) return DAG_TILE_SKIP;  // entirely in the future of every row
  // the nodes of the first and last row and key: four searches (dag_find_segment) with their loads in flight together
  const int at[4] = {i0, i1 - 1, j0, j1 - 1};
  int lo[4] = {0, 0, 0, 0}, hi[4] = {n, n, n, n};
  for (int left = n; left > 1; left = (left + 1) / 2) {
    int start[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) start[i] = tok_start[(lo[i] + hi[i]) >> 1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int mid = (lo[i] + hi[i]) >> 1;
      if (start[i] <= at[i]) lo[i] = mid; else hi[i] = mid;
    }
  }
  const int u_lo = lo[0], u_hi = lo[1], w_lo = lo[2], w_hi = lo[3];
  int allowed = 0;  // (at most 1024 x 1024)
  const int nw = w_hi - w_lo + 1;
  int u = u_lo, w = w_lo + sub;
  while (true) {
    while (w > w_hi && u <= u_hi) {
      w -= nw;
      ++u;
    }
    if (u > u_hi) break;
    const int ue = u + 1 < n ? tok_start[u + 1] : T, we = w + 1 < n ? tok_start[w + 1] : T;
    const int r0 = max(i0, tok_start[u]), r1 = min(i1, ue);
    const int c0 = max(j0, tok_start[w]), c1 = min(j1, we);
    if (w == u) {  // causal inside the node: row i sees min(i + 1, c1) - c0 keys
      const int a = max(r0, c0), e = min(r1, c1);
      if (e > a) allowed += (e - a) * ((a + 1 - c0) + (e - c0)) / 2;
      const int past = max(a, c1);
      if (r1 > past && c1 > c0) allowed += (r1 - past) * (c1 - c0);
    } else if (w < u && ((vis[(int64_t)u * W + (w >> 6)] >> (w & 63)) & 1)) {
      allowed += (r1 - r0) * (c1 - c0);
    }
    w += lanes;
  }
  if (lanes > 1) allowed = dag_wave_sum<1>(allowed);  // (in steps: the lanes of a group are neighbours)
  if (lanes > 2) allowed += (int)dag_other_group<2>((uint32_t)allowed);
  if (lanes > 4) allowed += (int)dag_other_group<4>((uint32_t)allowed);
  if (lanes > 8) allowed += (int)dag_other_group<8>((uint32_t)allowed);
  if (lanes > 16) allowed += (int)dag_other_group<16>((uint32_t)allowed);
  if (lanes > 32) allowed += (int)dag_other_group<32>((uint32_t)allowed);
  return allowed == 0 ? DAG_TILE_SKIP : allowed == (i1 - i0) * (j1 - j0) ? DAG_TILE_FULL : DAG_TILE_PARTIAL;
}

// One wave, for query tile qt, given the number of non-skip tiles of every row (cnt):
//  * CSR row start = sum of the counts in front of it, and launch slot = number of query tiles in
//    front of it in the order (tile count descending, index ascending), both from one pass over
//    cnt shared by the lanes.  The prefill kernel hands the launch list out dynamically, and with
//    the heaviest items first the workgroups finish within the duration of one of the lightest;
//  * ordered compaction of the row's non-skip tiles -- FULL tiles first (key tiles ascending),
//    then PARTIAL tiles (ascending) -- and the number of FULL tiles;
//  * the tile's launch record in its slot: everything the prefill kernel needs to start the
//    query tile, in 32 bytes {token offset of the sequence, tokens in the sequence, first row of
//    the tile, CSR row start, tiles in the row, tiles that need no mask, node offset of the
//    sequence, first key tile of the sequence}.
__device__ __forceinline__ void csr_row(int qt, int n_seqs, int total_qtiles, int tile_m, int tile_n, const int32_t* cnt,
                                        const int32_t* qtile_start, const int64_t* block_map_off, const int32_t* cu_seqlens,
                                        const int32_t* node_start, const int32_t* ktile_start, const uint8_t* block_map,
                                        const MetaOut& o) {
  const int lane = threadIdx.x & 63;
  const int mine = cnt[qt];
  int oi = 0, c0 = 0;
  for (int j = lane; j < total_qtiles; j += 64) {
    const int x = cnt[j];
    oi += (x > mine) || (x == mine && j < qt);
    c0 += j < qt ? x : 0;
  }
  oi = dag_wave_sum(oi);
  c0 = dag_wave_sum(c0);
  const int b = dag_find_segment(qtile_start, n_seqs, qt);
  const int T = cu_seqlens[b + 1] - cu_seqlens[b];
  const int KT = (T + tile_n - 1) / tile_n;
  const uint8_t* row = block_map + block_map_off[b] + (int64_t)(qt - qtile_start[b]) * KT;
  int out = c0, nf = 0, last_full = -1;
  for (int pass = 0; pass < 2; ++pass) {
    const uint8_t want = pass == 0 ? DAG_TILE_FULL : DAG_TILE_PARTIAL;
    for (int k0 = 0; k0 < KT; k0 += 64) {
      const int k = k0 + lane;
      const uint8_t f = k < KT ? row[k] : (uint8_t)DAG_TILE_SKIP;
      const uint64_t m = __ballot(f == want);
      if (f == want) {
        const int p = out + __popcll(m & ((1ull << lane) - 1));
        o.col[p] = k;
        o.flag[p] = f;
      }
      out += __popcll(m);
      if (pass == 0 && m) last_full = k0 + 63 - __builtin_clzll(m);
    }
    if (pass == 0) nf = out - c0;
  }
  if (lane != 0) return;
  o.rowptr[qt] = c0;
  if (qt == total_qtiles - 1) o.rowptr[total_qtiles] = c0 + mine;
  o.nfull[qt] = nf;
  o.order[oi] = qt;
  if (nf > 0 && (last_full + 1) * tile_n > T) --nf;  // a ragged last key tile needs the mask path
  int32_t* d = o.desc + (int64_t)oi * 8;
  d[0] = cu_seqlens[b];
  d[1] = T;
  d[2] = (qt - qtile_start[b]) * tile_m;
  d[3] = c0;
  d[4] = mine;
  d[5] = nf;
  d[6] = node_start[b];
  d[7] = ktile_start[b];
}

// One block per sequence: the tables of its nodes.  One more block (the last) does the sums over
// sequences and zeroes the per-row tile counts that k_tiles adds up.
template <typename Table>
__global__ void __launch_bounds__(256) k_seq_node(int n_seqs, Table table, const int32_t* node_off, const int32_t* node_len,
                                                  const uint64_t* anc, int W, int tile_m, int tile_n, MetaOut o,
                                                  int32_t* cnt, int total_qtiles, int anc_in_lds) {
  extern __shared__ uint64_t s_anc[];  // [n][W] ancestor words of the sequence, then int32 [n] + [n] below
  if constexpr (std::is_same<Table, NodeTable>::value) {
    __shared__ __attribute__((aligned(16))) uint32_t s_table[kArgWords];
    for (int i = threadIdx.x; i < kArgWords; i += 256) s_table[i] = table.w[i];
    __syncthreads();
    node_off = (const int32_t*)s_table;
    anc = (const uint64_t*)(s_table + ((n_seqs + 2) & ~1));
    node_len = (const int32_t*)(anc + (int64_t)node_off[n_seqs] * W);
  }
  if ((int)blockIdx.x == n_seqs) {
    for (int i = threadIdx.x; i < total_qtiles; i += 256) cnt[i] = 0;
    if (total_qtiles == 0 && threadIdx.x == 0) o.rowptr[0] = 0;
    seq_sums(n_seqs, node_off, node_len, tile_m, tile_n, o.cu_seqlens, o.qtile_start, o.block_map_off, o.node_start,
             o.ktile_start);
    return;
  }
  const int b = blockIdx.x;
  const int n0 = node_off[b], n = node_off[b + 1] - n0;
  // (the copy of the ancestor words is skipped for node tables too large for LDS; the walk below
  // then reads them from global memory)
  int32_t* s_pos_end = (int32_t*)(s_anc + (anc_in_lds ? (size_t)n * W : 0));  // [n] last position used by each node
  int32_t* s_len = s_pos_end + n;                                              // [n]
  for (int v = threadIdx.x; v < n; v += 256) s_len[v] = node_len[n0 + v];
  for (int i = threadIdx.x; i < n * W; i += 256) {
    const uint64_t bits = anc[(int64_t)n0 * W + i];
    const int v = i / W, w = i % W;
    if (anc_in_lds) s_anc[i] = bits;
    o.node_vis[(int64_t)n0 * W + i] = bits | (v >> 6 == w ? 1ull << (v & 63) : 0ull);
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const int64_t pairs = node_walk(n, W, s_len, anc_in_lds ? s_anc : anc + (int64_t)n0 * W, s_pos_end,
                                  o.node_tok_start + n0, o.node_pos_start + n0);
  if (threadIdx.x == 0) o.useful_pairs[b] = pairs;
}

// The first blocks: one thread, or LANES of them, per (query tile, key tile), its state in the block map.  Also adds up the
// non-skip tiles of every query tile's row (cnt, zeroed before): tiles are numbered row after row, so
// a block touches at most blockDim.x consecutive rows; it counts them in LDS and adds each row's
// share to cnt once.  The remaining blocks, 256 tokens each: node and position of every token.
// A thread is a chain of some fifteen loads, each of which waits for the one in front (which sequence, which nodes, do they
// see each other): with STAGED the tables of the whole batch are in LDS first, one load and a barrier, where they are small.
// A tile of short nodes is many pairs of nodes (64 of eight tokens each): LANES neighbouring threads share a tile's, up to as
// many tiles as then still fit the device at once.  70 nodes of 23 to 129 tokens 9.4 -> 5.1 us, 2 x 68 nodes of 21 to 185
// 9.9 -> 5.5 (the copies alone 9.2 and 8.6), 4 x 4608 fork-join 5.6 -> 4.8; 8 x 64 nodes of 144, one thread a tile, 11.6 -> 10.8.
constexpr int kStagedNodes = 512, kStagedSeqs = 64;
constexpr int64_t kSharedTiles = 1 << 16;
template <bool STAGED, int LANES>
__global__ void __launch_bounds__(256) k_tiles(int n_seqs, int64_t total_tiles, int tile_blocks, int total_tokens, int W,
                                               int tile_m, int tile_n, MetaOut o, int32_t* cnt, int total_nodes) {
  __shared__ int32_t s_tok[STAGED ? kStagedNodes : 1], s_cu[STAGED ? kStagedSeqs + 1 : 1], s_node[STAGED ? kStagedSeqs + 1 : 1];
  __shared__ int32_t s_qs[STAGED ? kStagedSeqs + 1 : 1];
  __shared__ int64_t s_off[STAGED ? kStagedSeqs + 1 : 1];
  __shared__ uint64_t s_vis[STAGED ? 2 * kStagedNodes : 1];
  const bool tokens = (int)blockIdx.x >= tile_blocks;
  if constexpr (STAGED) {
    for (int i = threadIdx.x; i < total_nodes; i += 256) s_tok[i] = o.node_tok_start[i];
    if (!tokens)
      for (int i = threadIdx.x; i < total_nodes * W; i += 256) s_vis[i] = o.node_vis[i];
    if ((int)threadIdx.x <= n_seqs) {
      s_cu[threadIdx.x] = o.cu_seqlens[threadIdx.x];
      s_node[threadIdx.x] = o.node_start[threadIdx.x];
      s_qs[threadIdx.x] = o.qtile_start[threadIdx.x];
      s_off[threadIdx.x] = o.block_map_off[threadIdx.x];
    }
    __syncthreads();
  }
  const int32_t* const tok_start = STAGED ? s_tok : o.node_tok_start;
  const int32_t* const cu_seqlens = STAGED ? s_cu : o.cu_seqlens;
  const int32_t* const node_start = STAGED ? s_node : o.node_start;
  const int32_t* const qtile_start = STAGED ? s_qs : o.qtile_start;
  const int64_t* const block_map_off = STAGED ? s_off : o.block_map_off;
  const uint64_t* const vis = STAGED ? s_vis : o.node_vis;
  if (tokens) {
    const int t = (blockIdx.x - tile_blocks) * 256 + threadIdx.x;
    if (t < total_tokens) {
      const int b = dag_find_segment(cu_seqlens, n_seqs, t);
      const int n0 = node_start[b], i = t - cu_seqlens[b];
      const int v = dag_find_segment(tok_start + n0, node_start[b + 1] - n0, i);
      o.tok_node[t] = v;
      o.pos_ids[t] = o.node_pos_start[n0 + v] + i - tok_start[n0 + v];
    }
    return;
  }
  __shared__ int s_rows[256];
  __shared__ int s_first;
  s_rows[threadIdx.x] = 0;
  const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) / LANES;
  const int sub = threadIdx.x % LANES;
  int gq = 0;  // query tile (row of the block map) over the whole batch
  uint8_t state = DAG_TILE_SKIP;
  if (idx < total_tiles) {
    const int b = dag_find_segment(block_map_off, n_seqs, idx);
    const int T = cu_seqlens[b + 1] - cu_seqlens[b];
    const int KT = (T + tile_n - 1) / tile_n;
    const int64_t loc = idx - block_map_off[b];
    const int a = (int)(loc / KT), kb = (int)(loc % KT);
    gq = qtile_start[b] + a;
    const int n0 = node_start[b];
    state = tile_state(T, node_start[b + 1] - n0, tok_start + n0, vis + (int64_t)n0 * W, W, a * tile_m,
                       min(T, (a + 1) * tile_m), kb * tile_n, min(T, (kb + 1) * tile_n), sub, LANES);
    if (sub == 0) o.block_map[idx] = state;
  }
  if (threadIdx.x == 0) s_first = gq;  // thread 0 is always valid (the grid covers total_tiles)
  __syncthreads();
  if (state != DAG_TILE_SKIP && sub == 0) atomicAdd(&s_rows[gq - s_first], 1);
  __syncthreads();
  if (s_rows[threadIdx.x] != 0) atomicAdd(cnt + s_first + threadIdx.x, s_rows[threadIdx.x]);
}

__global__ void __launch_bounds__(256) k_csr_order_desc(int n_seqs, int total_qtiles, int tile_m, int tile_n,
                                                        const int32_t* cnt, MetaOut o) {
  const int qt = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (qt >= total_qtiles) return;
  csr_row(qt, n_seqs, total_qtiles, tile_m, tile_n, cnt, o.qtile_start, o.block_map_off, o.cu_seqlens, o.node_start,
          o.ktile_start, o.block_map, o);
}

// Small batches: everything above in one workgroup, the intermediate tables in LDS.  Three copies and four
// launches are all latency there: 8 nodes of 600 tokens took 30 us, this kernel takes 8.  At its limits it
// is still the faster one (8 / 64 nodes, 2048 tokens: 10 / 16 us, the launches above 14 / 19 us); with twice
// the rows it was not (19 against 14 us), a wave taking four rows of the CSR one after another.
constexpr int kSmallTiles = 1024, kSmallRows = 32, kSmallTokens = 2048, kSmallSeqs = 64;
__global__ void __launch_bounds__(1024) k_meta_small(int n_seqs, NodeTable table, int W, int tile_m, int tile_n, MetaOut o,
                                                     int total_tiles, int total_qtiles, int total_tokens) {
  __shared__ __attribute__((aligned(16))) uint32_t s_table[kArgWords];
  __shared__ int32_t s_tok[kArgWords / 3], s_pos[kArgWords / 3], s_end[kArgWords / 3];
  __shared__ int32_t s_cu[kSmallSeqs + 1], s_node[kSmallSeqs + 1], s_qs[kSmallSeqs + 1], s_ks[kSmallSeqs + 1];
  __shared__ int64_t s_mo[kSmallSeqs + 1];
  __shared__ int s_cnt[kSmallRows];
  __shared__ uint8_t s_map[kSmallTiles];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < kArgWords) s_table[tid] = table.w[tid];
  if (tid < kSmallRows) s_cnt[tid] = 0;
  __syncthreads();
  const int32_t* off = (const int32_t*)s_table;
  uint64_t* anc = (uint64_t*)(s_table + ((n_seqs + 2) & ~1));
  const int32_t* len = (const int32_t*)(anc + (int64_t)off[n_seqs] * W);
  const int nodes = off[n_seqs];
  for (int b = wave; b < n_seqs; b += 16) {
    const int n0 = off[b];
    const int64_t pairs = node_walk(off[b + 1] - n0, W, len + n0, anc + (int64_t)n0 * W, s_end + n0, s_tok + n0, s_pos + n0);
    if (lane == 0) o.useful_pairs[b] = pairs;
  }
  seq_sums(n_seqs, off, len, tile_m, tile_n, s_cu, s_qs, s_mo, s_node, s_ks);  // (its barrier is also the walk's)
  for (int b = wave; b < n_seqs; b += 16)  // a node sees itself
    for (int v = lane; v < off[b + 1] - off[b]; v += 64) anc[(int64_t)(off[b] + v) * W + (v >> 6)] |= 1ull << (v & 63);
  __syncthreads();
  for (int b = tid; b <= n_seqs; b += 1024) {
    o.cu_seqlens[b] = s_cu[b];
    o.node_start[b] = s_node[b];
    o.qtile_start[b] = s_qs[b];
    o.ktile_start[b] = s_ks[b];
    o.block_map_off[b] = s_mo[b];
  }
  for (int i = tid; i < nodes * W; i += 1024) o.node_vis[i] = anc[i];
  for (int v = tid; v < nodes; v += 1024) {
    o.node_tok_start[v] = s_tok[v];
    o.node_pos_start[v] = s_pos[v];
  }
  int shift = 0;  // 1 << shift lanes of a tile: few tiles with many short nodes are shared by several lanes
  while (shift < 6 && total_tiles << (shift + 1) <= 1024) ++shift;
  const int lanes = 1 << shift, sub = tid & (lanes - 1);
  for (int idx = tid >> shift; idx < total_tiles; idx += 1024 >> shift) {
    const int b = dag_find_segment(s_mo, n_seqs, (int64_t)idx);
    const int T = s_cu[b + 1] - s_cu[b], KT = (T + tile_n - 1) / tile_n, loc = idx - (int)s_mo[b];
    const int a = loc / KT, kb = loc % KT, n0 = s_node[b];
    const uint8_t state = tile_state(T, s_node[b + 1] - n0, s_tok + n0, anc + (int64_t)n0 * W, W, a * tile_m,
                                     min(T, (a + 1) * tile_m), kb * tile_n, min(T, (kb + 1) * tile_n), sub, lanes);
    if (sub != 0) continue;
    s_map[idx] = state;
    o.block_map[idx] = state;
    if (state != DAG_TILE_SKIP) atomicAdd(&s_cnt[s_qs[b] + a], 1);
  }
  for (int t = tid; t < total_tokens; t += 1024) {
    const int b = dag_find_segment(s_cu, n_seqs, t);
    const int n0 = s_node[b], i = t - s_cu[b];
    const int v = dag_find_segment(s_tok + n0, s_node[b + 1] - n0, i);
    o.tok_node[t] = v;
    o.pos_ids[t] = s_pos[n0 + v] + i - s_tok[n0 + v];
  }
  __syncthreads();
  for (int qt = wave; qt < total_qtiles; qt += 16)
    csr_row(qt, n_seqs, total_qtiles, tile_m, tile_n, s_cnt, s_qs, s_mo, s_cu, s_node, s_ks, s_map, o);
}

}  // namespace

extern "C" int dag_prefill_tile_shape(int32_t hq, int32_t hkv, int32_t head_dim, dag_dtype_t dtype,
                                      int32_t* tile_m, int32_t* tile_n) {
  if (!tile_m || !tile_n) return DAG_ERR_NULL;
  if (hq < 1 || hkv < 1 || hq % hkv != 0) return DAG_ERR_UNSUPPORTED;
  if (head_dim != 64 && head_dim != 128) return DAG_ERR_UNSUPPORTED;
  if (dtype == DAG_F32) {
    *tile_m = 64;
    *tile_n = 64;
    return DAG_OK;
  }
  if (dtype != DAG_BF16) return DAG_ERR_UNSUPPORTED;
  // The block map is 64 x 64 for every head configuration: four-head items work on 64 query rows,
  // and the 256-row tiles of left-over heads are derived from four rows of this map.
  *tile_m = 64;
  *tile_n = 64;
  return DAG_OK;
}

extern "C" int dag_meta_sizes(const dag_desc_t* desc, dag_meta_sizes_t* out) {
  return host_dims(desc, nullptr, out);
}

extern "C" int dag_build_meta(const dag_desc_t* d, const dag_meta_t* m, void* ws, size_t ws_bytes,
                              void* stream_) {
  if (!d || !m) return DAG_ERR_NULL;
  dag_meta_sizes_t s;
  int rc = host_dims(d, nullptr, &s);
  if (rc != DAG_OK) return rc;
  if (m->n_seqs != d->n_seqs || m->words_per_node != d->words_per_node || m->tile_m != d->tile_m ||
      m->tile_n != d->tile_n || m->sizes.total_tokens != s.total_tokens ||
      m->sizes.total_qtiles != s.total_qtiles || m->sizes.total_tiles != s.total_tiles ||
      m->sizes.csr_capacity != s.csr_capacity || m->sizes.total_nodes != s.total_nodes)
    return DAG_ERR_BAD_LEN;
  if (d->n_seqs == 0) return DAG_OK;
  if (!m->cu_seqlens || !m->node_start || !m->qtile_start || !m->ktile_start || !m->block_map_off ||
      !m->qtile_rowptr || !m->useful_pairs)
    return DAG_ERR_NULL;
  if (s.total_tokens > 0 && (!m->tok_node || !m->pos_ids || !m->node_tok_start || !m->node_pos_start ||
                             !m->node_vis || !m->block_map || !m->qtile_col || !m->qtile_flag || !m->qtile_nfull || !m->qtile_order || !m->qtile_desc))
    return DAG_ERR_NULL;
  rc = host_validate_bits(d);
  if (rc != DAG_OK) return rc;
  if (!ws || ws_bytes < (size_t)s.workspace_bytes) return DAG_ERR_WORKSPACE;

  hipStream_t stream = (hipStream_t)stream_;
  const int W = d->words_per_node;
  const MetaOut o = {m->cu_seqlens, m->node_start, m->qtile_start, m->ktile_start, m->block_map_off, m->tok_node,
                     m->pos_ids, m->node_tok_start, m->node_pos_start, m->node_vis, m->block_map, m->qtile_rowptr,
                     m->qtile_col, m->qtile_flag, m->qtile_nfull, m->qtile_order, m->qtile_desc, m->useful_pairs};
  const int QT = (int)s.total_qtiles;
  // A capturing stream records the copies: its replays read the caller's arrays anew.
  hipStreamCaptureStatus capture = hipStreamCaptureStatusActive;
  const size_t words = (size_t)((d->n_seqs + 2) & ~1) + (size_t)s.total_nodes * (2 * W + 1);
  const bool as_arg = words <= kArgWords && hipStreamIsCapturing(stream, &capture) == hipSuccess &&
                      capture == hipStreamCaptureStatusNone;
  NodeTable table;
  if (as_arg) {
    uint32_t* w = table.w;
    memcpy(w, d->node_offsets, (size_t)(d->n_seqs + 1) * 4);
    w += (d->n_seqs + 2) & ~1;
    if (s.total_nodes > 0) {
      memcpy(w, d->anc_bits, (size_t)s.total_nodes * W * 8);
      memcpy(w + s.total_nodes * W * 2, d->node_len, (size_t)s.total_nodes * 4);
    }
    memset(table.w + words, 0, (kArgWords - words) * 4);
    if (s.total_tokens > 0 && s.total_tokens <= kSmallTokens && s.total_tiles <= kSmallTiles && QT <= kSmallRows &&
        d->n_seqs <= kSmallSeqs) {
      hipLaunchKernelGGL(k_meta_small, dim3(1), dim3(1024), 0, stream, d->n_seqs, table, W, d->tile_m, d->tile_n, o,
                         (int)s.total_tiles, QT, (int)s.total_tokens);
      DAG_LAUNCH_CHECK();
      return DAG_OK;
    }
  }
  char* p = (char*)dag_align_up((size_t)(uintptr_t)ws, 16);
  int32_t* d_off = (int32_t*)p;
  p += dag_align_up((size_t)(d->n_seqs + 1) * 4, 16);
  int32_t* d_len = (int32_t*)p;
  p += dag_align_up((size_t)s.total_nodes * 4, 16);
  uint64_t* d_anc = (uint64_t*)p;
  p += dag_align_up((size_t)s.total_nodes * W * 8, 16);
  int32_t* d_cnt = (int32_t*)p;
  int max_nodes = 0;
  for (int b = 0; b < d->n_seqs; ++b) {
    int n = d->node_offsets[b + 1] - d->node_offsets[b];
    if (n > max_nodes) max_nodes = n;
  }
  const size_t anc_bytes = (size_t)max_nodes * W * 8;
  const int anc_in_lds = anc_bytes <= 32768;
  const size_t lds = (size_t)max_nodes * 8 + 8 + (anc_in_lds ? anc_bytes : 0);
  if (as_arg) {
    hipLaunchKernelGGL(k_seq_node<NodeTable>, dim3(d->n_seqs + 1), dim3(256), lds, stream, d->n_seqs, table, nullptr,
                       nullptr, nullptr, W, d->tile_m, d->tile_n, o, d_cnt, QT, anc_in_lds);
  } else {
    DAG_HIP_CHECK(hipMemcpyAsync(d_off, d->node_offsets, (size_t)(d->n_seqs + 1) * 4, hipMemcpyHostToDevice, stream));
    if (s.total_nodes > 0) {
      DAG_HIP_CHECK(hipMemcpyAsync(d_len, d->node_len, (size_t)s.total_nodes * 4, hipMemcpyHostToDevice, stream));
      DAG_HIP_CHECK(hipMemcpyAsync(d_anc, d->anc_bits, (size_t)s.total_nodes * W * 8, hipMemcpyHostToDevice, stream));
    }
    hipLaunchKernelGGL(k_seq_node<NoTable>, dim3(d->n_seqs + 1), dim3(256), lds, stream, d->n_seqs, NoTable{}, d_off, d_len,
                       d_anc, W, d->tile_m, d->tile_n, o, d_cnt, QT, anc_in_lds);
  }
  DAG_LAUNCH_CHECK();
  if (s.total_tokens == 0) return DAG_OK;
  const bool shared = s.total_tiles <= kSharedTiles;
  const int64_t tile_blocks = dag_ceil_div(s.total_tiles * (shared ? 4 : 1), 256);
  const bool staged = s.total_nodes <= kStagedNodes && d->n_seqs <= kStagedSeqs && W <= 2;
  auto* const tiles = staged ? (shared ? k_tiles<true, 4> : k_tiles<true, 1>) : shared ? k_tiles<false, 4> : k_tiles<false, 1>;
  hipLaunchKernelGGL(tiles, dim3((unsigned)(tile_blocks + dag_ceil_div(s.total_tokens, 256))), dim3(256), 0, stream,
                     d->n_seqs, s.total_tiles, (int)tile_blocks, (int)s.total_tokens, W, d->tile_m, d->tile_n, o, d_cnt, (int)s.total_nodes);
  DAG_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_csr_order_desc, dim3((unsigned)((QT + 3) / 4)), dim3(256), 0, stream, d->n_seqs, QT, d->tile_m,
                     d->tile_n, d_cnt, o);
  DAG_LAUNCH_CHECK();
  return DAG_OK;
}
