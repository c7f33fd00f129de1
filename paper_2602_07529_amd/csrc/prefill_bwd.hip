// Backward of the DAG-masked prefill attention (the paper fine-tunes through the mask of Eq. 3,
// section 4.2): with P = softmax_row(scale Q K^T + M), O = P V and the incoming gradient dO,
//     delta_i = sum_d dO_id O_id,   dV = P^T dO,   dP = dO V^T,   dS = P o (dP - delta),
//     dQ = scale dS K,   dK = scale dS^T Q        (a KV head sums over its query heads).
// P is recomputed from the forward's log-sum-exp; the block map of the forward skips the tiles
// without a visible pair.  bf16 operands on the 32x32x16 MFMA, fp32 accumulation.  The kernels:
//   k_bwd_delta_tables   delta and -lse log2(e) per (token, query head), and small tables: the query chunks
//                 or the first visibility word of every token, weights of the key-tile pairs
//   k_bwd_orders  launch orders of the chunks and of the dK/dV workgroups (heaviest pairs first)
//   k_bwd_dq2     one workgroup per (64-row query tile, KV head, four of its query heads), eight
//                 waves; the K / V tiles of the tile's row of the forward's FULL-first CSR stream
//                 through an LDS ring and every tile is a fixed sequence of 48 slots (described at
//                 the kernel).  The heads that the groups of four leave over (G not a multiple of
//                 four) run as k_bwd_dq2<true>: one head on four consecutive query tiles per
//                 workgroup, with tile lists from bwd_wide_rows
//   k_bwd_dkv2    one workgroup per (pair of 64-key tiles, KV head), four waves; the Q / dO tiles of
//                 the query tiles that see the pair stream through an LDS ring, one (tile, query
//                 head) = 64 slots (described at the kernel); nothing is accumulated through
//                 atomics, so the results do not depend on the order of execution
//   k_bwd64_dq, k_bwd64_dkv   the same two for head dimension 64
//   k_nodes_dq2, k_nodes64_dq   dQ on the forward's query chunks instead of the block map's tiles, all heads of a group in one item
//   k_nodes_dkv2, k_nodes64_dkv   dK/dV with the query rows that see the keys as one compact stream, the
//                 keys in blocks cut at node borders (cut_keys);
//                 k_dkv_finish behind them for streams in pieces and for keys that a
//                 hidden Inf or NaN has reached
//   k_bwd_dq, k_bwd_dkv   the first versions (tiles staged through registers, compiler-scheduled),
//                 reached by a development switch only
// Register layout of a 32x32 MFMA result C = A B:  lane (L, H) = (lane % 32, lane / 32) holds
// column L and the 16 rows rho_H(e) = 8 (e / 4) + 4 H + e % 4.  A result is used again as the B
// operand of the next product (contraction over its rows) straight from the registers; the A
// operand of that product is then gathered from LDS in the same row order.
// Those A operands are transposed tiles (K^T for dQ; Q^T and dO^T for dK and dV): they are read
// from the row-major tiles in LDS with the transposing LDS load of gfx950, two 8-byte reads per
// operand, in the row order rho asks for.
// fp32 inputs take the plain kernels at the end of the file (the accuracy path).
#include <stdlib.h>
#include <type_traits>

#include "chunk_tables.h"
#include "common.h"
#include "prefill_launch.h"

namespace {

constexpr int BM = 64, BN = 64;  // tile shape of the bf16 block map
constexpr float LOG2E = 1.4426950408889634f;

struct BwdArgs {
  const uint16_t *q, *k, *v, *out, *dout;
  const float* lse;
  uint16_t *dq, *dk, *dv;
  float* delta;  // [T][hq]
  float* nlse2;  // [T][hq]  -lse log2(e)
  int32_t *kt_weight, *kt_order;        // [total key tiles] launch order of the dK/dV workgroups
  uint64_t* tok_vis0;                   // [T] first visibility word of every token's node
  int total_ktiles;
  const int32_t *cu_seqlens, *node_start, *tok_node, *qtile_start, *ktile_start;
  const int32_t* qtile_order;  // the forward's launch order: query tiles by descending number of visible key tiles
  const int32_t* qtile_desc;   // [launch slot][8]: token offset and length of the sequence, first row of the tile, CSR row start,
                               // tiles in the row, leading tiles without mask (FULL, not reaching past the end), node offset, -
  const int32_t* qtile_col;    // CSR of the visible key tiles of every query tile, the FULL ones first
  const uint8_t* qtile_flag;
  const uint64_t* node_vis;
  const int64_t* block_map_off;
  const uint8_t* block_map;
  int n_seqs, W, hq, hkv, G;
  long total_rows;  // T * hq
  float scale, sc;  // sc = scale * log2(e)
  // dQ: heads 0 .. dq_narrow - 1 of a KV head run NQ = four (head dimension 64: two) at a time on one
  // query tile, the others one at a time on NQ query tiles, whose tile lists bwd_wide_rows writes:
  // the list of the tiles NQ c .. of a sequence lies where row NQ c of its dense block map does
  int dq_narrow;
  int total_qtiles;
  int32_t* kt_again;  // [total key tiles] set where k_dkv_finish has to look (in the place of tok_vis0, which dQ has read by then)
  int32_t* wide_col;    // [dense map] key tiles that one of the query tiles sees, those that all of them see in full first
  int32_t *wide_n, *wide_nfast;  // [total query tiles] length of the list, leading entries without tests (at every NQ-th tile)
  int32_t* wide_list;   // [total query tiles + 1] the first tiles of the groups, sequence after sequence; last element: their number
  // dQ on query chunks (k_node_rows): the chunk table of pack_rows rows, heads of a KV head in an item, the nodes' runs
  ChunkTables chunk;
  int64_t slots;
  int pack_heads, pack_rows;
  const int32_t *runs, *tok_depth;
  // dK / dV on streams of query rows
  bool dkv_stream;
  const int32_t* node_tok_start;
  // streams cut into pieces (see bwd_order): {key tile, piece | pieces of the pair << 16} in launch order, their number, the
  // sums of the pieces that share a pair; null: a workgroup takes the whole stream of its pair
  int2* pieces;
  int32_t* split_first;  // [max_split / 2] first piece of every split pair
  int32_t* n_pieces;     // [2] pieces, split pairs
  f32x4* part;    // [split piece][hkv][4 waves][dK, dV: 32 dims][4][64 lanes]
  int max_split;  // room for this many pieces of split pairs (a KV head)
  int32_t* block_start;  // [total key tiles] first keys of a sequence's blocks (see cut_keys; T: no block); null: blocks are pairs of key tiles
  bool again;     // k_dkv_finish may read the inputs once more
  int dq_pieces, dq_piece;  // dQ on chunks: workgroups that may share a chunk, and tiles that each has at least, set per launch (see dq_cuts)
};

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int rho(int e, int H) { return 8 * (e >> 2) + 4 * H + (e & 3); }

__device__ __forceinline__ bf16x8 pack8(const float* x) {
  typedef __attribute__((ext_vector_type(8))) float f32x8;
  const f32x8 f = {x[0], x[1], x[2], x[3], x[4], x[5], x[6], x[7]};
  return __builtin_convertvector(f, bf16x8);
}

// Eq. 3 for a (query token i of node ni, key token j of node nj) pair of one sequence.  With at
// most 64 nodes per sequence (one visibility word) the test is a few selects, no branch and no load.
__device__ __forceinline__ bool visible(const BwdArgs& a, int nbase, int ni, int i, int nj, int j, uint64_t vis0) {
  if (a.W == 1) {
    const bool anc = (vis0 >> (nj & 63)) & 1u;
    return nj == ni ? j <= i : anc;
  }
  if (nj == ni) return j <= i;
  const uint64_t w = nj < 64 ? vis0 : a.node_vis[(int64_t)(nbase + ni) * a.W + (nj >> 6)];
  return (w >> (nj & 63)) & 1u;
}

// Tables kept in LDS per workgroup hold this many tiles (262,144 tokens); longer sequences read the
// rest from global memory.  (A build with a small DAG_BWD_LDS_TILES runs the tests through that path.)
#ifndef DAG_BWD_LDS_TILES
#define DAG_BWD_LDS_TILES 4096
#endif
constexpr int MAX_QT_LDS = DAG_BWD_LDS_TILES;  // query tiles of a sequence whose block-map column is kept in LDS

// A operand of a product whose contraction runs over the ROWS of a row-major LDS tile (K^T for dQ;
// Q^T and dO^T for dK and dV), read with the transposing LDS load of gfx950 (ds_read_b64_tr_b16):
// within 16 consecutive lanes, lane p hands in the address of four consecutive 16-bit elements and
// lane i receives, as component j, element i % 4 of the four that lane 4 j + i / 4 pointed at.
// With lane p pointing at tile[row 4 H + p / 4 (+ 8)][col 16 (lane / 16 % 2) + 4 (p % 4)], lane
// (L, H) of the wave gets tile[4 H + j (+ 8)][L], j = 0 .. 3: column L of the rows rho_H(0 .. 7), the
// row order in which the B operand (a previous result) holds its eight contraction elements.
// `tile` points at the first of the 16 rows and the first of the 32 columns of the operand.
template <int LD>
__device__ __forceinline__ bf16x8 read_transposed(const uint16_t* tile, int lane) {
  typedef short v4i16 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) v4i16* lds_v4_t;
  const int p = lane & 15, g = lane >> 4;
  const uint16_t* a0 = tile + (4 * (g >> 1) + (p >> 2)) * LD + 16 * (g & 1) + 4 * (p & 3);
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4_t)a0);
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4_t)(a0 + 8 * LD));
  typedef short v8i16 __attribute__((ext_vector_type(8)));
  const v8i16 x = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, x);
}

// The per-wave state of a dQ workgroup (64-row query tile x KV head x up to 4 of its query heads;
// two waves per head, each with 32 query rows: one row per lane and half wave).
template <int D>
struct DqLane {
  bf16x8 qf[D / 16], dof[D / 16];  // the row's Q and dO as B operands
  float lse2, dl;                  // its log-sum-exp (log2 units) and delta
  int i, ni;                       // its index in the sequence and its node
  uint64_t vis0;                   // first visibility word of that node
  bool row_ok;
  size_t qoff;                     // element offset of the row in q / dout / dq
};

template <int D>
__device__ __forceinline__ void dq_store(const BwdArgs& a, const DqLane<D>& me, int H, const f32x16* dQ) {
  if (!me.row_ok) return;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      u32x2 o;
      o[0] = dag_pack_bf2(dQ[db][4 * e4] * a.scale, dQ[db][4 * e4 + 1] * a.scale);
      o[1] = dag_pack_bf2(dQ[db][4 * e4 + 2] * a.scale, dQ[db][4 * e4 + 3] * a.scale);
      *(u32x2*)(a.dq + me.qoff + 32 * db + 8 * e4 + 4 * H) = o;
    }
}

// The visible key tiles of a query tile, FULL ones first (the forward's CSR row), copied to LDS at
// set-up; rows longer than the arrays read the rest from global memory.  get() is an
// inline-assembly LDS read that waits for itself: the loads of k_bwd_dq2's ring write LDS too, and
// a compiler-visible LDS read might be made to wait for all of them.
constexpr int MAX_ROW_LDS = DAG_BWD_LDS_TILES;
template <int CAP>
struct TileList {
  const int32_t* col;   // the row in global memory
  const uint8_t* flag;  // (first kernel only)
  uint32_t lds_col, lds_flag;  // LDS byte addresses of the copies
  template <int NT>
  __device__ __forceinline__ void fill(int32_t* sCol, int n) {
    for (int x = threadIdx.x; x < min(n, CAP); x += NT) sCol[x] = col[x];
    lds_col = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)sCol;
  }
  template <int NT>
  __device__ __forceinline__ void fill(int32_t* sCol, uint8_t* sFlg, int n) {
    fill<NT>(sCol, n);
    for (int x = threadIdx.x; x < min(n, CAP); x += NT) sFlg[x] = flag[x];
    lds_flag = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)sFlg;
  }
  __device__ __forceinline__ int tile(int n) const {
    if (n < CAP) {
      uint32_t v;
      asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(lds_col + 4u * (uint32_t)n) : "memory");
      return __builtin_amdgcn_readfirstlane((int)v);
    }
    return __builtin_amdgcn_readfirstlane(col[n]);
  }
  __device__ __forceinline__ int flag_of(int n) const {
    if (n < CAP) {
      uint32_t v;
      asm volatile("ds_read_u8 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(lds_flag + (uint32_t)n) : "memory");
      return __builtin_amdgcn_readfirstlane((int)v);
    }
    return __builtin_amdgcn_readfirstlane((int)flag[n]);
  }
};

// The walk of a dQ workgroup over entries n0 .. n1 - 1 of its tile list, one key tile at a time:
// the tile's K and V rows go through LDS (row-major, padded) for all the waves; the next tile is
// fetched into registers while the current one is multiplied (constant per-thread offsets, rows
// past the end re-read the last row and are zeroed on the way to LDS, no load depends on another).
template <int D, int NT, typename List>
__device__ __forceinline__ void dq_general_walk(const BwdArgs& a, unsigned char* smem, const List& tl, int n0, int n1, int T,
                                                int cu, int hk, int nbase, const DqLane<D>& me, f32x16* dQ) {
  constexpr int LD = D + 8;  // padded rows: the 16-byte operand reads of 32 consecutive rows spread over the banks
  uint16_t* const sK = (uint16_t*)smem;   // [BN][LD]
  uint16_t* const sV = sK + BN * LD;      // [BN][LD]
  int* const sNode = (int*)(sV + BN * LD);
  const int tid = threadIdx.x, lane = tid & 63, L = lane & 31, H = lane >> 5;
  constexpr int NPQ = (BN * (D / 8) + NT - 1) / NT;  // 16-byte pieces per thread and staged tile
  u32x4 rk[NPQ], rv[NPQ];
  int r_node = 0;
  uint32_t row_off[NPQ];
#pragma unroll
  for (int x = 0; x < NPQ; ++x) {
    const int c = min(tid + NT * x, BN * (D / 8) - 1);
    row_off[x] = (uint32_t)(c / (D / 8)) * (uint32_t)(a.hkv * D) + (uint32_t)(c % (D / 8)) * 8;
  }
  const uint32_t one_row = (uint32_t)(a.hkv * D);
  auto fetch = [&](int kt) {
    const int j0 = kt * BN, n_in = min(BN, T - j0);
    const size_t slab = ((size_t)(cu + j0) * a.hkv + hk) * D;
    const uint16_t* pk = a.k + slab;
    const uint16_t* pv = a.v + slab;
#pragma unroll
    for (int x = 0; x < NPQ; ++x) {
      const int c = min(tid + NT * x, BN * (D / 8) - 1), r = c / (D / 8);
      const uint32_t off = r < n_in ? row_off[x] : row_off[x] - (uint32_t)(r - (n_in - 1)) * one_row;
      rk[x] = *(const u32x4*)(pk + off);
      rv[x] = *(const u32x4*)(pv + off);
    }
    if (tid < BN) r_node = a.tok_node[cu + j0 + min(tid, n_in - 1)];
  };
  auto commit = [&](int kt) {
    const int n_in = min(BN, T - kt * BN);
#pragma unroll
    for (int x = 0; x < NPQ; ++x) {
      const int c = tid + NT * x, r = c / (D / 8), ch = c % (D / 8);
      if (c < BN * (D / 8)) {
        if (r >= n_in) rk[x] = rv[x] = u32x4{0, 0, 0, 0};
        *(u32x4*)(sK + r * LD + ch * 8) = rk[x];
        *(u32x4*)(sV + r * LD + ch * 8) = rv[x];
      }
    }
    if (tid < BN) sNode[tid] = r_node;
  };
  if (n0 >= n1) return;
  int kt_next = tl.tile(n0);
  fetch(kt_next);
  for (int n = n0; n < n1; ++n) {
    const int kt = kt_next;
    const int flag = tl.flag_of(n);
    const int j0 = kt * BN;
    __syncthreads();  // everybody is done with the tile in LDS
    commit(kt);
    __syncthreads();
    if (n + 1 < n1) {
      kt_next = tl.tile(n + 1);
      fetch(kt_next);  // in flight during the products below
    }
    const bool need_mask = flag == 1;
#pragma unroll 1
    for (int hh = 0; hh < 2; ++hh) {
      f32x16 S, dP;
#pragma unroll
      for (int e = 0; e < 16; ++e) S[e] = dP[e] = 0.f;
#pragma unroll
      for (int s = 0; s < D / 16; ++s) {  // S^T = K Q^T, dP^T = V dO^T: rows = keys, column = this lane's query row
        S = mfma32(*(const bf16x8*)(sK + (32 * hh + L) * LD + 16 * s + 8 * H), me.qf[s], S);
        dP = mfma32(*(const bf16x8*)(sV + (32 * hh + L) * LD + 16 * s + 8 * H), me.dof[s], dP);
      }
      float ds[16];
      if (!need_mask && j0 + BN <= T) {  // every in-range row sees every key of the tile: no tests
#pragma unroll
        for (int e = 0; e < 16; ++e) ds[e] = __builtin_amdgcn_exp2f(fmaf(S[e], a.sc, -me.lse2)) * (dP[e] - me.dl);
      } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int kk = 32 * hh + rho(e, H), j = j0 + kk;
          bool ok = me.row_ok && j < T;
          if (need_mask) ok = ok & visible(a, nbase, me.ni, me.i, sNode[kk], j, me.vis0);
          const float p = __builtin_amdgcn_exp2f(fmaf(S[e], a.sc, -me.lse2));
          ds[e] = ok ? p * (dP[e] - me.dl) : 0.f;
        }
      }
      const bf16x8 b0 = pack8(ds), b1 = pack8(ds + 8);
#pragma unroll
      for (int db = 0; db < D / 32; ++db) {  // dQ^T += K^T dS^T
        dQ[db] = mfma32(read_transposed<LD>(sK + (32 * hh) * LD + 32 * db, lane), b0, dQ[db]);
        dQ[db] = mfma32(read_transposed<LD>(sK + (32 * hh + 16) * LD + 32 * db, lane), b1, dQ[db]);
      }
    }
  }
}

// The set-up both dQ kernels share: the descriptor of the launch slot, then which row this lane
// owns and what it needs of it (no load depends on more than the descriptor).
struct DqTile {
  int cu, T, row0, c0, N, nfast, nbase;
};
__device__ __forceinline__ DqTile dq_tile(const BwdArgs& a) {
  const int32_t* d = a.qtile_desc + (size_t)blockIdx.x * 8;  // heaviest tiles first
  DqTile t;
  t.cu = d[0], t.T = d[1], t.row0 = d[2], t.c0 = d[3], t.N = d[4], t.nfast = d[5], t.nbase = d[6];
  return t;
}
// (g: query head of the KV head, i: this lane's row of the sequence)
template <int D>
__device__ __forceinline__ void dq_setup_row(const BwdArgs& a, const DqTile& t, int hk, int g, bool ok, int i, DqLane<D>& me) {
  const int h = hk * a.G + min(g, a.G - 1), H = (threadIdx.x & 63) >> 5;
  me.i = i;
  me.row_ok = me.i < t.T && ok;
  const int ic = min(me.i, t.T - 1);
  me.qoff = ((size_t)(t.cu + ic) * a.hq + h) * D;
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    me.qf[s] = *(const bf16x8*)(a.q + me.qoff + 16 * s + 8 * H);
    me.dof[s] = *(const bf16x8*)(a.dout + me.qoff + 16 * s + 8 * H);
  }
  me.lse2 = a.lse[(size_t)(t.cu + ic) * a.hq + h] * LOG2E;
  me.dl = a.delta[(size_t)(t.cu + ic) * a.hq + h];
  me.ni = a.tok_node[t.cu + ic];
  me.vis0 = a.runs ? 0 : a.tok_vis0[t.cu + ic];
}
// (row0: first row of this wave pair's 64-row query tile)
template <int D>
__device__ __forceinline__ void dq_setup_at(const BwdArgs& a, const DqTile& t, int hk, int g, bool head_ok, int row0, DqLane<D>& me) {
  dq_setup_row<D>(a, t, hk, g, head_ok, row0 + 32 * ((threadIdx.x >> 6) & 1) + (threadIdx.x & 31), me);
}
// Query chunks: (row, head) pair p of an item, row-major: its row and its head (heads <= 8, p < 256: exact).
__device__ __forceinline__ int2 dq_pair(int p, int heads) {
  const int row = (int)((uint32_t)p * ((65536u + heads - 1) / heads) >> 16);
  return {row, p - row * heads};
}
template <int D, int HG>
__device__ __forceinline__ void dq_setup(const BwdArgs& a, const DqTile& t, int hk, DqLane<D>& me) {
  const int g = blockIdx.z * HG + (threadIdx.x >> 7);  // two waves per query head
  dq_setup_at<D>(a, t, hk, g, g < a.dq_narrow, t.row0, me);
}

// First dQ kernel (every head dimension and head grouping): the general walk over all tiles.
template <int D, int HG>
__global__ void __launch_bounds__(128 * HG) k_bwd_dq(BwdArgs a) {
  constexpr int NT = 128 * HG;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int32_t sCol[MAX_ROW_LDS];
  __shared__ uint8_t sFlg[MAX_ROW_LDS];
  const DqTile t = dq_tile(a);
  const int hk = blockIdx.y;
  DqLane<D> me;
  dq_setup<D, HG>(a, t, hk, me);
  f32x16 dQ[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) dQ[db][e] = 0.f;
  TileList<MAX_ROW_LDS> tl;
  tl.col = a.qtile_col + t.c0;
  tl.flag = a.qtile_flag + t.c0;
  tl.template fill<NT>(sCol, sFlg, t.N);
  __syncthreads();
  dq_general_walk<D, NT>(a, smem, tl, 0, t.N, t.T, t.cu, hk, t.nbase, me, dQ);
  dq_store<D>(a, me, (threadIdx.x & 63) >> 5, dQ);
}

template <int D>
__device__ __forceinline__ void bwd_delta(const BwdArgs& a, int block) {
  // D / 8 lanes per (token, query head) row, 16 bytes of out and of dout per lane
  constexpr int LPR = D / 8, RPB = 256 / LPR;
  const long row = (long)block * RPB + threadIdx.x / LPR;
  const int part = threadIdx.x % LPR;
  float s = 0.f;
  if (row < a.total_rows) {
    const u32x4 o = *(const u32x4*)(a.out + (size_t)row * D + part * 8);
    const u32x4 g = *(const u32x4*)(a.dout + (size_t)row * D + part * 8);
#pragma unroll
    for (int e = 0; e < 4; ++e) s += dag_bf_lo(o[e]) * dag_bf_lo(g[e]) + dag_bf_hi(o[e]) * dag_bf_hi(g[e]);
  }
#pragma unroll
  for (int o = LPR / 2; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  if (part == 0 && row < a.total_rows) {
    a.delta[row] = s;
    a.nlse2[row] = -a.lse[row] * LOG2E;
  }
}

// Launch order of the dK/dV workgroups: heaviest first.  A workgroup takes a pair of key tiles
// (the even tile of a sequence and its successor); its weight is the number of query tiles that
// see the pair (the prefix keys of a plan are seen by every later tile, the keys of a branch by a
// few), odd tiles get -1 and sort last.  One wave per key tile, twice: weights, then ranks by
// counting (ties by index), which is fine for the few thousand tiles of a batch.
__device__ __forceinline__ void bwd_weight(const BwdArgs& a, int kt, int lane) {
  const int b = dag_find_segment(a.ktile_start, a.n_seqs, kt);
  const int ktl = kt - a.ktile_start[b];
  const int T = a.cu_seqlens[b + 1] - a.cu_seqlens[b];
  const int QT = (T + BM - 1) / BM, KT = (T + BN - 1) / BN;
  const uint8_t* bm = a.block_map + a.block_map_off[b];
  int n = 0;
  if (!(ktl & 1))
    for (int qt = lane; qt < QT; qt += 64)
      n += (bm[(int64_t)qt * KT + ktl] | (ktl + 1 < KT ? bm[(int64_t)qt * KT + ktl + 1] : 0)) != 0;
  n = dag_wave_sum(n);
  if (lane == 0) a.kt_weight[kt] = (ktl & 1) ? -1 : n;
}
// Blocks of keys whose borders are the nodes' where those allow it.  The stream of a block has every row that sees one of its
// keys, and its tiles take masks but for those of rows that see all of them: 128 keys from the start of a sequence on
// multiply 1.73 times the visible pairs of 4 x 64 random nodes of 32 to 256 tokens, 1263 of 5319 tiles without masks.  A block that
// ends at the last border of nodes 64 to 128 keys behind its first key, and where there is none has 128: 1.49 times, 2513 of
// 4579 tiles.  Cut at every border short nodes leave most of a workgroup idle (1.3 to 2.1 times the tiles for nodes of 35 to 60
// tokens), at least 96 keys a block are 0.5 % slower than 64, and with 64 there are no more blocks than key tiles.
// Where the siblings of a fork have about 100 tokens, blocks of 128 keys cost less: a sequence takes what needs less
// time by the tiles of the streams, one with masks 1.25 times one without, and DKV_BLOCK_STEPS iterations a workgroup.
// Forward and backward of 4 x 64 random nodes, 16 / 8 heads of dimension 64: 835 -> 788 us; 21 other batches 1.012 times as fast,
// random ones with long nodes 1.03 to 1.13 (0.984 at worst).
// (A workgroup a sequence.  The blocks follow one from the other, 80 clocks each: the first wave finds them while the others weigh the blocks
// of 128, and then all weigh those.  Four lanes a block, the nodes and the first keys in LDS.  With all waves finding the blocks first, and
// their keys and nodes read from memory, the launch in front of dQ took 24.0 instead of 19.2 us for one sequence of 67 nodes, 9800
// tokens, 12.9 instead of 11.8 for a fork of 18, 6600 tokens; without cuts 9.4 and 7.4.  Blocks weighed by whole waves, a node a
// lane, took 5 to 28 us.)
constexpr int BLOCK_MIN = 64, DKV_BLOCK_STEPS = 8, MAX_CUT_BLOCKS = 1024;
__device__ __forceinline__ void cut_keys(const BwdArgs& a, int b) {
  __shared__ uint64_t s_word[128][2];  // what a node sees
  __shared__ int s_first[129];
  __shared__ int s_start[MAX_CUT_BLOCKS + 1];  // first keys of the blocks cut at borders
  __shared__ int s_weight[MAX_CUT_BLOCKS];
  __shared__ float s_cost[2][4];
  __shared__ int s_blocks;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n0 = a.node_start[b], n = a.node_start[b + 1] - n0, cu = a.cu_seqlens[b], T = a.cu_seqlens[b + 1] - cu;
  const int slots = (T + BN - 1) / BN, n_even = (slots + 1) / 2;
  int32_t* const start = a.block_start + a.ktile_start[b];
  int32_t* const weight = a.kt_weight + a.ktile_start[b];
  if (tid <= 128) s_first[tid] = tid < n ? a.node_tok_start[n0 + tid] : T;
  s_word[tid >> 1][tid & 1] = (tid & 1) < a.W && (tid >> 1) < n ? a.node_vis[(int64_t)(n0 + (tid >> 1)) * a.W + (tid & 1)] : 0;
  __syncthreads();
  auto node_of = [&](int key) {
    int u = 0;
#pragma unroll
    for (int step = 64; step > 0; step >>= 1) u += s_first[u + step] <= key ? step : 0;
    return u;
  };
  // the block [key0, key1), by its four lanes, each with a quarter of the nodes: its tiles, and what it costs
  const int quarter = (n + 3) / 4, part = tid & 3;
  auto weigh = [&](int key0, int key1, int& tiles) {
    const int u0 = node_of(key0), u1 = node_of(key1 - 1);
    uint64_t range[2];  // bits u0 .. u1
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const int from = max(u0 - 64 * y, 0), to = min(u1 - 64 * y, 63);
      range[y] = from <= to ? (~0ull >> (63 - to)) & (~0ull << from) : 0ull;
    }
    int rows = 0, sure = 0;  // of the stream, and those of them that see all of the keys
#pragma unroll 3  // (62 registers; four times 97, 16.7 us, and the rows of delta in this launch run at half the occupancy: 1147 -> 1172 us in all for 34,000 tokens of 16 heads)
    for (int u = part * quarter; u < min((part + 1) * quarter, n); ++u) {
      const uint64_t w0 = s_word[u][0], w1 = s_word[u][1];
      const int first = u == u0 ? key0 : s_first[u], end = s_first[u + 1];
      const bool any = ((w0 & range[0]) | (w1 & range[1])) != 0, all = ((~w0 & range[0]) | (~w1 & range[1])) == 0;
      rows += any ? end - first : 0;
      sure += all ? end - (u == u1 ? key1 : first) : 0;
    }
    rows = dag_wave_sum<2>(rows);
    sure = dag_wave_sum<2>(sure);
    tiles = (rows + BM - 1) / BM;
    return a.G * (1.25f * tiles - 0.25f * (sure / BM)) + DKV_BLOCK_STEPS;
  };
  float cost[2] = {0.f, 0.f};  // blocks of 128 keys, blocks cut at borders
  if (slots <= MAX_CUT_BLOCKS && w == 0) {
    const int first0 = s_first[lane], first1 = s_first[64 + lane];
    int n_cut = 0, mine = 0;
    for (int key0 = 0; key0 < T; ++n_cut) {
      mine = lane == (n_cut & 63) ? key0 : mine;
      if ((n_cut & 63) == 63) s_start[n_cut - 63 + lane] = mine;
      const uint32_t lo = key0 + BLOCK_MIN, hi = key0 + 2 * BN;
      const uint64_t m0 = __builtin_amdgcn_ballot_w64((uint32_t)first0 - lo <= hi - lo), m1 = n > 64 ? __builtin_amdgcn_ballot_w64((uint32_t)first1 - lo <= hi - lo) : 0;
      key0 = hi;
      if (m0 != 0) key0 = __builtin_amdgcn_readlane(first0, 63 - __builtin_clzll(m0));
      if (m1 != 0) key0 = __builtin_amdgcn_readlane(first1, 63 - __builtin_clzll(m1));
      if ((uint32_t)T <= hi) key0 = T;
    }
    if (lane < (n_cut & 63)) s_start[(n_cut & ~63) + lane] = mine;
    if (lane == 0) s_start[n_cut] = T, s_blocks = n_cut;
  } else if (w > 0) {
    for (int i0 = 0; i0 < n_even; i0 += 48) {
      const int at = i0 + ((tid - 64) >> 2), i = min(at, n_even - 1);
      int tiles;
      const float c = weigh(i * 2 * BN, min((i + 1) * 2 * BN, T), tiles);
      if (at == i && part == 0) {
        cost[0] += c;
        weight[i] = tiles;
      }
    }
  }
  __syncthreads();
  bool even = slots > MAX_CUT_BLOCKS;  // (a sequence that has more blocks keeps them)
  const int n_cut = even ? 0 : s_blocks;
  for (int i0 = 0; i0 < n_cut; i0 += 64) {
    const int at = i0 + (tid >> 2), i = min(at, n_cut - 1);
    int tiles;
    const float c = weigh(s_start[i], s_start[i + 1], tiles);
    if (at == i && part == 0) {
      cost[1] += c;
      s_weight[i] = tiles;
    }
  }
#pragma unroll
  for (int y = 0; y < 2; ++y) {
    const float c = dag_wave_sum(cost[y]);
    if (lane == 0) s_cost[y][w] = c;
  }
  __syncthreads();
  if (!even) even = s_cost[0][0] + s_cost[0][1] + s_cost[0][2] + s_cost[0][3] < 1.03f * (s_cost[1][0] + s_cost[1][1] + s_cost[1][2] + s_cost[1][3]);
  for (int x = tid; x < slots; x += 256) {  // (behind the barrier: the weights of the blocks of 128 are other threads')
    const bool block = x < (even ? n_even : n_cut);
    start[x] = !block ? T : even ? x * 2 * BN : s_start[x];
    if (!block || !even) weight[x] = block ? s_weight[x] : -1;
  }
}
// The keys [x, y) of the workgroup of key tile kt (the ktl-th of its sequence).
__device__ __forceinline__ int2 dkv_keys(const BwdArgs& a, int kt, int ktl, int T) {
  if (!a.block_start) return int2{ktl * BN, min((ktl + 2) * BN, T)};
  return int2{a.block_start[kt], (ktl + 1) * BN < T ? a.block_start[kt + 1] : T};
}
// First visibility word of every token's node, so that the dQ kernels on the block map's tiles can fetch it for
// their rows without a load that depends on another load.
__device__ __forceinline__ void bwd_token_vis(const BwdArgs& a, int t) {
  const int b = dag_find_segment(a.cu_seqlens, a.n_seqs, t);
  a.tok_vis0[t] = a.node_vis[(int64_t)(a.node_start[b] + a.tok_node[t]) * a.W];
}

// What the other kernels read, as far as it comes from the inputs alone: the chunks of dQ or the
// words of its rows on the block map's tiles, the weights of the key tiles, delta.  One launch, because none of
// them waits for another and a launch of any of them costs 4.6 us, however little it does; the longest chains
// first.  Five launches were 23 us of the 114 that 33 nodes of 80 tokens take forward and backward.
struct PrepareBlocks {
  int nodes, tokens, weights, delta;  // blocks of each
};
template <int D>
__global__ void __launch_bounds__(256) k_bwd_delta_tables(BwdArgs a, PrefillArgs p, PrepareBlocks n) {
  int x = blockIdx.x;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (x < n.nodes) {
    const int gv = 4 * x + w;
    if (gv >= p.total_nodes) return;
    if (a.W == 1)
      node_rows<1>(gv, p.n_seqs, (int)p.total_nodes, a.pack_rows, a.slots, p.node_start, p.cu_seqlens, p.tok_node, p.node_tok_start, p.node_vis, p.node_runs, a.chunk);
    else
      node_rows<2>(gv, p.n_seqs, (int)p.total_nodes, a.pack_rows, a.slots, p.node_start, p.cu_seqlens, p.tok_node, p.node_tok_start, p.node_vis, p.node_runs, a.chunk);
    return;
  }
  x -= n.nodes;
  if (x < n.tokens) {
    if (a.runs) {
      token_depths(p, (int64_t)x * 256);
    } else {
      const int64_t t = (int64_t)x * 256 + threadIdx.x;
      if (t < a.total_rows / a.hq) bwd_token_vis(a, (int)t);
    }
    return;
  }
  x -= n.tokens;
  if (x < n.weights) {
    if (a.block_start)
      cut_keys(a, x);
    else if (4 * x + w < a.total_ktiles)
      bwd_weight(a, 4 * x + w, lane);
    return;
  }
  bwd_delta<D>(a, x - n.weights);
}

// Pairs that many rows see are cut into pieces, each a range of the stream and a workgroup of its own, summed by
// k_dkv_finish: the root of a plan is seen by all of its rows, and its one workgroup ran on when all others were done
// (4 x 75 nodes, five heads of dimension 64 on one KV head: 1020 of 1280 us, in pieces 127 + 15; 4 x 64 nodes, 16 / 8
// heads: 513, in pieces 420).  A piece has at most the tiles that a workgroup gets where all are shared out evenly, and
// at least DKV_MIN_STEPS iterations (a piece starts and ends in about five, its sums are 128 KiB at dimension 128).  w >
// cap tiles make ceil(w / cap) < 2 w / cap pieces, so 2 W / cap slots hold those of all W tiles.  Split pairs are the
// heaviest: their pieces come first in the launch order.  Forward and backward of 28 shapes with nodes of 50 to 500
// tokens, 1 to 8 KV heads, against whole streams: 1.63 times as fast (0.99 to 4.7); pieces of a third, half and twice
// the even share 1.60, 1.61, 1.53; of 16 iterations at least 1.60; none in pairs below 1.25 times the even share 1.59.
constexpr int DKV_MIN_STEPS = 8;
__device__ __forceinline__ int dkv_pieces(int w, int cap) { return w > cap ? (w + cap - 1) / cap : 1; }
__device__ __forceinline__ void bwd_order(const BwdArgs& a, int kt, int lane) {
  const int mine = a.kt_weight[kt];
  int rank = 0, sum = 0;
  for (int x = lane; x < a.total_ktiles; x += 64) {
    const int w = a.kt_weight[x];
    rank += w > mine || (w == mine && x < kt);
    sum += max(w, 0);
  }
  rank = dag_wave_sum(rank);
  if (lane == 0 && a.dkv_stream) a.kt_again[kt] = 0;
  if (!a.pieces) {
    if (lane == 0) a.kt_order[rank] = kt;
    return;
  }
  const int total = dag_wave_sum(sum);
  const int cap = max((DKV_MIN_STEPS + a.G - 1) / a.G, (int)((2 * (int64_t)total + a.max_split - 1) / a.max_split));
  int first = 0, all = 0, pairs = 0;
  for (int x = lane; x < a.total_ktiles; x += 64) {
    const int w = a.kt_weight[x], n = w >= 0 ? dkv_pieces(w, cap) : 0;
    all += n;
    pairs += n > 1;
    first += w > mine || (w == mine && x < kt) ? n : 0;
  }
  first = dag_wave_sum(first);
  all = dag_wave_sum(all);
  pairs = dag_wave_sum(pairs);
  if (kt == 0 && lane == 0) a.n_pieces[0] = all, a.n_pieces[1] = pairs;
  const int n = mine >= 0 ? dkv_pieces(mine, cap) : 0;
  for (int p = lane; p < n; p += 64) a.pieces[first + p] = int2{kt, p | n << 16};
  if (lane == 0 && n > 1) a.split_first[rank] = first;
}

template <int D>
constexpr int dkv_smem_bytes() {
  // Q and dO rows of one query tile for one query head and their transposed images, lse / delta of
  // the rows, node ids and first visibility words of the rows
  return 2 * BM * (D + 8) * 2 + 2 * BM * 4 + BM * 4 + BM * 8;
}

// The walk of one workgroup of the dK/dV kernels (pair of key tiles x KV head; wave w owns keys
// 32 w .. 32 w + 31 of the pair, with their K and V rows as B operands in registers and dK^T, dV^T
// accumulators for them) over the query tiles from the last one down and over the query heads of
// the group, one (tile, head) at a time: its Q and dO rows go through LDS (row-major, padded) for
// all four waves, the next (tile, head) is fetched into registers while the current one is
// computed.  `pair_flag(qt)` returns flag of tile 0 | flag of tile 1 << 2 of the pair for query
// tile qt, or 0 where the walk is to leave the tile out.  Pairs of a tile that are all visible
// run without a single test, the others evaluate Eq. 3 and the sequence end per element.
template <int D, typename PairFlag>
__device__ __forceinline__ void dkv_general_walk(const BwdArgs& a, unsigned char* smem, PairFlag&& pair_flag, int QT, int T,
                                                 int cu, int hk, int nbase, int my_kt, int nj, int j, bool key_ok,
                                                 const bf16x8* kf, const bf16x8* vf, f32x16* dK, f32x16* dV) {
  constexpr int LD = D + 8, DB = D / 32;
  constexpr int NP = BM * (D / 8) / 256;  // 16-byte pieces per thread and staged tile
  uint16_t* const sQ = (uint16_t*)smem;                  // [BM][LD]
  uint16_t* const sdO = sQ + BM * LD;                    // [BM][LD]
  float* const sLse = (float*)(sdO + BM * LD);           // [BM]  (log2 units)
  float* const sDl = sLse + BM;                          // [BM]
  int* const sNodeR = (int*)(sDl + BM);                  // [BM]
  uint64_t* const sVis0 = (uint64_t*)(sNodeR + BM);      // [BM]
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, L = lane & 31, H = lane >> 5;
  auto next_tile = [&](int qt) {  // last query tile <= qt with a visible pair, -1 if none
    while (qt >= 0 && pair_flag(qt) == 0) --qt;
    return qt;
  };
  // register stage of one (tile, head)
  // (addresses: a wave-uniform 64-bit base per tile and head plus 32-bit per-thread offsets that
  // never change; rows past the end of the sequence re-read its last row and are zeroed afterwards,
  // so no load sits under a branch; no load depends on another one: a wait for the first would
  // also wait for everything issued before it)
  u32x4 rq[NP], rdo[NP];
  float r_lse = 0.f, r_dl = 0.f;
  int r_node = 0;
  uint64_t r_vis = 0;
  uint32_t row_off[NP];  // element offset of this thread's piece x inside a 64-row slab of q / dout
#pragma unroll
  for (int x = 0; x < NP; ++x) {
    const int c = tid + 256 * x;
    row_off[x] = (uint32_t)(c / (D / 8)) * (uint32_t)(a.hq * D) + (uint32_t)(c % (D / 8)) * 8;
  }
  const uint32_t last_off = (uint32_t)(a.hq * D);  // one row
  auto fetch = [&](int qt, int g) {
    const int r0 = qt * BM;
    const int h = hk * a.G + g;
    const size_t slab = ((size_t)(cu + r0) * a.hq + h) * D;
    const uint16_t* pq = a.q + slab;
    const uint16_t* pdo = a.dout + slab;
    const int n_in = min(BM, T - r0);  // rows of the tile inside the sequence (>= 1)
#pragma unroll
    for (int x = 0; x < NP; ++x) {
      const int c = tid + 256 * x, r = c / (D / 8);
      const uint32_t off = r < n_in ? row_off[x] : row_off[x] - (uint32_t)(r - (n_in - 1)) * last_off;
      rq[x] = *(const u32x4*)(pq + off);
      rdo[x] = *(const u32x4*)(pdo + off);
    }
    if (tid < BM) {
      const int rr = min(tid, n_in - 1);
      const size_t row = (size_t)(cu + r0 + rr) * a.hq + h;
      r_lse = a.lse[row];
      r_dl = a.delta[row];
      r_node = a.tok_node[cu + r0 + rr];
      r_vis = a.tok_vis0[cu + r0 + rr];
    }
  };
  auto commit = [&](int qt_of_regs) {
    const int n_in = min(BM, T - qt_of_regs * BM);
#pragma unroll
    for (int x = 0; x < NP; ++x) {
      const int c = tid + 256 * x, r = c / (D / 8), ch = c % (D / 8);
      if (r >= n_in) rq[x] = rdo[x] = u32x4{0, 0, 0, 0};
      *(u32x4*)(sQ + r * LD + ch * 8) = rq[x];
      *(u32x4*)(sdO + r * LD + ch * 8) = rdo[x];
    }
    if (tid < BM) {
      sLse[tid] = tid < n_in ? r_lse * LOG2E : 0.f;
      sDl[tid] = tid < n_in ? r_dl : 0.f;
      sNodeR[tid] = r_node;
      sVis0[tid] = r_vis;
    }
  };

  int qt = next_tile(QT - 1), g = 0;
  if (qt >= 0) fetch(qt, g);
  while (qt >= 0) {
    __syncthreads();  // everybody is done with the tile in LDS
    commit(qt);
    __syncthreads();
    const int cur_qt = qt;
    // (every global load the products depend on comes before the fetch: a wait for a later load
    // would also wait for the fetch, the counter being in order)
    const int flag = __builtin_amdgcn_readfirstlane((pair_flag(cur_qt) >> (2 * (w >> 1))) & 3);
    if (++g == a.G) {
      g = 0;
      qt = next_tile(qt - 1);
    }
    if (qt >= 0) fetch(qt, g);  // in flight during the products below
    if (flag != 0) {
      const int r0 = cur_qt * BM;
      const bool need_mask = flag == 1;
#pragma unroll 1
      for (int rb = 0; rb < BM / 32; ++rb) {
        f32x16 S, dP;
#pragma unroll
        for (int e = 0; e < 16; ++e) S[e] = dP[e] = 0.f;
        // (all operand reads of a phase are issued before its first MFMA: one wave per SIMD has
        // nobody to hide the LDS latency behind, so the reads are kept far ahead of their use)
        bf16x8 aq[D / 16], ado[D / 16];
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
          aq[s] = *(const bf16x8*)(sQ + (32 * rb + L) * LD + 16 * s + 8 * H);
          ado[s] = *(const bf16x8*)(sdO + (32 * rb + L) * LD + 16 * s + 8 * H);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {  // S = Q K^T, dP = dO V^T: rows = query rows, column = this lane's key
          S = mfma32(aq[s], kf[s], S);
          dP = mfma32(ado[s], vf[s], dP);
        }
        // the transposed operands of the second phase: on their way during the exponentials
        bf16x8 at_do[2 * DB], at_q[2 * DB];
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          at_do[2 * db] = read_transposed<LD>(sdO + (32 * rb) * LD + 32 * db, lane);
          at_do[2 * db + 1] = read_transposed<LD>(sdO + (32 * rb + 16) * LD + 32 * db, lane);
          at_q[2 * db] = read_transposed<LD>(sQ + (32 * rb) * LD + 32 * db, lane);
          at_q[2 * db + 1] = read_transposed<LD>(sQ + (32 * rb + 16) * LD + 32 * db, lane);
        }
        __builtin_amdgcn_sched_barrier(0);
        float p[16], ds[16];
        // lse and delta of the 16 rows of this lane: four groups of four consecutive rows
        f32x4 l4[4], d4[4];
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          l4[e4] = *(const f32x4*)(sLse + 32 * rb + 8 * e4 + 4 * H);
          d4[e4] = *(const f32x4*)(sDl + 32 * rb + 8 * e4 + 4 * H);
        }
        if (!need_mask && r0 + BM <= T && (my_kt + 1) * BN <= T) {  // every pair of the tile is visible: no tests
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            p[e] = __builtin_amdgcn_exp2f(fmaf(S[e], a.sc, -l4[e >> 2][e & 3]));
            ds[e] = p[e] * (dP[e] - d4[e >> 2][e & 3]);
          }
        } else {
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int r = 32 * rb + rho(e, H), i = r0 + r;
            bool ok = key_ok && i < T;
            if (need_mask) ok = ok & visible(a, nbase, sNodeR[r], i, nj, j, sVis0[r]);
            const float pe = __builtin_amdgcn_exp2f(fmaf(S[e], a.sc, -l4[e >> 2][e & 3]));
            p[e] = ok ? pe : 0.f;
            ds[e] = p[e] * (dP[e] - d4[e >> 2][e & 3]);
          }
        }
        const bf16x8 p0 = pack8(p), p1 = pack8(p + 8), s0 = pack8(ds), s1 = pack8(ds + 8);
#pragma unroll
        for (int db = 0; db < DB; ++db) {  // dV^T += dO^T P, dK^T += Q^T dS
          dV[db] = mfma32(at_do[2 * db], p0, dV[db]);
          dV[db] = mfma32(at_do[2 * db + 1], p1, dV[db]);
          dK[db] = mfma32(at_q[2 * db], s0, dK[db]);
          dK[db] = mfma32(at_q[2 * db + 1], s1, dK[db]);
        }
      }
    }
  }
}

// Writes the dK and dV rows of a wave's 32 keys (column = this lane's key, rows = d: every lane
// writes its key's row).
template <int D>
__device__ __forceinline__ void dkv_store(const BwdArgs& a, size_t koff, bool key_ok, int H, const f32x16* dK, const f32x16* dV) {
  if (!key_ok) return;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      u32x2 ok2, ov2;
      ok2[0] = dag_pack_bf2(dK[db][4 * e4] * a.scale, dK[db][4 * e4 + 1] * a.scale);
      ok2[1] = dag_pack_bf2(dK[db][4 * e4 + 2] * a.scale, dK[db][4 * e4 + 3] * a.scale);
      ov2[0] = dag_pack_bf2(dV[db][4 * e4], dV[db][4 * e4 + 1]);
      ov2[1] = dag_pack_bf2(dV[db][4 * e4 + 2], dV[db][4 * e4 + 3]);
      *(u32x2*)(a.dk + koff + 32 * db + 8 * e4 + 4 * H) = ok2;
      *(u32x2*)(a.dv + koff + 32 * db + 8 * e4 + 4 * H) = ov2;
    }
}

// First dK/dV kernel (every head dimension): the general walk over all tiles.
template <int D>
__global__ void __launch_bounds__(256) k_bwd_dkv(BwdArgs a) {
  constexpr int DB = D / 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ uint8_t sFlag[MAX_QT_LDS];                  // block-map column of the pair: flag of tile 0 | flag of tile 1 << 2
  // (the KV head is the fast index of the launch: workgroups go to the XCDs round robin, so with 8
  // KV heads every XCD's L2 holds the Q / dO tiles of one head group only, and the workgroups of a
  // group walk over the query tiles from the last one down, i.e. side by side)
  const int hk = blockIdx.x % a.hkv, kt = a.kt_order[blockIdx.x / a.hkv];  // heaviest pairs first
  const int b = dag_find_segment(a.ktile_start, a.n_seqs, kt);
  const int ktl = kt - a.ktile_start[b];
  if (ktl & 1) return;  // the workgroup of the even tile takes the pair (odd tiles come last in the order)
  const int cu = a.cu_seqlens[b], T = a.cu_seqlens[b + 1] - cu;
  const int QT = (T + BM - 1) / BM, KT = (T + BN - 1) / BN;
  const uint8_t* bm = a.block_map + a.block_map_off[b];
  const int nbase = a.node_start[b];
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, L = lane & 31, H = lane >> 5;
  const int my_kt = ktl + (w >> 1);          // this wave's key tile
  const int j = ktl * BN + 32 * w + L;       // this lane's key
  const bool key_ok = j < T;
  const int jc = min(j, T - 1);
  const size_t koff = ((size_t)(cu + jc) * a.hkv + hk) * D;
  bf16x8 kf[D / 16], vf[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    kf[s] = *(const bf16x8*)(a.k + koff + 16 * s + 8 * H);
    vf[s] = *(const bf16x8*)(a.v + koff + 16 * s + 8 * H);
  }
  const int nj = a.tok_node[cu + jc];
  f32x16 dK[DB], dV[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) dK[db][e] = dV[db][e] = 0.f;

  // (the map is read once: a load of it inside the loop would sit, with its full latency, in front
  // of every tile; sequences with more query tiles than the array holds read the map directly)
  const bool flags_in_lds = QT <= MAX_QT_LDS;
  if (flags_in_lds) {
    for (int x = tid; x < QT; x += 256) {
      const int f0 = bm[(int64_t)x * KT + ktl];
      const int f1 = ktl + 1 < KT ? bm[(int64_t)x * KT + ktl + 1] : 0;
      sFlag[x] = (uint8_t)(f0 | (f1 << 2));
    }
    __syncthreads();
  }
  auto pair_flag = [&](int qt) {
    if (flags_in_lds) return (int)sFlag[qt];
    const int f0 = bm[(int64_t)qt * KT + ktl];
    const int f1 = ktl + 1 < KT ? bm[(int64_t)qt * KT + ktl + 1] : 0;
    return f0 | (f1 << 2);
  };
  dkv_general_walk<D>(a, smem, pair_flag, QT, T, cu, hk, nbase, my_kt, nj, j, key_ok, kf, vf, dK, dV);
  dkv_store<D>(a, koff, key_ok, H, dK, dV);
}

// ---------------------------------------------------------------------------------------------
// k_bwd_dkv2: the dK/dV kernel for head dimension 128 with the data movement and the instruction
// order of the forward kernel.  Same decomposition as k_bwd_dkv (pair of key tiles x KV head, wave
// w owns keys 32 w .. 32 w + 31, iteration = (query tile, query head)), but
//   * the Q and dO tiles go from global memory straight into LDS (16 bytes per lane, no staging
//     registers) through a ring of NST stages; one bare s_barrier per iteration, in its middle:
//     it publishes the stage of the NEXT iteration (every wave has waited for its own loads of
//     that stage before) and frees the stage of the previous one, which the loads of iteration
//     n + NST - 1 then fill, one load per MFMA slot;
//   * a wave-level load writes 1 KiB of consecutive LDS, a block of 4 rows laid out
//     [chunk / 4][row % 4][chunk % 4][16 B], blocks 1024 + 16 bytes apart: four consecutive lanes
//     fetch 64 consecutive bytes, the 16-byte row reads (A operands of S = Q K^T, dP = dO V^T) of 16
//     consecutive rows and the 8-byte transposing reads (A operands of dV^T += dO^T P,
//     dK^T += Q^T dS) of 16 consecutive lanes both fall into 16 different bank groups;
//   * an iteration is written slot by slot (operand read of the MFMA PF slots ahead, wait, one
//     MFMA, a share of the exponentials; a scheduling barrier after every slot): scores and dP of
//     the two 32-row halves (32 MFMAs), then dV / dK of the two halves (32 MFMAs), with the
//     exponentials of half 0 in the slots of the score MFMAs of half 1 and those of half 1 in the
//     slots of the dV / dK MFMAs of half 0.  The operand reads are inline assembly with explicit
//     lgkmcnt waits (LDS reads return in order); nothing branches while such reads are in flight,
//     so no copy of a register that is still being written can be made
//     (tests/test_asm_lds_reads.py checks the generated code for exactly that);
//   * two such loops run one after the other: the iterations whose pairs are all visible (both key
//     tiles FULL, nothing past the end of the sequence), then the masked and ragged ones: Eq. 3 of
//     a (query tile, key) pair is one 64-bit word per lane, built once per query tile from the runs
//     of equal node ids among its rows (tile_visibility) and applied with two instructions per
//     element; the ancestor test uses the key's column of the visibility matrix, built once per
//     workgroup.  Both loops find their tiles through a bitmap per kind of the pair's block-map
//     column.
// Every iteration passes the barrier once and issues LPS loads per wave (past the end of the walk:
// loads of the sequence's first tile, never consumed), so the vmcnt waits are constants.
// With one wave per SIMD (the accumulators and the K / V operands of 32 keys need 192 registers)
// nothing of a wave overlaps its own MFMAs: an iteration costs the 64 MFMAs plus the time to
// issue everything else.
// Head dimension 64 (k_bwd64_dkv) runs the same code with half the slots: 16 score MFMAs, then 16 of
// dV / dK, two scores per slot.  Accumulators and operands take 96 instead of 192 registers and a ring
// of four stages 71 instead of 137 KB, so two workgroups share a compute unit and each SIMD has two
// waves: the exponentials of one run beside the MFMAs of the other.  A 1 KiB block then holds 8
// rows of 128 bytes, 16-byte chunk c of row r at position 8 r + (c ^ swz64(r)), blocks 1024 + 64 bytes
// apart: eight lanes fetch one row, and both kinds of operand read fall into different banks.
// Random DAGs of 4 x 64 nodes of 32 to 256 tokens, 16 query / 8 KV heads: 2000 us with k_bwd_dkv, 517 so.
__host__ __device__ constexpr int swz64(int r) { return ((r >> 1) & 1) * 2 + ((r >> 2) & 1); }
// What the ring's tiles look like, for both pipelined kernels: 64 rows of D elements in blocks of 1 KiB.
template <int D>
struct RingTile {
  static constexpr int RPB = 512 / D;                 // rows per block
  static constexpr int NBLK = 64 / RPB;               // blocks per tile
  static constexpr int BLK = 1024 + (D == 128 ? 16 : 64);
  static constexpr int TILEB = NBLK * BLK;
  // what lane `lane` of a wave-level load fetches: row of the block, element offset inside the row
  __device__ static int src_row(int lane) { return D == 128 ? (lane >> 2) & 3 : lane >> 3; }
  __device__ static uint32_t src_col(int lane) {
    return D == 128 ? (uint32_t)(4 * (lane >> 4) + (lane & 3)) * 8 : (uint32_t)((lane & 7) ^ swz64(lane >> 3)) * 8;
  }
  // per-lane part of the address of a row operand (row L of 32, chunk 2 s + H): for even and for odd
  // k-steps s (one register for both where the chunks lie in order)
  __device__ static uint32_t row_lane(int L, int H, int odd) {
    return D == 128 ? (uint32_t)((L >> 2) * BLK + (L & 3) * 64 + H * 16 + odd * 32)
                    : (uint32_t)((L >> 3) * BLK + (L & 7) * 128 + ((2 * odd + H) ^ swz64(L & 7)) * 16);
  }
  static constexpr int row_imm(int half, int s) {  // ... and the rest, after that part for k-step s
    return D == 128 ? 8 * half * BLK + (s / 2) * 256 : 4 * half * BLK + (s / 2) * 64;
  }
  // per-lane part of the address of a transposing read (rows 4 H + .., 32 columns), and the rest: 16-row
  // group x of the tile, rows + 8 when `second`, columns 32 db ..
  __device__ static uint32_t tr_lane(int lane) {
    const int H = lane >> 5, g1 = (lane >> 4) & 1, p = lane & 15;
    return D == 128 ? (uint32_t)(H * BLK + (p >> 2) * 64 + g1 * 32 + (p & 3) * 8)
                    : (uint32_t)((4 * H + (p >> 2)) * 128 + ((2 * g1 + ((p >> 1) & 1)) ^ swz64(4 * H + (p >> 2))) * 16 + (p & 1) * 8);
  }
  static constexpr int tr_imm(int x, int second, int db) {
    return D == 128 ? (4 * x + 2 * second) * BLK + db * 256 : (2 * x + second) * BLK + db * 64;
  }
};
template <int D>
struct Dkv {
  using R = RingTile<D>;
  static constexpr int NST = 4;                    // ring depth
  static constexpr int NPB = R::NBLK / 4;          // blocks of a tile that one wave fetches
  static constexpr int LPS = 2 * NPB + 1;          // wave-level loads per stage and wave: Q blocks, dO blocks, 1 of row data
  static constexpr int PF = D == 128 ? 5 : 3;      // operands in flight ahead of their MFMA
  static constexpr int TILEB = R::TILEB;
  static constexpr int RD = 2 * TILEB;             // row data: -lse log2(e) [64], delta [64], node id [64]
  static constexpr int STAGEB = RD + 768;
  static constexpr int HS = D / 8;                 // slots of the score MFMAs of one 32-row half
  static constexpr int NSC = 2 * HS, NSLOT = 4 * HS;
  static constexpr int EPS = 16 / HS;              // scores turned into P and dS per slot (slots HS .. 3 HS - 1)
  static constexpr int VAHEAD = D == 128 ? 8 : 3;  // the row data of four rows are read this many slots before their first use
  static constexpr int XR = D == 128 ? 2 : 1;      // row-data reads per group of four rows: -lse and delta
  // V is negated, and the sums of -dP start from delta: no vector instruction subtracts it (but on the block map's tiles at head dimension
  // 128).  At head dimension 64 it is read in front of the iteration (half 0) or at this slot.
  // 32 of 171 (dimension 64) and 32 of 153 vector instructions an iteration: 4 x 64 random nodes, 16 / 8 heads of dimension 64 831 -> 810 us, 32 / 8 of
  // 128 2583 -> 2532, fork-joins 1.00 to 1.01 times as fast.
  static constexpr int DELTA_SLOT = HS - PF;
  static constexpr int opnd_reads(int o) { return o < NSC ? 1 : 2; }
  // The scores of rows 4 x .. 4 x + 3 of half h are taken from slot HS (1 + h) + 4 x / EPS on; the XR reads
  // of their row data go out VAHEAD >= PF slots earlier, i.e. before the operand read that slot waits
  // for, so they have arrived with it.
  static constexpr int extra_reads(int slot) {
    return (D != 128 && slot == DELTA_SLOT ? 4 : 0) + row_reads(slot);
  }
  static constexpr int row_reads(int slot) {
    return slot >= HS - VAHEAD && slot < 3 * HS - VAHEAD && (slot - (HS - VAHEAD)) % (4 / EPS) == 0 ? XR : 0;
  }
  static constexpr int issued_through(int k) {  // LDS reads issued up to and including those of operand k
    int t = 0;
    for (int o = 0; o <= k; ++o) t += (o >= PF ? extra_reads(o - PF) : 0) + opnd_reads(o);
    return t;
  }
  static constexpr int wait_at(int i) {  // reads that may still be pending when MFMA i starts
    const int last = i + PF < NSLOT ? i + PF : NSLOT - 1;
    const int n = issued_through(last) - issued_through(i);
    return n < 15 ? n : 15;
  }
  // The turned iteration (see turned_iter): row operands in the first and third quarter, transposed ones in the second and the
  // last; the row data of four rows every eight slots.  The first element of a half follows TURN_GAP slots behind the end of its
  // scores.
  static constexpr int TURN_GAP = 4;
  static constexpr bool turned_row(int i) { return i / 16 % 2 == 0; }
  static constexpr int TURN_SYNC = 2 * HS - PF;  // the next tile is there; its first operand is fetched in this slot, delta of its half 0 in front of it
  static constexpr int turned_extra(int slot) { return (slot % 8 == TURN_GAP ? 1 : 0) + (slot == TURN_SYNC ? 4 : 0); }
  static constexpr int turned_issued(int k) {
    int t = 0;
    for (int o = 0; o <= k; ++o) t += (o >= PF ? turned_extra(o - PF) : 0) + (turned_row(o) ? 1 : 2);
    return t;
  }
  static constexpr int turned_wait(int i) {
    const int last = i + PF < NSLOT ? i + PF : NSLOT - 1;
    int n = turned_issued(last) - turned_issued(i);
    for (int slot = last + 1 - PF; slot <= i; ++slot) n += turned_extra(slot);  // (behind the last operand)
    return i == NSLOT - 1 ? 0 : n < 15 ? n : 15;
  }
  // byte offset (after the per-lane part) of operand i
  static constexpr int row_imm(int i) {  // i < NSC: row operand of half i / HS, k-step (i % HS) / 2, of Q (even) or dO (odd)
    return (i & 1) * TILEB + R::row_imm(i / HS, (i % HS) / 2);
  }
  static constexpr int tr_imm(int i, int second) {  // i >= NSC: transposed operand (dims 32 db .., 16 rows) of dO (even) or Q (odd)
    const int j = i - NSC, h = j / HS, jj = j % HS, db = jj / 4, hh = (jj / 2) % 2;
    return ((jj & 1) ? 0 : TILEB) + R::tr_imm(2 * h + hh, second, db);
  }
};


// Eq. 3 for one 64 x 64 tile as a 64-bit word per lane: bit c says
// whether element c of the tile -- query row c for a lane that holds a key, key c for a lane that
// holds a query row -- and the lane's own token see each other.  The tokens of a sequence lie node
// after node, so the tile's 64 elements are a few runs of one node each: the runs are found with
// one ballot over the node ids (LDS, `ids`: byte address of the 64 ids) and every run is switched
// on as a whole -- for the lane's own node the elements that pass the causal test (`own`), for
// another node n all or nothing by bit n % 64 of `word_of(n)` (word n / 64 of the lane's row or column
// of the visibility matrix).  Elements from n_in on lie behind the end of the sequence.  Called where no operand read
// is in flight (the LDS reads here wait for themselves; the loop branches on wave-uniform values).
template <typename WordOf>
__device__ __forceinline__ uint64_t tile_visibility(uint32_t ids, int lane, uint32_t my_node, uint64_t own, int n_in,
                                                    WordOf&& word_of) {
  uint32_t n_here, n_before;
  asm volatile("ds_read_b32 %0, %2\n\tds_read_b32 %1, %3\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(n_here), "=&v"(n_before)
               : "v"(ids + 4u * (uint32_t)lane), "v"(ids + 4u * (uint32_t)max(lane - 1, 0))
               : "memory");
  uint64_t starts = __builtin_amdgcn_ballot_w64(lane == 0 || n_here != n_before);
  uint64_t m = 0;
  while (starts != 0) {
    const int s0 = __builtin_ctzll(starts);
    starts &= starts - 1;
    const int s1 = starts != 0 ? __builtin_ctzll(starts) : 64;
    const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)n_here, s0);
    const uint64_t run = (s1 == 64 ? ~0ull : (1ull << s1) - 1) & ~((1ull << s0) - 1);
    const uint64_t sel = n == my_node ? own : 0ull - ((word_of(n) >> (n & 63u)) & 1ull);
    m |= run & sel;
  }
  return n_in >= 64 ? m : m & ((1ull << n_in) - 1);
}
// x when bit BIT of the word is set, else 0: the bit as a signed one-bit field (0 or all ones), then
// one AND -- no comparison, no condition register (written out: from the plain expression the
// compiler makes a test, a compare and a select).
template <int BIT>
__device__ __forceinline__ float keep_if_bit(float x, uint32_t word) {
  float r;
  asm("v_bfe_i32 %0, %2, %3, 1\n\tv_and_b32 %0, %0, %1" : "=&v"(r) : "v"(x), "v"(word), "n"(BIT));
  return r;
}

// The score MFMAs of k_bwd_dkv2 written out, with their results in vector registers and the B
// operand (the K / V rows of the wave's keys, fixed for the workgroup) in accumulation registers.
// A kernel with more than 256 registers gets the accumulation-register form for every MFMA the
// compiler selects, and the vector instructions that turn scores into probabilities would first
// have to copy every score out of there; the dK / dV accumulators stay where they are.  The
// compiler does not know what these statements are: the last MFMA of a chain is followed by 20
// idle states, more than the 19 a vector instruction must keep from a 16-pass MFMA whose result
// it reads; a chain's own accumulation is two MFMAs apart (the S and dP chains alternate).
__device__ __forceinline__ f32x16 mfma32_first_v(bf16x8 a, bf16x8 b_acc) {
  f32x16 d;
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b_acc));
  return d;
}
__device__ __forceinline__ f32x16 mfma32_next_v(bf16x8 a, bf16x8 b_acc, f32x16 c) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b_acc));
  return c;
}
__device__ __forceinline__ f32x16 mfma32_last_v(bf16x8 a, bf16x8 b_acc, f32x16 c) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0\n\ts_nop 15\n\ts_nop 3" : "+v"(c) : "v"(a), "v"(b_acc));
  return c;
}

template <int N>
__device__ __forceinline__ void wait_vmcnt_only() {  // s_waitcnt vmcnt(N) (gfx9 encoding)
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
template <int N>
__device__ __forceinline__ void wait_lgkmcnt_only() {
  __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {  // byte address inside LDS of a __shared__ pointer
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}
template <int A, int B, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (A < B) {
    f(std::integral_constant<int, A>{});
    static_for<A + 1, B>(f);
  }
}

// NODES: the query rows come as one compact stream instead of the block map's query tiles: the rows of the nodes
// that see every node of the workgroup's keys (and of the last key's node the rows behind the keys), then
// the rows of the other nodes that see one of them, the keys' own among them, each part in token order,
// gathered row by row.  The tiles made of the first part alone run without tests.  Random DAGs of 4 x 64 nodes of 32 to 256 tokens, 16 / 8 heads of dimension
// 64: 571 us on the block map's tiles, 529 so; 4 x 4608 fork-join, 32 / 8 heads of dimension 128: 1381 -> 1303 us.
template <int D, bool NODES>
__device__ __forceinline__ void dkv_ring_body(const BwdArgs& a) {
  using C = Dkv<D>;
  using R = RingTile<D>;
  constexpr int DB = D / 32, NST = C::NST, LPS = C::LPS, NPB = C::NPB, PF = C::PF, TILEB = C::TILEB, RD = C::RD;
  constexpr int STAGEB = C::STAGEB, HS = C::HS, NSC = C::NSC, NSLOT = C::NSLOT, EPS = C::EPS;
  typedef __attribute__((address_space(3))) void* lds_ptr_t;
  typedef __attribute__((address_space(1))) const void* gbl_ptr_t;
  typedef short v4i16 __attribute__((ext_vector_type(4)));
  typedef short v8i16 __attribute__((ext_vector_type(8)));
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int KIND_WORDS = (MAX_QT_LDS + 63) / 64;
  __shared__ uint8_t sFlag[NODES ? 1 : MAX_QT_LDS];  // block-map column of the pair: flag of tile 0 | flag of tile 1 << 2
  __shared__ uint64_t sKind[2][NODES ? 1 : KIND_WORDS];
  const int hk = blockIdx.x % a.hkv, slot = blockIdx.x / a.hkv;  // heaviest pairs first
  int2 piece = {0, 1 << 16};
  if (NODES && a.pieces) {
    if (slot >= a.n_pieces[0]) return;
    piece = a.pieces[slot];
  } else {
    piece.x = a.kt_order[slot];
  }
  const int kt = piece.x;
  const int b = dag_find_segment(a.ktile_start, a.n_seqs, kt);
  const int ktl = kt - a.ktile_start[b];
  if ((!NODES || !a.block_start) && (ktl & 1)) return;  // the workgroup of the even tile takes the pair
  const int cu = a.cu_seqlens[b], T = a.cu_seqlens[b + 1] - cu;
  const int2 keys = NODES ? dkv_keys(a, kt, ktl, T) : int2{ktl * BN, min((ktl + 2) * BN, T)};
  const int key0 = keys.x, key1 = keys.y;
  const int QT = (T + BM - 1) / BM, KT = (T + BN - 1) / BN;
  const uint8_t* bm = a.block_map + a.block_map_off[b];
  const int nbase = a.node_start[b];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, L = lane & 31, H = lane >> 5;
  const int my_kt = ktl + (w >> 1);
  const int j = key0 + 32 * w + L;  // this lane's key
  const bool key_ok = j < key1;
  const int jc = min(j, key1 - 1);
  const size_t koff = ((size_t)(cu + jc) * a.hkv + hk) * D;
  bf16x8 kf[D / 16], vf[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    kf[s] = *(const bf16x8*)(a.k + koff + 16 * s + 8 * H);
    vf[s] = *(const bf16x8*)(a.v + koff + 16 * s + 8 * H);
    if constexpr (D != 128 || NODES) vf[s] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, vf[s]) ^ 0x80008000u);
  }
  const int nj = a.tok_node[cu + jc];
  // the nodes that see this lane's key: bit ni % 64 of seen_by[ni / 64] = bit nj of node ni's words,
  // i.e. the key's column of the sequence's visibility matrix (the first 128 nodes of it; sequences
  // with more take every word they need from memory)
  uint64_t seen_by[2] = {0, 0};
  // NODES: the stream as runs of consecutive tokens {first position, token - position} (at most 129); its length and that of its first part, its tiles without tests; the position of this lane's key in it
  __shared__ int2 sRun[NODES ? 144 : 1];  // (1152 bytes: the ring behind it stays on a multiple of 128; 16 bytes off it cost 5 %)
  int n_pos = 0, n_first = 0, n_fast = 0, key_pos = 0, n_runs = 0;
  if (NODES || a.W <= 2) {
    const int n_nodes = a.node_start[b + 1] - nbase;
    uint64_t word[2][2];  // word y of node 64 x + lane
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
        word[x][y] = y < a.W && 64 * x + lane < n_nodes ? a.node_vis[(int64_t)(nbase + 64 * x + lane) * a.W + y] : 0;
    uint64_t todo = ~0ull;  // the wave's keys belong to a few nodes: one at a time, its bit of 64 nodes per ballot
    while (todo != 0) {
      const int n = __builtin_amdgcn_readlane(nj, __builtin_ctzll(todo));
      todo &= ~__builtin_amdgcn_ballot_w64(nj == n);
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const uint64_t column = __builtin_amdgcn_ballot_w64(((n < 64 ? word[x][0] : word[x][1]) >> (n & 63)) & 1ull);
        if (nj == n) seen_by[x] = column;
      }
    }
    if constexpr (NODES) {
      const int u0 = a.tok_node[cu + key0], u1 = a.tok_node[cu + key1 - 1];  // the keys' nodes
      // Rows [from, to) of node 64 x + lane in either part.  Of the keys' own nodes the rows in front of the
      // first key see none of them, and those behind the last key what their node sees.
      int from[2][2], to[2][2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const int n = 64 * x + lane;
        const int first = n < n_nodes ? a.node_tok_start[nbase + n] : T, end = n + 1 < n_nodes ? a.node_tok_start[nbase + n + 1] : T;
        // bits u0 .. u1 of the node's words
        uint64_t hit = 0, miss = 0;
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const int lo = max(u0 - 64 * y, 0), hi = min(u1 - 64 * y, 63);
          const uint64_t range = lo <= hi ? (~0ull >> (63 - hi)) & (~0ull << lo) : 0ull;
          hit |= word[x][y] & range;
          miss |= ~word[x][y] & range;
        }
        const int begin = max(first, key0), stop = n < n_nodes && hit != 0 ? end : begin;
        const int split = miss != 0 || n < u1 ? stop : n == u1 ? min(key1, stop) : begin;  // the second part's rows lie in front of it
        from[0][x] = split, to[0][x] = stop;
        from[1][x] = begin, to[1][x] = split;
      }
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        int end_before = -1;  // of the part's last node in the word in front
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const int mine = to[part][x] - from[part][x];
          int incl = mine;
          for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(incl, off);
            if (lane >= off) incl += y;
          }
          const int pos = n_pos + incl - mine;
          n_pos += __builtin_amdgcn_readlane(incl, 63);
          const int my_end = mine > 0 ? to[part][x] : -1;
          int prev = __shfl_up(my_end, 1);
          if (lane == 0) prev = end_before;
          end_before = __builtin_amdgcn_readlane(my_end, 63);
          const uint64_t starts = __builtin_amdgcn_ballot_w64(mine > 0 && prev != from[part][x]);
          const int own = __shfl(pos - from[part][x], nj & 63);
          if (part == 1 && nj >> 6 == x) key_pos = own + jc;
          if (w == 0 && (starts >> lane) & 1)
            sRun[n_runs + __builtin_popcountll(starts & ((1ull << lane) - 1))] = int2{pos, cu + from[part][x] - pos};
          n_runs += __builtin_popcountll(starts);
        }
        if (part == 0) {
          n_first = n_pos;
          n_fast = n_pos / BM;
        }
      }
    }
  }
  auto word_of = [&](uint32_t n) __attribute__((always_inline)) -> uint64_t {  // (n is wave-uniform)
    if (a.W <= 2) return n < 64 ? seen_by[0] : seen_by[1];
    // bit n % 64 = the bit of the key's node in node n's words
    int key_node = nj;
    asm volatile("" : "+v"(key_node));  // (the rare case keeps no address in registers)
    return ((a.node_vis[(int64_t)(nbase + (int)n) * a.W + (key_node >> 6)] >> (key_node & 63)) & 1ull) << (n & 63u);
  };
  f32x16 dK[DB], dV[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) dK[db][e] = dV[db][e] = 0.f;

  // bit 4 of a pair's flags: the iteration runs in the steady-state loop (both key tiles exist, every
  // pair of both is visible, nothing reaches past the end of the sequence)
  auto with_fast_bit = [&](int qt, int f) {
    return f | ((f == (2 | (2 << 2)) && (qt + 1) * BM <= T && (ktl + 2) * BN <= T) ? 16 : 0);
  };
  // Two pipelined loops: the iterations without tests, then the masked ones.
  auto kind_of = [&](int f) { return (f & 16) ? 0 : (f & 15) != 0 ? 1 : 2; };  // 2: nothing to do
  // The column is kept in LDS as the flags and as one bitmap per kind of iteration (bit qt % 64 of
  // word qt / 64: tile qt has a visible pair and is of that kind), so that a walk finds its next
  // tile with one 64-bit read per 64 tiles instead of one probe per tile.
  const bool flags_in_lds = !NODES && QT <= MAX_QT_LDS;
  if (flags_in_lds) {
    for (int x0 = 0; x0 < QT; x0 += 256) {
      const int x = x0 + tid;
      int f = 0;
      if (x < QT) {
        const int f0 = bm[(int64_t)x * KT + ktl];
        const int f1 = ktl + 1 < KT ? bm[(int64_t)x * KT + ktl + 1] : 0;
        f = with_fast_bit(x, f0 | (f1 << 2));
        sFlag[x] = (uint8_t)f;
      }
      const int kind = kind_of(f);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint64_t word = __builtin_amdgcn_ballot_w64(kind == k);
        if (lane == 0 && x0 + 64 * w < QT) sKind[k][(x0 >> 6) + w] = word;
      }
    }
  }
  __syncthreads();
  const uint32_t flag_base = lds_addr(sFlag), kind_base = lds_addr(sKind);
  // (the flags are read with an inline-assembly LDS read that waits for itself: the ring's loads
  // write LDS too, and a compiler-visible LDS read might be made to wait for all of them)
  auto pair_flag = [&](int qt) {
    if (flags_in_lds) {
      uint32_t v;
      asm volatile("ds_read_u8 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(flag_base + (uint32_t)qt) : "memory");
      return __builtin_amdgcn_readfirstlane((int)v);
    }
    const int f0 = bm[(int64_t)qt * KT + ktl];
    const int f1 = ktl + 1 < KT ? bm[(int64_t)qt * KT + ktl + 1] : 0;
    return __builtin_amdgcn_readfirstlane(with_fast_bit(qt, f0 | (f1 << 2)));
  };
  auto kind_word = [&](int kind, int wi) {
    uint64_t v;
    asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(kind_base + (uint32_t)(kind * KIND_WORDS + wi) * 8u) : "memory");
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  };
  auto last_of_kind = [&](int kind, int qt) {  // last query tile <= qt of the kind (with a visible pair), -1 if none
    if (!flags_in_lds) {
      for (; qt >= 0; --qt) {
        if (kind_of(pair_flag(qt)) == kind) break;
      }
      return qt;
    }
    if (qt < 0) return -1;
    int wi = qt >> 6;
    uint64_t word = kind_word(kind, wi) & (~0ull >> (63 - (qt & 63)));
    while (word == 0) {
      if (--wi < 0) return -1;
      word = kind_word(kind, wi);
    }
    return 64 * wi + 63 - __builtin_clzll(word);
  };

  // ---- loads of one stage, in LPS pieces per wave (piece p of (tile qt, head g) into stage st)
  const uint32_t row_stride = (uint32_t)(a.hq * D);  // elements
  const uint32_t chunk8 = R::src_col(lane);  // this lane's 16-byte chunk of a row
  const int rsub = R::src_row(lane);
  // Row data, 4 bytes per lane, one load per wave: wave 0 fetches -lse log2(e), wave 1 delta, wave 2
  // the node ids of the rows (for the masked iterations), wave 3 -lse log2(e) once more (every wave
  // issues the same number of loads, so that the vmcnt waits are the same constants for all).
  // Element index in the source: (token of the row) * rd_mul + head * rd_hmul -- no branch where
  // the loads are issued.
  const float* rd_src = w == 1 ? a.delta : w == 2 ? (const float*)a.tok_node : a.nlse2;
  const int rd_mul = w == 2 ? 1 : a.hq, rd_hmul = w == 2 ? 0 : 1, rd_dst = w == 1 ? 256 : w == 2 ? 512 : 0;
  // The addresses of a stage's loads are prepared once per iteration, outside the slots (wave-uniform
  // bases, four per-lane row offsets, one per-lane row-data pointer); a slot then only sets the LDS
  // destination and issues its load.
  struct IssueCtx {
    const uint16_t *qb, *dob;  // first row of the tile, this head
    uint32_t voff[NPB];        // element offset of this lane's chunk in block w + 4 i (rows past the sequence end re-read its last row)
    const float* rd;           // this lane's row-data word
  };
  // NODES: the tile whose loads are issued next: element offsets of this lane's chunks, the token of its row
  // data, where the tile is in the runs
  uint32_t it_voff[NPB];
  int it_tok = cu, run_at = 0, run_beg = 0, run_d = 0;
  auto run_of = [&](int e) __attribute__((always_inline)) {  // (inline assembly for the reason given at pair_flag)
    uint64_t v;
    asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(lds_addr(sRun) + 8u * (uint32_t)e) : "memory");
    return int2{__builtin_amdgcn_readfirstlane((int)(uint32_t)v), __builtin_amdgcn_readfirstlane((int)(v >> 32))};
  };
  auto enter_run = [&](int e) __attribute__((always_inline)) {
    const int2 run = run_of(e);
    run_at = e;
    run_beg = run.x;
    run_d = run.y;
  };
  // (tiles are entered in descending order, from run n_runs - 1 at the start of a walk)
  auto enter_tile = [&](int n) __attribute__((always_inline)) {
    const int p0 = n * BM, last = min(p0 + BM, n_pos) - 1;
    while (run_beg > last) enter_run(run_at - 1);
    int pos[NPB], tok[NPB];
    const int rd_pos = min(p0 + lane, last);  // (positions past the end re-read the last one and are masked)
    it_tok = rd_pos + run_d;
#pragma unroll
    for (int i = 0; i < NPB; ++i) {
      pos[i] = min(p0 + R::RPB * (w + 4 * i) + rsub, last);
      tok[i] = pos[i] + run_d;
    }
    while (run_beg > p0) {  // (wave-uniform) the tile begins in the run in front
      const int to = run_beg;
      enter_run(run_at - 1);
      it_tok = rd_pos < to ? rd_pos + run_d : it_tok;
#pragma unroll
      for (int i = 0; i < NPB; ++i) tok[i] = pos[i] < to ? pos[i] + run_d : tok[i];
    }
#pragma unroll
    for (int i = 0; i < NPB; ++i) it_voff[i] = (uint32_t)tok[i] * row_stride + chunk8;
  };
  auto prepare_issue = [&](int qt, int g) __attribute__((always_inline)) {
    IssueCtx c;
    if constexpr (NODES) {  // (past the end of the walk: its last tile once more, never consumed)
      const int h = hk * a.G + g;
      c.qb = a.q + h * D;
      c.dob = a.dout + h * D;
#pragma unroll
      for (int i = 0; i < NPB; ++i) c.voff[i] = it_voff[i];
      c.rd = rd_src + ((size_t)it_tok * rd_mul + rd_hmul * h);
      return c;
    }
    const int qv = max(qt, 0);
    const int r0 = qv * BM, n_in = min(BM, T - r0), h = hk * a.G + g;
    const size_t slab = ((size_t)(cu + r0) * a.hq + h) * D;
    c.qb = a.q + slab;
    c.dob = a.dout + slab;
#pragma unroll
    for (int i = 0; i < NPB; ++i) c.voff[i] = (uint32_t)min(R::RPB * (w + 4 * i) + rsub, n_in - 1) * row_stride + chunk8;
    c.rd = rd_src + ((size_t)(cu + r0 + min(lane, n_in - 1)) * rd_mul + rd_hmul * h);
    return c;
  };
  auto issue_piece = [&](int p, const IssueCtx& c, int st) __attribute__((always_inline)) {
    unsigned char* const sb = smem + st * STAGEB;
    if (p < 2 * NPB) {
      const int blk = w + 4 * (p % NPB);
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)((p < NPB ? c.qb : c.dob) + c.voff[p % NPB]),
                                       (lds_ptr_t)(sb + (p < NPB ? 0 : TILEB) + blk * R::BLK), 16, 0, 0);
    } else {
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)c.rd, (lds_ptr_t)(sb + RD + rd_dst), 4, 0, 0);
    }
  };
  auto sync_mid = [&]() __attribute__((always_inline)) {
    wait_vmcnt_only<LPS>();        // this wave's loads of the next iteration's stage have landed
    __builtin_amdgcn_s_barrier();  // (bare: a __syncthreads would drain the loads in flight)
    asm volatile("" ::: "memory");
  };

  // per-lane parts of the LDS operand addresses
  const uint32_t roff[2] = {R::row_lane(L, H, 0), R::row_lane(L, H, 1)};
  const uint32_t toff = R::tr_lane(lane);
  const uint32_t smem_base = lds_addr(smem);
  const float sc = a.sc;

  // ---- the iteration without tests, slot by slot
  // (with masks: vis_lo / vis_hi = this lane's visibility word of the tile, shifted so that bit
  // 32 h + 8 (e / 4) + e % 4 belongs to element e of half h, i.e. to row 64 qt + 4 H + that number)
  auto pipelined_iter = [&](auto msk_c, int cs, const IssueCtx& ictx, int is, uint32_t vis_lo, uint32_t vis_hi) __attribute__((always_inline)) {
    constexpr bool MSK = decltype(msk_c)::value;
    const uint32_t sbase = smem_base + (uint32_t)cs * STAGEB;
    const uint32_t ra[2] = {sbase + roff[0], D == 128 ? sbase + roff[0] + 32 : sbase + roff[1]};
    const uint32_t ta = sbase + toff, va = sbase + RD + 16 * H;
    bf16x8 op[NSLOT];
    v4i16 lo[NSLOT], hi[NSLOT];
    f32x4 nl[2][4], dl[2][4];
    f32x16 S[2], dP[2];
    float pt[2][16], dt[2][16];
    bf16x8 pp[2][2], dss[2][2];
    // row data of rows 32 h + 8 x + 4 H .. + 3: -lse, delta, node ids
    auto fetch_val = [&](auto hc, auto xc) __attribute__((always_inline)) {
      constexpr int h = decltype(hc)::value, x = decltype(xc)::value;
      const uint32_t v = va;  // (named here: captures inside discarded branches trip the compiler)
      f32x4(*const nlp)[4] = nl;
      f32x4(*const dlp)[4] = dl;
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(nlp[h][x]) : "v"(v), "n"(128 * h + 32 * x));
      if constexpr (D == 128) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dlp[h][x]) : "v"(v), "n"(256 + 128 * h + 32 * x));
    };
    auto fetch_delta = [&](auto hc) __attribute__((always_inline)) {
      constexpr int h = decltype(hc)::value, at = 256 + 128 * h;
      f32x4(*const dlp)[4] = dl;
      const uint32_t v = va;
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dlp[h][0]) : "v"(v), "n"(at));
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dlp[h][1]) : "v"(v), "n"(at + 32));
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dlp[h][2]) : "v"(v), "n"(at + 64));
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dlp[h][3]) : "v"(v), "n"(at + 96));
    };
    auto fetch = [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      constexpr int odd = ((i % HS) / 2) & 1;  // (k-step of a row operand)
      const uint32_t r = D == 128 ? ra[0] : ra[odd], t = ta;
      bf16x8* const opp = op;
      v4i16* const lop = lo;
      v4i16* const hip_ = hi;
      if constexpr (i < NSC)
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(opp[i]) : "v"(r), "n"(C::row_imm(i) + (D == 128 ? 32 * odd : 0)));
      else if constexpr (i < NSLOT)
        asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                     : "=&v"(lop[i]), "=&v"(hip_[i])
                     : "v"(t), "n"(C::tr_imm(i, 0)), "n"(C::tr_imm(i, 1)));
    };
    if constexpr (D != 128) fetch_delta(std::integral_constant<int, 0>{});
    static_for<0, PF>(fetch);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NSLOT>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      if constexpr (D != 128 && i == C::DELTA_SLOT) fetch_delta(std::integral_constant<int, 1>{});
      if constexpr (i == NSC) {
        sync_mid();
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (C::row_reads(i) != 0) {
        constexpr int u = (i + C::VAHEAD - HS) / (4 / EPS);  // rows 4 u .. 4 u + 3 of the 64
        fetch_val(std::integral_constant<int, u / 4>{}, std::integral_constant<int, u % 4>{});
      }
      fetch(std::integral_constant<int, i + PF>{});
      wait_lgkmcnt_only<C::wait_at(i)>();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (i < NSC) {
        constexpr int rb = i / HS, s = (i % HS) / 2;
        const bf16x8 b_acc = (i & 1) == 0 ? kf[s] : vf[s];
        f32x16& acc = (i & 1) == 0 ? S[rb] : dP[rb];
        if constexpr (D != 128) {
          const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
          const f32x4* const c = dl[rb];
          const f32x16 from = {c[0][0], c[0][1], c[0][2], c[0][3], c[1][0], c[1][1], c[1][2], c[1][3], c[2][0], c[2][1], c[2][2], c[2][3], c[3][0], c[3][1], c[3][2], c[3][3]};
          acc = mfma32(op[i], b_acc, s > 0 ? acc : (i & 1) == 0 ? zero : from);
        } else if constexpr (s == 0)
          acc = mfma32_first_v(op[i], b_acc);
        else if constexpr (s < D / 16 - 1)
          acc = mfma32_next_v(op[i], b_acc, acc);
        else
          acc = mfma32_last_v(op[i], b_acc, acc);
      } else {
        constexpr int jx = i - NSC, h = jx / HS, jj = jx % HS, db = jj / 4, hh = (jj / 2) % 2;
        const v8i16 x = {lo[i][0], lo[i][1], lo[i][2], lo[i][3], hi[i][0], hi[i][1], hi[i][2], hi[i][3]};
        const bf16x8 opx = __builtin_bit_cast(bf16x8, x);
        if constexpr ((jj & 1) == 0)
          dV[db] = mfma32(opx, pp[h][hh], dV[db]);
        else
          dK[db] = mfma32(opx, dss[h][hh], dK[db]);
      }
      if constexpr (i >= NSC && i < NSC + LPS) issue_piece(i - NSC, ictx, is);
      if constexpr (i >= HS && i < 3 * HS) static_for<EPS * (i - HS), EPS * (i - HS) + EPS>([&](auto nc) __attribute__((always_inline)) {  // scores of half 0, then of half 1
        constexpr int h = decltype(nc)::value / 16, e = decltype(nc)::value % 16;
        float pe = __builtin_amdgcn_exp2f(fmaf(S[h][e], sc, nl[h][e >> 2][e & 3]));
        if constexpr (MSK) pe = keep_if_bit<8 * (e >> 2) + (e & 3)>(pe, h == 0 ? vis_lo : vis_hi);  // Eq. 3 and the end of the sequence
        pt[h][e] = pe;
        dt[h][e] = D == 128 ? pe * (dP[h][e] - dl[h][e >> 2][e & 3]) : pe * -dP[h][e];  // (V is negated)
        if constexpr ((e & 1) == 1) {
          const uint32_t pw = dag_pack_bf2(pt[h][e - 1], pt[h][e]), dw = dag_pack_bf2(dt[h][e - 1], dt[h][e]);
          typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
          const bf16x2 pb = __builtin_bit_cast(bf16x2, pw), db2 = __builtin_bit_cast(bf16x2, dw);
          pp[h][e >> 3][(e & 7) - 1] = pb[0];
          pp[h][e >> 3][e & 7] = pb[1];
          dss[h][e >> 3][(e & 7) - 1] = db2[0];
          dss[h][e >> 3][e & 7] = db2[1];
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // ---- The iteration of streams at head dimension 128, turned: a tile's two halves of 32 rows half an iteration apart, so that every
  // slot has an MFMA and half an element of the exponentials.  One wave has its SIMD to itself, and what does not fit
  // between two MFMAs (32 clocks) adds to the iteration: with all exponentials in the middle 32 of the 64 slots (pipelined_iter) those slots
  // were too full and the others idle.  Quarters of 16 slots: scores of half 1 of this tile; dV / dK of half 0; scores
  // of half 0 of the next tile; dV / dK of half 1.  The exponentials of half 1 start TURN_GAP slots behind its scores, those of the next
  // tile's half 0 likewise, and so run over into the next iteration (with masks what is done of them then waits for the
  // next tile's word and is packed behind it).  In the gap more instructions issue than the 19 wait states between the last
  // MFMA of a chain and a vector instruction that reads its result, so that the scores need no idle states (20 behind each
  // chain, 60 us of 1170); dV / dK take the rows 0 .. 15 of a half first.
  struct Turned {
    f32x16 S[2], dP[2];
    float pt[2][16], dt[2][16];
    bf16x8 pp[2][2], dss[2][2];
    f32x4 nl[2][4], dl[2][4];
  };
  auto turned_score = [&](Turned& t, auto hc, auto ec) __attribute__((always_inline)) {  // row element e of half h: P
    constexpr int h = decltype(hc)::value, e = decltype(ec)::value;
    t.pt[h][e] = __builtin_amdgcn_exp2f(fmaf(t.S[h][e], sc, t.nl[h][e >> 2][e & 3]));
  };
  auto turned_pack = [&](Turned& t, auto hc, auto ec) __attribute__((always_inline)) {  // ... elements e - 1 and e
    constexpr int h = decltype(hc)::value, e = decltype(ec)::value;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    const bf16x2 pb = __builtin_bit_cast(bf16x2, dag_pack_bf2(t.pt[h][e - 1], t.pt[h][e])), db2 = __builtin_bit_cast(bf16x2, dag_pack_bf2(t.dt[h][e - 1], t.dt[h][e]));
    t.pp[h][e >> 3][(e & 7) - 1] = pb[0];
    t.pp[h][e >> 3][e & 7] = pb[1];
    t.dss[h][e >> 3][(e & 7) - 1] = db2[0];
    t.dss[h][e >> 3][e & 7] = db2[1];
  };
  auto turned_rows = [&](Turned& t, uint32_t base, auto hc, auto xc) __attribute__((always_inline)) {  // row data of rows 32 h + 8 x + 4 H .. + 3
    constexpr int h = decltype(hc)::value, x = decltype(xc)::value;
    f32x4(*const nlp)[4] = t.nl;
    const uint32_t v = base;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(nlp[h][x]) : "v"(v), "n"(128 * h + 32 * x));
  };
  auto turned_delta = [&](Turned& t, uint32_t base, auto hc) __attribute__((always_inline)) {  // delta of the rows of half h
    constexpr int h = decltype(hc)::value, at = 256 + 128 * h;
    f32x4* const to = t.dl[h];
    const uint32_t v = base;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(to[0]) : "v"(v), "n"(at));
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(to[1]) : "v"(v), "n"(at + 32));
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(to[2]) : "v"(v), "n"(at + 64));
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(to[3]) : "v"(v), "n"(at + 96));
  };
  auto turned_first_dp = [&](Turned& t, bf16x8 op, auto hc) __attribute__((always_inline)) {
    const f32x4* const c = t.dl[decltype(hc)::value];
    const f32x16 from = {c[0][0], c[0][1], c[0][2], c[0][3], c[1][0], c[1][1], c[1][2], c[1][3], c[2][0], c[2][1], c[2][2], c[2][3], c[3][0], c[3][1], c[3][2], c[3][3]};
    return mfma32_next_v(op, vf[0], from);
  };
  auto turned_iter = [&](auto msk_c, Turned& t, int cs, const IssueCtx& ictx, int is, uint32_t vis_lo, uint32_t vis_hi) __attribute__((always_inline)) {
    constexpr bool MSK = decltype(msk_c)::value;
    const uint32_t sbase = smem_base + (uint32_t)cs * STAGEB, nbase_ = smem_base + (uint32_t)(cs + 1 == NST ? 0 : cs + 1) * STAGEB;
    const uint32_t ra = sbase + roff[0], rn = nbase_ + roff[0], ta = sbase + toff, va = sbase + RD + 16 * H, vn = nbase_ + RD + 16 * H;
    bf16x8 op[NSLOT];
    v4i16 lo[NSLOT], hi[NSLOT];
    auto fetch = [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      const uint32_t r = i < 32 ? ra : rn, tt = ta;
      bf16x8* const opp = op;
      v4i16* const lop = lo;
      v4i16* const hip_ = hi;
      if constexpr (i < NSLOT) {
        if constexpr (C::turned_row(i)) {
          constexpr int o = i < 16 ? HS + i : i - 32;  // half 1 of this tile, half 0 of the next
          asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(opp[i]) : "v"(r), "n"(C::row_imm(o) + 32 * (((o % HS) / 2) & 1)));
        } else {
          constexpr int r = i % 16, o = NSC + (i < 32 ? 0 : HS) + r % 8 / 2 * 4 + r / 8 * 2 + (r & 1);
          asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                       : "=&v"(lop[i]), "=&v"(hip_[i])
                       : "v"(tt), "n"(C::tr_imm(o, 0)), "n"(C::tr_imm(o, 1)));
        }
      }
    };
    turned_delta(t, va, std::integral_constant<int, 1>{});
    static_for<0, PF>(fetch);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NSLOT>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value, q = i / 16, r = i % 16;
      constexpr int ISSUE = C::TURN_SYNC;
      if constexpr (i == ISSUE) {
        sync_mid();
        __builtin_amdgcn_sched_barrier(0);
        turned_delta(t, vn, std::integral_constant<int, 0>{});
      }
      if constexpr (i % 8 == C::TURN_GAP) {
        constexpr int x = (i / 8 + 3) % 4, h = i < 8 || i > 40 ? 0 : 1;  // used eight slots later
        turned_rows(t, i > 40 ? vn : va, std::integral_constant<int, h>{}, std::integral_constant<int, x>{});
      }
      fetch(std::integral_constant<int, i + PF>{});
      wait_lgkmcnt_only<C::turned_wait(i)>();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (C::turned_row(i)) {
        constexpr int h = q == 0 ? 1 : 0, s = r / 2;
        const bf16x8 b_acc = (r & 1) == 0 ? kf[s] : vf[s];
        f32x16& acc = (r & 1) == 0 ? t.S[h] : t.dP[h];
        if constexpr (r == 0)
          acc = mfma32_first_v(op[i], b_acc);
        else if constexpr (r == 1)
          acc = turned_first_dp(t, op[i], std::integral_constant<int, h>{});
        else
          acc = mfma32_next_v(op[i], b_acc, acc);
      } else {
        constexpr int h = q == 1 ? 0 : 1, db = r % 8 / 2, hh = r / 8;
        const v8i16 x = {lo[i][0], lo[i][1], lo[i][2], lo[i][3], hi[i][0], hi[i][1], hi[i][2], hi[i][3]};
        const bf16x8 opx = __builtin_bit_cast(bf16x8, x);
        if constexpr ((r & 1) == 0)
          dV[db] = mfma32(opx, t.pp[h][hh], dV[db]);
        else
          dK[db] = mfma32(opx, t.dss[h][hh], dK[db]);
      }
      if constexpr (i >= ISSUE && i < ISSUE + LPS) issue_piece(i - ISSUE, ictx, is);
      {  // an element every two slots: P, then dS (and the pair's packing)
        constexpr int j = (i + 16 - C::TURN_GAP) % NSLOT, h = j / 32, e = j / 2 % 16;
        constexpr int LATE = 8 - C::TURN_GAP / 2;  // elements of half 0 that the iteration in front has done
        std::integral_constant<int, h> hc;
        std::integral_constant<int, e> ec;
        if constexpr (j % 2 == 0) {
          turned_score(t, hc, ec);
          if constexpr (MSK && i < 48 + C::TURN_GAP) t.pt[h][e] = keep_if_bit<8 * (e >> 2) + (e & 3)>(t.pt[h][e], h == 0 ? vis_lo : vis_hi);
        } else {
          t.dt[h][e] = t.pt[h][e] * -t.dP[h][e];
          if constexpr (e % 2 == 1 && !(MSK && i >= 48 + C::TURN_GAP)) turned_pack(t, hc, ec);
        }
        if constexpr (MSK && i < 2 * LATE) {
          constexpr int e0 = i / 2;
          float& x = i % 2 == 0 ? t.pt[0][e0] : t.dt[0][e0];
          x = keep_if_bit<8 * (e0 >> 2) + (e0 & 3)>(x, vis_lo);
          if constexpr (i % 4 == 3) turned_pack(t, std::integral_constant<int, 0>{}, std::integral_constant<int, e0>{});
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // What the first iteration of a walk finds done: the last half of an iteration on the tile in stage cs.
  auto turned_start = [&](auto msk_c, Turned& t, int cs) __attribute__((always_inline)) {
    const uint32_t sbase = smem_base + (uint32_t)cs * STAGEB, r = sbase + roff[0], va = sbase + RD + 16 * H;
    static_for<0, 3>([&](auto xc) __attribute__((always_inline)) { turned_rows(t, va, std::integral_constant<int, 0>{}, xc); });
    turned_delta(t, va, std::integral_constant<int, 0>{});
    static_for<0, HS>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value, s = i / 2;
      bf16x8 op;
      asm volatile("ds_read_b128 %0, %1 offset:%2\n\ts_waitcnt lgkmcnt(0)" : "=v"(op) : "v"(r), "n"(C::row_imm(i) + 32 * (s & 1)));
      const bf16x8 b_acc = (i & 1) == 0 ? kf[s] : vf[s];
      f32x16& acc = (i & 1) == 0 ? t.S[0] : t.dP[0];
      if constexpr (i == 0)
        acc = mfma32_first_v(op, b_acc);
      else if constexpr (i == 1)
        acc = turned_first_dp(t, op, std::integral_constant<int, 0>{});
      else if constexpr (s < D / 16 - 1)
        acc = mfma32_next_v(op, b_acc, acc);
      else
        acc = mfma32_last_v(op, b_acc, acc);
    });
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, 8 - C::TURN_GAP / 2>([&](auto ec) __attribute__((always_inline)) {
      constexpr int e = decltype(ec)::value;
      turned_score(t, std::integral_constant<int, 0>{}, ec);
      t.dt[0][e] = t.pt[0][e] * -t.dP[0][e];
      if constexpr (e % 2 == 1 && !decltype(msk_c)::value) turned_pack(t, std::integral_constant<int, 0>{}, ec);
    });
  };

  // ---- the walk of one kind of iteration: query tiles from the last one down (as do the other workgroups of the
  // KV head: they share the rows of the sequence's end in L2), the heads of the group inside
  const int n_tiles = (n_pos + BM - 1) / BM, cuts = piece.y >> 16, cut = piece.y & 0xffff;  // (NODES)
  const int tile0 = cut * (n_tiles / cuts) + min(cut, n_tiles % cuts), tile1 = tile0 + n_tiles / cuts + (cut < n_tiles % cuts);
  auto ring_loop = [&](auto msk_c) __attribute__((always_inline)) {
    constexpr int KIND = decltype(msk_c)::value ? 1 : 0;
    const int n0 = KIND == 0 ? tile0 : max(tile0, n_fast), n1 = KIND == 0 ? min(tile1, n_fast) : tile1;  // (NODES)
    auto next_tile = [&](int qt) { return last_of_kind(KIND, qt); };
    auto advance = [&](int& qt, int& g) {
      if constexpr (NODES) {
        if (++g == a.G) {
          g = 0;
          if (--qt >= n0) enter_tile(qt);
        }
        return;
      }
      if (qt < 0) return;
      if (++g == a.G) {
        g = 0;
        qt = next_tile(qt - 1);
      }
    };
    int cq = NODES ? n1 - 1 : next_tile(QT - 1);  // the tile being computed
    if (NODES ? n0 >= n1 : cq < 0) return;
    if constexpr (NODES) {
      enter_run(n_runs - 1);
      enter_tile(cq);
    }
    int iq = cq, ig = 0;                 // the iteration whose loads are issued next
#pragma unroll 1
    for (int st = 0; st < NST - 1; ++st) {
      const IssueCtx c = prepare_issue(iq, ig);
#pragma unroll
      for (int p = 0; p < LPS; ++p) issue_piece(p, c, st);
      advance(iq, ig);
    }
    wait_vmcnt_only<(NST - 2) * LPS>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    int cs = 0, is = NST - 1;
    constexpr bool TURNED = D == 128 && NODES;
    Turned t;
    if constexpr (TURNED) turned_start(msk_c, t, cs);
    // (register classes, at the top of every iteration: the dK / dV accumulators stay in the
    // accumulation registers over the whole loop; without the hint the allocator moves three of
    // the eight back and forth every iteration)
    while (NODES ? cq >= n0 : cq >= 0) {  // one query tile: (with masks) its visibility word once, then an iteration per head
      bool active = !NODES || key0 + 32 * w < key1;  // a visible pair in this wave's key tile (tiles without tests: a lane past the last key computes what nobody stores)
      uint64_t vis = 0;
      if constexpr (KIND == 1 && NODES) {
        const int at = key_pos - cq * BM;  // the key's own row in the tile: the rows of its node see it from there on
        const int sure = n_first - cq * BM;    // rows of the first part: every key sees them
        const uint64_t own = (at <= 0 ? ~0ull : at >= 64 ? 0ull : ~0ull << at) | (sure >= 64 ? ~0ull : sure <= 0 ? 0ull : (1ull << sure) - 1);
        vis = tile_visibility(smem_base + (uint32_t)cs * STAGEB + RD + 512, lane, (uint32_t)nj, own, n_pos - cq * BM, word_of);
        active = __builtin_amdgcn_ballot_w64(key_ok && vis != 0) != 0;
        vis = key_ok ? vis >> (4 * H) : 0ull;
      } else if constexpr (KIND == 1) {
        active = ((pair_flag(cq) >> (2 * (w >> 1))) & 3) != 0;
        if (active) {
          // the rows of tile cq that this lane's key is visible to: own node from the key's row on
          const int first = j - cq * BM;  // first such row of the tile (may lie before or behind it)
          const uint64_t own = first <= 0 ? ~0ull : first >= 64 ? 0ull : ~0ull << first;
          vis = tile_visibility(smem_base + (uint32_t)cs * STAGEB + RD + 512, lane, (uint32_t)nj, own, T - cq * BM, word_of);
          vis = key_ok ? vis >> (4 * H) : 0ull;  // bit 32 h + 8 (e / 4) + e % 4: element e of half h
        }
      }
#pragma unroll 1
      for (int g = 0; g < a.G; ++g) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
          if constexpr (D == 128) asm volatile("" : "+a"(dK[db]), "+a"(dV[db]));
        const IssueCtx ic = prepare_issue(iq, ig);
        if constexpr (TURNED) {  // (a wave to a SIMD: those that have nothing to do wait for the others either way)
          turned_iter(msk_c, t, cs, ic, is, (uint32_t)vis, (uint32_t)(vis >> 32));
        } else if ((KIND == 0 && !NODES) || active) {
          pipelined_iter(msk_c, cs, ic, is, (uint32_t)vis, (uint32_t)(vis >> 32));
        } else {  // only the ring's business
          sync_mid();
#pragma unroll
          for (int p = 0; p < LPS; ++p) issue_piece(p, ic, is);
        }
        advance(iq, ig);
        cs = cs + 1 == NST ? 0 : cs + 1;
        is = is + 1 == NST ? 0 : is + 1;
      }
      cq = NODES ? cq - 1 : next_tile(cq - 1);
    }
    wait_vmcnt_only<0>();  // (the loads past the end of the walk)
    __builtin_amdgcn_s_barrier();  // every wave is done with the ring before the next loop refills it
    asm volatile("" ::: "memory");
  };
  ring_loop(std::false_type{});
  ring_loop(std::true_type{});
  int key = 32 * w + L;
  asm volatile("" : "+v"(key));  // (recomputed here: its offsets need no registers across the loops)
  const int j_out = key0 + key;
  if (NODES && cuts > 1) {
    f32x4* to = a.part + ((size_t)(slot * a.hkv + hk) * 4 + w) * (8 * DB * 64) + lane;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        to[(4 * db + e4) * 64] = f32x4{dK[db][4 * e4], dK[db][4 * e4 + 1], dK[db][4 * e4 + 2], dK[db][4 * e4 + 3]};
        to[(4 * DB + 4 * db + e4) * 64] = f32x4{dV[db][4 * e4], dV[db][4 * e4 + 1], dV[db][4 * e4 + 2], dV[db][4 * e4 + 3]};
      }
    return;
  }
  dkv_store<D>(a, ((size_t)(cu + min(j_out, T - 1)) * a.hkv + hk) * D, j_out < key1, H, dK, dV);
  if constexpr (NODES) {  // sums that are not numbers: k_dkv_finish looks into it
    float any = 0.f;  // (maximum, unlike fmaxf, hands a NaN on)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int e = 0; e < 16; ++e) any = __builtin_elementwise_maximum(__builtin_elementwise_maximum(dK[db][e], dV[db][e]), any);
    if (j_out < key1 && any != any) a.kt_again[kt] = 1;
  }
}
__global__ void __launch_bounds__(256) k_bwd_dkv2(BwdArgs a) { dkv_ring_body<128, false>(a); }
__global__ void __launch_bounds__(256, 2) k_bwd64_dkv(BwdArgs a) { dkv_ring_body<64, false>(a); }
__global__ void __launch_bounds__(256) k_nodes_dkv2(BwdArgs a) { dkv_ring_body<128, true>(a); }
__global__ void __launch_bounds__(256, 2) k_nodes64_dkv(BwdArgs a) { dkv_ring_body<64, true>(a); }

// Behind the streams: their masked tiles multiply a hidden row's Q and dO by zero, and 0 x Inf or NaN is NaN.  A
// wave of a workgroup whose sums are not numbers, and whose keys some row that is not finite does not see (at
// least one of them), takes its keys again, row by row with nothing but the visible ones, until no number is
// left.  A kernel of its own, because the streams have no register left for it (a few of them spilled, in the
// loop, wherever this went); with nothing to do it takes 4.5 us of 890 (4 x 64 random nodes, 16 / 8 heads of dimension 64).
template <int D>
__device__ void dkv_again(const BwdArgs& a, int kt, int hk, int w) {
  const int b = dag_find_segment(a.ktile_start, a.n_seqs, kt);
  const int cu = a.cu_seqlens[b], T = a.cu_seqlens[b + 1] - cu, nbase = a.node_start[b];
  const int lane = threadIdx.x & 63, H = lane >> 5;
  const int2 keys = dkv_keys(a, kt, kt - a.ktile_start[b], T);
  const int j0 = keys.x + 32 * w, j = j0 + (lane & 31), jc = min(j, keys.y - 1);
  if (j0 >= keys.y) return;
  const bool key_ok = j < keys.y;
  const int node = a.tok_node[cu + jc], u0 = a.tok_node[cu + j0], j1 = min(j0 + 31, keys.y - 1), u1 = a.tok_node[cu + j1];
  auto sees = [&](int ni, int u) { return ((a.node_vis[(int64_t)(nbase + ni) * a.W + (u >> 6)] >> (u & 63)) & 1) != 0; };
  bool suspect = false;
  for (int i0 = keys.x; i0 < T && !suspect; i0 += 64) {  // a row per lane
    const int i = min(i0 + lane, T - 1), ni = a.tok_node[cu + i];
    bool all = i >= j1;
    for (int u = u0; u <= u1; ++u) all = all && sees(ni, u);
    bool bad = false;
    if (!all)
      for (int g = 0; g < a.G; ++g) {
        const size_t row = (size_t)(cu + i) * a.hq + hk * a.G + g;
        bad |= dag_row_not_finite<D>(a.q + row * D) || dag_row_not_finite<D>(a.dout + row * D) || !(fabsf(a.nlse2[row]) < INFINITY) ||
               !(fabsf(a.delta[row]) < INFINITY);
      }
    suspect = __builtin_amdgcn_ballot_w64(bad) != 0;
  }
  if (!suspect) return;
  f32x16 dK[D / 32], dV[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) dK[db][e] = dV[db][e] = 0.f;
  const size_t koff = ((size_t)(cu + jc) * a.hkv + hk) * D;
#pragma unroll 1
  for (int i = j0; i < T; ++i) {
    const int ni = a.tok_node[cu + i];
    const bool ok = key_ok && (ni == node ? j <= i : sees(ni, node));
    bool number = false;
#pragma unroll 1
    for (int g = 0; g < a.G; ++g) {
      const size_t row = (size_t)(cu + i) * a.hq + hk * a.G + g;
      const uint16_t *qp = a.q + row * D, *dop = a.dout + row * D;
      float s = 0.f, dp = 0.f;
#pragma unroll
      for (int x = 0; x < D / 16; ++x) {
        const u32x4 qr = *(const u32x4*)(qp + 16 * x + 8 * H), dr = *(const u32x4*)(dop + 16 * x + 8 * H);
        const u32x4 kr = *(const u32x4*)(a.k + koff + 16 * x + 8 * H), vr = *(const u32x4*)(a.v + koff + 16 * x + 8 * H);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s = fmaf(dag_bf_hi(kr[e]), dag_bf_hi(qr[e]), fmaf(dag_bf_lo(kr[e]), dag_bf_lo(qr[e]), s));
          dp = fmaf(dag_bf_hi(vr[e]), dag_bf_hi(dr[e]), fmaf(dag_bf_lo(vr[e]), dag_bf_lo(dr[e]), dp));
        }
      }
      s += __shfl_xor(s, 32);
      dp += __shfl_xor(dp, 32);
      const float pe = __builtin_amdgcn_exp2f(fmaf(s, a.sc, a.nlse2[row])), ds = pe * (dp - a.delta[row]);
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {  // dimensions 32 db + 8 e4 + 4 H .. + 3
          const u32x2 qr = *(const u32x2*)(qp + 32 * db + 8 * e4 + 4 * H), dr = *(const u32x2*)(dop + 32 * db + 8 * e4 + 4 * H);
          const float q4[4] = {dag_bf_lo(qr[0]), dag_bf_hi(qr[0]), dag_bf_lo(qr[1]), dag_bf_hi(qr[1])};
          const float d4[4] = {dag_bf_lo(dr[0]), dag_bf_hi(dr[0]), dag_bf_lo(dr[1]), dag_bf_hi(dr[1])};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float k0 = dK[db][4 * e4 + e], v0 = dV[db][4 * e4 + e];
            const float k1 = ok ? fmaf(ds, q4[e], k0) : k0, v1 = ok ? fmaf(pe, d4[e], v0) : v0;
            dK[db][4 * e4 + e] = k1;
            dV[db][4 * e4 + e] = v1;
            number |= k1 == k1 || v1 == v1;
          }
        }
    }
    if (__builtin_amdgcn_ballot_w64(key_ok && number) == 0) break;
  }
  dkv_store<D>(a, koff, key_ok, H, dK, dV);
}
// The workgroups behind those of the key tiles add up the pieces of the split pairs, in the order of the stream (32 keys
// each, dK and dV in four parts).
template <int D>
__global__ void __launch_bounds__(256) k_dkv_finish(BwdArgs a) {
  constexpr int NR = D / 16;  // sums of four dimensions that a lane adds up
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, L = lane & 31, H = lane >> 5;
  int kt = blockIdx.x, hk = 0, hk_end = a.hkv, group = w;
  if (kt < a.total_ktiles) {
    if (!a.again || a.kt_again[kt] == 0) return;
  } else {
    const int x = blockIdx.x - a.total_ktiles, pair = (x >> 2) / a.hkv;
    group = x & 3;
    hk = (x >> 2) % a.hkv;
    hk_end = hk + 1;
    if (pair >= a.n_pieces[1]) return;
    const int slot = a.split_first[pair];
    const int2 piece = a.pieces[slot];
    kt = piece.x;
    const int n = piece.y >> 16;
    const size_t step = (size_t)a.hkv * 4 * (D / 4 * 64);
    const f32x4* from = a.part + ((size_t)(slot * a.hkv + hk) * 4 + group) * (D / 4 * 64) + w * NR * 64 + lane;
    f32x4 sum[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) sum[r] = from[r * 64];
#pragma unroll 4
    for (int p = 1; p < n; ++p) {
      from += step;
#pragma unroll
      for (int r = 0; r < NR; ++r) sum[r] += from[r * 64];
    }
    const int b = dag_find_segment(a.ktile_start, a.n_seqs, kt);
    const int cu = a.cu_seqlens[b], T = a.cu_seqlens[b + 1] - cu;
    const int2 keys = dkv_keys(a, kt, kt - a.ktile_start[b], T);
    const int j = keys.x + 32 * group + L;
    const float scale = w < 2 ? a.scale : 1.f;
    uint16_t* to = (w < 2 ? a.dk : a.dv) + ((size_t)(cu + min(j, T - 1)) * a.hkv + hk) * D + (w & 1) * (D / 2) + 4 * H;
    bool bad = false;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      bad |= j < keys.y && (sum[r][0] != sum[r][0] || sum[r][1] != sum[r][1] || sum[r][2] != sum[r][2] || sum[r][3] != sum[r][3]);
      const u32x2 o = {dag_pack_bf2(sum[r][0] * scale, sum[r][1] * scale), dag_pack_bf2(sum[r][2] * scale, sum[r][3] * scale)};
      if (j < keys.y) *(u32x2*)(to + 8 * r) = o;
    }
    if (!__syncthreads_or(bad) || !a.again || w != 0) return;
  }
  for (; hk < hk_end; ++hk) dkv_again<D>(a, kt, hk, group);
}

// Tile lists of the dQ workgroups that take one query head on a group of NQ = four (head dimension
// 128) or two query tiles (the heads that do not fill a workgroup on one tile): one wave per query
// tile of the batch, those of every NQ-th tile of a sequence work.  The list of tiles NQ c ..
// NQ c + NQ - 1 holds every key tile that one of them sees; the key tiles that all of them see in full, with all their rows and keys inside the sequence, come
// first (they run without tests), both parts ascending.
template <int NQ>
__device__ void bwd_wide_rows(const BwdArgs& a, int x, int lane) {
  const int b = dag_find_segment(a.qtile_start, a.n_seqs, x);
  const int qt = x - a.qtile_start[b];
  if (qt % NQ) return;
  const int T = a.cu_seqlens[b + 1] - a.cu_seqlens[b];
  const int QT = (T + BM - 1) / BM, KT = (T + BN - 1) / BN;
  const uint8_t* bm = a.block_map + a.block_map_off[b];
  const int64_t base = a.block_map_off[b] + (int64_t)qt * KT;
  const bool rows_in = (qt + NQ) * BM <= T;
  constexpr int ALL_FULL = 0xAA >> (8 - 2 * NQ);
  auto entries = [&](int kt) {
    int f8 = 0;
    if (kt < KT)
      for (int i = 0; i < NQ; ++i)
        if (qt + i < QT) f8 |= (int)bm[(int64_t)(qt + i) * KT + kt] << (2 * i);
    return f8;
  };
  int n = 0, nfast = 0;
  for (int k0 = 0; k0 < KT; k0 += 64) {
    const int kt = k0 + lane, f8 = entries(kt);
    nfast += __builtin_popcountll(__builtin_amdgcn_ballot_w64(rows_in && f8 == ALL_FULL && (kt + 1) * BN <= T));
    n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(f8 != 0));
  }
  int at_fast = 0, at_rest = nfast;
  const uint64_t below = (1ull << lane) - 1;
  for (int k0 = 0; k0 < KT; k0 += 64) {
    const int kt = k0 + lane, f8 = entries(kt);
    const bool fast = rows_in && f8 == ALL_FULL && (kt + 1) * BN <= T, rest = f8 != 0 && !fast;
    const uint64_t mf = __builtin_amdgcn_ballot_w64(fast), mr = __builtin_amdgcn_ballot_w64(rest);
    if (fast || rest) {
      const int64_t at = base + (fast ? at_fast + __builtin_popcountll(mf & below) : at_rest + __builtin_popcountll(mr & below));
      a.wide_col[at] = kt;
    }
    at_fast += __builtin_popcountll(mf);
    at_rest += __builtin_popcountll(mr);
  }
  if (lane == 0) {
    a.wide_n[x] = n;
    a.wide_nfast[x] = nfast;
    // the groups of the batch, numbered through (the launch of the dQ workgroups runs over these
    // numbers: over the query tiles, with e.g. three of four workgroups leaving at once, the ones
    // that stay would all have the same index modulo four and land on two of the eight XCDs)
    int before = 0;
    for (int bb = 0; bb < b; ++bb) before += (a.qtile_start[bb + 1] - a.qtile_start[bb] + NQ - 1) / NQ;
    a.wide_list[before + qt / NQ] = x;
    if (qt == 0 && a.qtile_start[b + 1] == a.total_qtiles) a.wide_list[a.total_qtiles] = before + (QT + NQ - 1) / NQ;  // (the last sequence with tokens)
  }
}

// The tables that need those of the launch in front, a wave each: launch order of the chunks, of the dK / dV workgroups, and
// (with it for the same reason) the lists above.
struct OrderBlocks {
  int chunks, wide, order;
};
template <int NQ>
__global__ void __launch_bounds__(256) k_bwd_orders(BwdArgs a, OrderBlocks n) {
  int x = blockIdx.x;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (x < n.order) {
    if (4 * x + w < a.total_ktiles) bwd_order(a, 4 * x + w, lane);
    return;
  }
  x -= n.order;
  if (x < n.wide) {
    if (4 * x + w < a.total_qtiles) bwd_wide_rows<NQ>(a, 4 * x + w, lane);
    return;
  }
  x -= n.wide;
  const int slot = 4 * x + w;
  if (slot < a.slots) wide_order(slot, (int)a.slots, a.chunk.cnt, a.chunk.pre, a.chunk.desc, a.chunk.count);
}

// ---------------------------------------------------------------------------------------------
// k_bwd_dq2: the dQ kernel for head dimension 128 and four query heads per workgroup, with the data
// movement and instruction order of k_bwd_dkv2.  Eight waves (head g = wave / 2, query rows
// 32 (wave % 2) ..), two per SIMD, so that the vector and LDS instructions of one overlap the
// MFMAs of the other.  The K and V tiles of the key tiles whose pairs are all visible go through
// a ring of NST stages in the block layout described at k_bwd_dkv2 (4 loads per wave and stage),
// one bare barrier per tile in its middle; a tile is 48 slots: S^T = K Q^T and dP^T = V dO^T of
// the two 32-key halves (32 MFMAs, 16-byte row reads), then dQ^T += K^T dS^T of the two halves
// (16 MFMAs, transposing reads), with the exponentials of half 0 under the score MFMAs of half 1
// and those of half 1 under the dQ MFMAs of half 0.  The masked and ragged tiles follow in a second
// such loop (Eq. 3 of the tile as one 64-bit word per lane, a lane being a query row here:
// tile_visibility over the node ids of the tile's keys, which ride the ring as one more load).
// Head dimension 64 (k_bwd64_dq) runs the same code with half the slots and half the waves (two
// query heads, or one head on two query tiles): its ring takes 71 KB, so two such workgroups share a
// compute unit, and head groups of two and six need no padding.  (The same DAGs: 813 us with
// k_bwd_dq, 336 so.)
template <int D>
struct Dq {
  using R = RingTile<D>;
  static constexpr int NST = 4;
  static constexpr int NPAIR = D == 128 ? 4 : 2;   // wave pairs = query heads (or query tiles of one head) per workgroup
  static constexpr int PF = 4;                     // operands in flight ahead of their MFMA
  static constexpr int TILEB = R::TILEB;
  static constexpr int NPB = R::NBLK / (2 * NPAIR);  // blocks of a tile that one wave fetches
  static constexpr int ND = 2 * TILEB;             // node ids of the tile's keys [64] (masked tiles)
  static constexpr int STAGEB = ND + 256;          // K tile, V tile, node ids
  static constexpr int HS = D / 8;                 // slots of the score MFMAs of one 32-key half
  static constexpr int NDQ = D / 16;               // slots of the dQ MFMAs of one half
  static constexpr int NSC = 2 * HS, NSLOT = NSC + 2 * NDQ;
  // tiles of the list kept in LDS (two workgroups per compute unit at head dimension 64)
  static constexpr int LIST = D == 128 || MAX_ROW_LDS < 2048 ? MAX_ROW_LDS : 2048;
  static constexpr int opnd_reads(int o) { return o < NSC ? 1 : 2; }
  static constexpr int issued_through(int k) {  // LDS reads issued up to and including those of operand k
    int t = 0;
    for (int o = 0; o <= k; ++o) t += opnd_reads(o);
    return t;
  }
  static constexpr int wait_at(int i) {  // reads that may still be pending when MFMA i starts
    const int last = i + PF < NSLOT ? i + PF : NSLOT - 1;
    const int n = issued_through(last) - issued_through(i);
    return n < 15 ? n : 15;
  }
  static constexpr int row_imm(int i) {  // half i / HS, k-step (i % HS) / 2, of K (even) or V (odd)
    return (i & 1) * TILEB + R::row_imm(i / HS, (i % HS) / 2);
  }
  static constexpr int tr_imm(int i, int second) {  // i >= NSC: K^T operand of key half (i - NSC) / NDQ, 16-key group x, dims 32 db ..
    const int j = i - NSC, hh = j / NDQ, x = (j % NDQ) / (D / 32), db = j % (D / 32);
    return R::tr_imm(2 * hh + x, second, db);
  }
};

// WIDE: the same workgroup turned by ninety degrees -- one query head on four (two) consecutive query
// tiles (wave pair p takes tile 4 c + p), for the heads that do not fill a group: the waves still
// share every staged K / V tile.  The tile list is the one bwd_wide_rows wrote.
// NODES: on query chunks instead of query tiles (the forward's tables, k_node_rows): the keys of a chunk stream
// in the order of what its node sees, gathered row by row, so that only its last tiles take a mask, and
// that mask is arithmetic on positions.  Random DAGs of 4 x 64 nodes of 32 to 256 tokens, 16 / 8 heads of
// dimension 64: 336 us on the block map's tiles, 240 on chunks.
// The 32 NW columns of an item are (row, head) pairs, row-major, of all heads of the group (more than eight evenly divided), as in the
// forward: no head is left over for a launch of its own on chunks of 256 rows, which random DAGs leave half empty, and the
// pairs without a row are whole waves at the end, which fetch their share of the tiles and leave the matrix pipe to
// the others.  Forward and backward: 40 / 8 heads, 3 x 82 random nodes 425 -> 340 us, 48 / 8 heads, 3 x 45 663 -> 509; 4 x 64 nodes,
// 16 / 8 heads of dimension 64 808 -> 786; 26 batches 1.045 times as fast (0.997 at worst).
// Few chunks leave compute units idle, and a chunk is a chain of 2 us a tile: its tiles are then shared out over up to
// `pieces` workgroups of at least DQ_PIECE tiles, whose sums k_dq_sum adds up (2214 tokens of one head 70 -> 33 + 5 us, 3515 tokens, 8 / 2 heads: 106 -> 42 + 5).
// Forward and backward of 40 batches of up to 9000 tokens: of at least 3, 4, 9, 12 tiles 1.00, 1.01, 0.99, 0.99 times as fast (0.97,
// 0.99, 0.88, 0.77 at worst), at most 8 or 32 workgroups 1.00.
constexpr int DQ_PIECE = 6, DQ_LONG_PIECE = 16, DQ_MAX_PIECES = 16;
__device__ __forceinline__ int dq_cuts(int tiles, int pieces, int piece) { return max(min(pieces, tiles / piece), 1); }
template <int D, bool WIDE, bool NODES, bool PIECES = false>
__device__ __forceinline__ void dq_ring_body(const BwdArgs& a) {
  using C = Dq<D>;
  using R = RingTile<D>;
  constexpr int NPAIR = C::NPAIR, NT = 128 * NPAIR, NW = 2 * NPAIR, NST = C::NST, PF = C::PF, NPB = C::NPB, TILEB = C::TILEB;
  constexpr int ND = C::ND, STAGEB = C::STAGEB, HS = C::HS, NDQ = C::NDQ, NSC = C::NSC, NSLOT = C::NSLOT;
  typedef __attribute__((address_space(3))) void* lds_ptr_t;
  typedef __attribute__((address_space(1))) const void* gbl_ptr_t;
  typedef short v4i16 __attribute__((ext_vector_type(4)));
  typedef short v8i16 __attribute__((ext_vector_type(8)));
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int32_t sCol[NODES ? 1 : C::LIST];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, L = lane & 31, H = lane >> 5;
  const int pair = w >> 1;  // (WIDE) which of the query tiles
  DqTile t;
  int64_t wide_base = 0;
  int cuts = 1, tile0 = 0, tile1 = 0;
  if constexpr (NODES) {
    const int chunk = PIECES ? blockIdx.x / a.dq_pieces : blockIdx.x, cut = PIECES ? blockIdx.x % a.dq_pieces : 0;
    if (chunk >= *a.chunk.count) return;  // (the launch is sized by a bound)
    const int32_t* d = a.chunk.desc + (size_t)chunk * 8;
    t.cu = d[0], t.T = d[1], t.row0 = d[2], t.c0 = d[3], t.N = d[4], t.nfast = d[5], t.nbase = d[6];
    if constexpr (PIECES) cuts = dq_cuts(t.N, a.dq_pieces, a.dq_piece);
    if (cut >= cuts) return;
    tile0 = cut * (t.N / cuts) + min(cut, t.N % cuts);
    tile1 = tile0 + t.N / cuts + (cut < t.N % cuts);
  } else if constexpr (!WIDE) {
    t = dq_tile(a);
  } else {
    const int groups = a.wide_list[a.total_qtiles];
    if ((int)blockIdx.x >= groups) return;  // (the whole workgroup: the launch is sized by a bound)
    const int x = a.wide_list[groups - 1 - (int)blockIdx.x];  // the long rows at the end of a sequence first
    const int b = dag_find_segment(a.qtile_start, a.n_seqs, x);
    const int qt = x - a.qtile_start[b];
    t.cu = a.cu_seqlens[b], t.T = a.cu_seqlens[b + 1] - t.cu, t.row0 = qt * BM, t.c0 = 0;
    t.N = a.wide_n[x], t.nfast = a.wide_nfast[x], t.nbase = a.node_start[b];
    wide_base = a.block_map_off[b] + (int64_t)qt * ((t.T + BN - 1) / BN);
  }
  const int hk = blockIdx.y, cu = t.cu, T = t.T;
  DqLane<D> me;
  bool idle = false;
  if constexpr (NODES) {
    const int2 p = dq_pair(32 * w + L, a.pack_heads);
    const int g = (int)blockIdx.z * a.pack_heads + p.y;
    dq_setup_row<D>(a, t, hk, g, p.x < a.pack_rows && g < a.G, t.row0 + min(p.x, a.pack_rows - 1), me);
    idle = dq_pair(32 * w, a.pack_heads).x >= min(a.pack_rows, t.T - t.row0);
  } else if constexpr (!WIDE)
    dq_setup<D, NPAIR>(a, t, hk, me);
  else
    dq_setup_at<D>(a, t, hk, a.dq_narrow + (int)blockIdx.z, true, t.row0 + BM * pair, me);
  f32x16 dQ[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int e = 0; e < 16; ++e) dQ[db][e] = 0.f;
  TileList<C::LIST> tl;
  if constexpr (!NODES) {
    tl.col = WIDE ? a.wide_col + wide_base : a.qtile_col + t.c0;
    tl.template fill<NT>(sCol, t.N);
    __syncthreads();
  }
  // NODES: the runs of the chunk's node, run e in lane e {first position, token - position}; where the issue
  // cursor is in them; the tokens of its own node in front of this lane's row
  const int anc = t.nbase, n_pos = t.nbase + min(t.row0 + (NODES ? a.pack_rows : 0), t.T);
  int run_pos = 0, run_delta = 0, run_at = 0, run_end = 0, run_d = 0, depth = 0;
  if constexpr (NODES) {
    const int2 run = ((const int2*)a.runs)[t.c0 + lane];
    run_pos = run.x;
    run_delta = run.y;
    depth = a.tok_depth[cu + min(me.i, T - 1)];
    asm volatile("" ::"v"(run_pos), "v"(run_delta), "v"(depth));
    run_d = __builtin_amdgcn_readlane(run_delta, 0);
    run_end = __builtin_amdgcn_readlane(run_pos, 1);
  }
  const int NF = t.nfast;  // entries 0 .. NF - 1 of the list: every pair visible, inside the sequence

  // ---- loads of one stage: wave w fetches blocks w and w + NW of the K tile and of the V tile; for
  // masked tiles every wave also fetches the node ids of the keys (the same 256 bytes from all
  // of them: the number of loads a wave has in flight must not depend on the wave)
  const uint32_t row_stride = (uint32_t)(a.hkv * D);
  const uint32_t chunk8 = R::src_col(lane);
  const int rsub = R::src_row(lane);
  struct IssueCtx {
    const uint16_t *kb, *vb;
    uint32_t voff[NPB];
    const int32_t* nodes;  // this lane's key of the tile
  };
  auto prepare_issue = [&](int n, int n_end) __attribute__((always_inline)) {
    IssueCtx c;
    if constexpr (NODES) {
      c.kb = a.k + hk * D;
      c.vb = a.v + hk * D;
      const int last = min(n * BN + BN, n_pos) - 1;
      int tok[NPB], pos[NPB];
#pragma unroll
      for (int i = 0; i < NPB; ++i) {  // (positions past the end re-read the last one and are masked)
        pos[i] = min(n * BN + R::RPB * (w + NW * i) + rsub, last);
        tok[i] = n < n_end ? pos[i] + run_d : cu;  // (past the end of the walk: any row, never consumed)
      }
      while (n < n_end && run_end <= last) {  // (wave-uniform) the tile reaches into the next run
        run_at = run_at + 1;
        const int from = run_end;
        run_d = __builtin_amdgcn_readlane(run_delta, run_at);
        run_end = run_at < 63 ? __builtin_amdgcn_readlane(run_pos, run_at + 1) : INT32_MAX;
#pragma unroll
        for (int i = 0; i < NPB; ++i) tok[i] = pos[i] >= from ? pos[i] + run_d : tok[i];
      }
#pragma unroll
      for (int i = 0; i < NPB; ++i) c.voff[i] = (uint32_t)tok[i] * row_stride + chunk8;
      return c;
    }
    const int kv = n < n_end ? tl.tile(n) : 0;  // (past the end of the walk: the sequence's first tile, never consumed)
    const int j0 = kv * BN, n_in = min(BN, T - j0);
    const size_t slab = ((size_t)(cu + j0) * a.hkv + hk) * D;
    c.kb = a.k + slab;
    c.vb = a.v + slab;
#pragma unroll
    for (int i = 0; i < NPB; ++i) c.voff[i] = (uint32_t)min(R::RPB * (w + NW * i) + rsub, n_in - 1) * row_stride + chunk8;
    c.nodes = a.tok_node + cu + j0 + min(lane, n_in - 1);
    return c;
  };
  auto issue_piece = [&](int p, const IssueCtx& c, int st) __attribute__((always_inline)) {
    unsigned char* const sb = smem + st * STAGEB;
    if (p < 2 * NPB) {
      const int blk = w + NW * (p % NPB);
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)((p < NPB ? c.kb : c.vb) + c.voff[p % NPB]),
                                       (lds_ptr_t)(sb + (p < NPB ? 0 : TILEB) + blk * R::BLK), 16, 0, 0);
    } else {
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)c.nodes, (lds_ptr_t)(sb + ND), 4, 0, 0);
    }
  };
  const uint32_t roff[2] = {R::row_lane(L, H, 0), R::row_lane(L, H, 1)};
  const uint32_t toff = R::tr_lane(lane);
  const uint32_t smem_base = lds_addr(smem);
  const float sc = a.sc, nl = -me.lse2, dl = me.dl;
  // Minus delta in sixteen registers, which the sums of dP start from: no vector instruction subtracts it (32 of 153 a tile).  Forward
  // and backward of seven batches at dimension 64, where vector instructions count, 1.012 times as fast, of nine at 128 1.003.
  f32x16 ndl;
#pragma unroll
  for (int e = 0; e < 16; ++e) ndl[e] = -dl;
  asm volatile("" : "+v"(ndl));
  const int nq = me.ni, iq_row = me.i;
  const bool row_ok = me.row_ok;
  const uint64_t* const vis_row = NODES ? a.node_vis : a.node_vis + (int64_t)(t.nbase + nq) * a.W;
  const uint64_t vis0 = NODES ? 0 : me.vis0, vis1 = !NODES && a.W > 1 ? vis_row[1] : 0;  // (sequences with more than 128 nodes fetch the word they need)
  asm volatile("" ::"v"(vis0), "v"(vis1));  // (their arrival belongs here, not between the ring's loads)
  auto word_of = [&](uint32_t n) __attribute__((always_inline)) -> uint64_t { return n < 64 ? vis0 : n < 128 ? vis1 : vis_row[n >> 6]; };  // (n is wave-uniform)

  // ---- one key tile, slot by slot; MSK: with Eq. 3 (one visibility word per node) and the end of the
  // sequence applied per element from the lane's visibility word of the tile
  // (with masks: vis_lo / vis_hi = this lane's visibility word of the tile, shifted so that bit
  // 32 hh + 8 (e / 4) + e % 4 belongs to element e of half hh, i.e. to key 64 kt + 4 H + that number)
  auto pipelined_tile = [&](auto msk_c, int cs, const IssueCtx& ictx, int is, uint32_t vis_lo, uint32_t vis_hi) __attribute__((always_inline)) {
    constexpr bool MSK = decltype(msk_c)::value;
    constexpr int LPS = 2 * NPB + (MSK && !NODES ? 1 : 0), PFM = PF;
    const uint32_t sbase = smem_base + (uint32_t)cs * STAGEB;
    const uint32_t ra[2] = {sbase + roff[0], sbase + roff[1]}, ta = sbase + toff;
    bf16x8 op[NSLOT];
    v4i16 lo[NSLOT], hi[NSLOT];
    f32x16 S[2], dP[2];
    float dt[2][16];
    bf16x8 bds[2][2];
    auto fetch = [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      constexpr int odd = ((i % HS) / 2) & 1;  // (k-step of a row operand)
      const uint32_t r = D == 128 ? ra[0] : ra[odd], t = ta;  // (named here: captures inside discarded branches trip the compiler)
      bf16x8* const opp = op;
      v4i16* const lop = lo;
      v4i16* const hip_ = hi;
      if constexpr (i < NSC)
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(opp[i]) : "v"(r), "n"(C::row_imm(i) + (D == 128 ? 32 * odd : 0)));
      else if constexpr (i < NSLOT)
        asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                     : "=&v"(lop[i]), "=&v"(hip_[i])
                     : "v"(t), "n"(C::tr_imm(i, 0)), "n"(C::tr_imm(i, 1)));
    };
    auto score = [&](auto hc, auto ec) __attribute__((always_inline)) {  // dS of key e of half h (this lane's row), packed in pairs
      constexpr int h = decltype(hc)::value, e = decltype(ec)::value;
      dt[h][e] = __builtin_amdgcn_exp2f(fmaf(S[h][e], sc, nl)) * dP[h][e];
      // Eq. 3 and the end of the sequence (behind the product: V of a hidden key may be anything)
      if constexpr (MSK) dt[h][e] = keep_if_bit<8 * (e >> 2) + (e & 3)>(dt[h][e], h == 0 ? vis_lo : vis_hi);
      if constexpr ((e & 1) == 1) {
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
        const bf16x2 pk = __builtin_bit_cast(bf16x2, dag_pack_bf2(dt[h][e - 1], dt[h][e]));
        bds[h][e >> 3][(e & 7) - 1] = pk[0];
        bds[h][e >> 3][e & 7] = pk[1];
      }
    };
    static_for<0, PFM>(fetch);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NSLOT>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
      if constexpr (i == NSC) {
        wait_vmcnt_only<LPS>();        // this wave's loads of the next tile's stage have landed
        __builtin_amdgcn_s_barrier();  // (bare: a __syncthreads would drain the loads in flight)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      fetch(std::integral_constant<int, i + PFM>{});
      wait_lgkmcnt_only<C::wait_at(i)>();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (i < NSC) {
        constexpr int hh = i / HS, s = (i % HS) / 2;
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if constexpr ((i & 1) == 0)
          S[hh] = mfma32(op[i], me.qf[s], s == 0 ? zero : S[hh]);
        else
          dP[hh] = mfma32(op[i], me.dof[s], s == 0 ? ndl : dP[hh]);
      } else {
        constexpr int j = i - NSC, hh = j / NDQ, x = (j % NDQ) / (D / 32), db = j % (D / 32);
        const v8i16 t8 = {lo[i][0], lo[i][1], lo[i][2], lo[i][3], hi[i][0], hi[i][1], hi[i][2], hi[i][3]};
        dQ[db] = mfma32(__builtin_bit_cast(bf16x8, t8), bds[hh][x], dQ[db]);
      }
      if constexpr (i >= NSC && i < NSC + LPS) issue_piece(i - NSC, ictx, is);
      if constexpr (i >= HS && i < NSC)
        static_for<16 / HS * (i - HS), 16 / HS * (i - HS + 1)>([&](auto ec) __attribute__((always_inline)) { score(std::integral_constant<int, 0>{}, ec); });
      if constexpr (i >= NSC && i < NSC + NDQ)
        static_for<16 / NDQ * (i - NSC), 16 / NDQ * (i - NSC + 1)>([&](auto ec) __attribute__((always_inline)) { score(std::integral_constant<int, 1>{}, ec); });
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // ---- the pipelined walk over entries n0 .. n1 - 1 of the tile list
  auto ring_loop = [&](auto msk_c, int n0, int n1) __attribute__((always_inline)) {
    constexpr int LPS = 2 * NPB + (decltype(msk_c)::value && !NODES ? 1 : 0);
    if (n0 >= n1) return;
    int in = n0;  // list entry whose loads are issued next
#pragma unroll 1
    for (int st = 0; st < NST - 1; ++st, ++in) {
      const IssueCtx c = prepare_issue(in, n1);
#pragma unroll
      for (int p = 0; p < LPS; ++p) issue_piece(p, c, st);
    }
    wait_vmcnt_only<(NST - 2) * LPS>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    int cs = 0, is = NST - 1;
    for (int n = n0; n < n1; ++n, ++in) {
      const IssueCtx ic = prepare_issue(in, n1);
      uint64_t vis = 0;
      if constexpr (decltype(msk_c)::value && NODES) {
        // the positions in front of the group, and those of the row's own node up to its own
        auto first_bits = [](int c) { return c >= 64 ? ~0ull : c <= 0 ? 0ull : (1ull << c) - 1; };
        const int own = anc + iq_row - n * BN;  // the row's position inside the tile
        vis = first_bits(anc - n * BN) | (first_bits(own + 1) & ~first_bits(own - depth));
        vis = row_ok ? vis >> (4 * H) : 0ull;
      } else if constexpr (decltype(msk_c)::value) {
        // the keys of the tile that this lane's row sees: own node up to the row itself
        // (WIDE: none at all when the wave pair's own query tile does not see the key tile -- the
        // few such tiles along the diagonal are multiplied through with zeros)
        const int kt = tl.tile(n);
        const int last = iq_row - kt * BN;  // last such key of the tile (may lie before or behind it)
        const uint64_t own = last < 0 ? 0ull : last >= 63 ? ~0ull : (2ull << last) - 1;
        vis = tile_visibility(smem_base + (uint32_t)cs * STAGEB + ND, lane, (uint32_t)nq, own, T - kt * BN, word_of);
        vis = row_ok ? vis >> (4 * H) : 0ull;
      }
      if (NODES && idle) {  // only the ring's business
        wait_vmcnt_only<LPS>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int p = 0; p < LPS; ++p) issue_piece(p, ic, is);
      } else {
        pipelined_tile(msk_c, cs, ic, is, (uint32_t)vis, (uint32_t)(vis >> 32));
      }
      cs = cs + 1 == NST ? 0 : cs + 1;
      is = is + 1 == NST ? 0 : is + 1;
    }
    wait_vmcnt_only<0>();          // (the loads past the end of the walk)
    __builtin_amdgcn_s_barrier();  // every wave is done with the ring before it is filled again
    asm volatile("" ::: "memory");
  };
  if constexpr (!NODES) tile1 = t.N;
  ring_loop(std::false_type{}, tile0, min(NF, tile1));
  ring_loop(std::true_type{}, max(NF, tile0), tile1);  // the masked and the ragged tiles
  // The masked tiles of a chunk multiply a hidden key's K by zero, and 0 x Inf or NaN is NaN: as in dK / dV above
  // the dQ rows of such a wave are taken again from the visible keys.
  if constexpr (NODES) {
    float any = 0.f;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int e = 0; e < 16; e += 2) any = __builtin_elementwise_maximum(__builtin_elementwise_maximum(dQ[db][e], dQ[db][e + 1]), any);
    const int2* const runs = (const int2*)a.runs + t.c0;
    const int pos_end = min(tile1 * BN, n_pos);
    bool suspect = false;
    if (__builtin_amdgcn_ballot_w64(row_ok && any != any) != 0) {
#pragma unroll 1
      for (int p0 = max(NF, tile0) * BN; p0 < pos_end && !suspect; p0 += 64) {  // a key per lane
        const int p = min(p0 + lane, pos_end - 1);
        int tok = cu;
        for (int e = 0; e < 64 && runs[e].x < p0 + 64; ++e) tok = p >= runs[e].x ? p + runs[e].y : tok;
        suspect = __builtin_amdgcn_ballot_w64(dag_row_not_finite<D>(a.k + ((size_t)tok * a.hkv + hk) * D)) != 0;
      }
    }
    if (suspect) {
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) dQ[db][e] = 0.f;
      const int own = anc + iq_row;
      int run = 0;
#pragma unroll 1
      for (int p = tile0 * BN; p < pos_end; ++p) {
        while (run < 63 && runs[run + 1].x <= p) ++run;
        const size_t row = (size_t)(p + runs[run].y) * a.hkv + hk;
        const uint16_t *kp = a.k + row * D, *vp = a.v + row * D;
        const bool ok = row_ok && (p < anc || (p <= own && p >= own - depth));
        float s = 0.f, dp = 0.f;
#pragma unroll
        for (int x = 0; x < D / 16; ++x) {
          const u32x4 kr = *(const u32x4*)(kp + 16 * x + 8 * H), vr = *(const u32x4*)(vp + 16 * x + 8 * H);
          const u32x4 qr = __builtin_bit_cast(u32x4, me.qf[x]), dr = __builtin_bit_cast(u32x4, me.dof[x]);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s = fmaf(dag_bf_hi(kr[e]), dag_bf_hi(qr[e]), fmaf(dag_bf_lo(kr[e]), dag_bf_lo(qr[e]), s));
            dp = fmaf(dag_bf_hi(vr[e]), dag_bf_hi(dr[e]), fmaf(dag_bf_lo(vr[e]), dag_bf_lo(dr[e]), dp));
          }
        }
        s += __shfl_xor(s, 32);
        dp += __shfl_xor(dp, 32);
        const float ds = __builtin_amdgcn_exp2f(fmaf(s, sc, nl)) * (dp - dl);
        bool number = false;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4) {
            const u32x2 kr = *(const u32x2*)(kp + 32 * db + 8 * e4 + 4 * H);
            const float k4[4] = {dag_bf_lo(kr[0]), dag_bf_hi(kr[0]), dag_bf_lo(kr[1]), dag_bf_hi(kr[1])};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float before = dQ[db][4 * e4 + e], after = ok ? fmaf(ds, k4[e], before) : before;
              dQ[db][4 * e4 + e] = after;
              number |= after == after;
            }
          }
        if (__builtin_amdgcn_ballot_w64(row_ok && number) == 0) break;
      }
    }
  }
  if (PIECES && cuts > 1) {
    f32x4* const to = a.part + ((((size_t)blockIdx.x * a.hkv + hk) * gridDim.z + blockIdx.z) * NW + w) * (D / 4 * 32) + lane;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4)
        to[(4 * db + e4) * 64] = f32x4{dQ[db][4 * e4], dQ[db][4 * e4 + 1], dQ[db][4 * e4 + 2], dQ[db][4 * e4 + 3]};
    return;
  }
  dq_store<D>(a, me, H, dQ);
}
// Sums of the chunks whose tiles several workgroups share, in the order of the tiles: a wave per sixteen dimensions of a wave of
// the dQ kernel, everything of eight pieces fetched at once.
template <int D>
__global__ void __launch_bounds__(256) k_dq_sum(BwdArgs a, int nz) {
  constexpr int NW = 2 * Dq<D>::NPAIR, PARTS = D / 16, AT_ONCE = 8;
  const int x = blockIdx.x * 4 + (threadIdx.x >> 6), part = x % PARTS, w = x / PARTS % NW, z = x / (PARTS * NW) % nz;
  const int hk = x / (PARTS * NW) / nz % a.hkv, chunk = x / (PARTS * NW) / nz / a.hkv;
  const int lane = threadIdx.x & 63, L = lane & 31, H = lane >> 5;
  if (chunk >= *a.chunk.count) return;
  const int32_t* const d = a.chunk.desc + (size_t)chunk * 8;
  const int n = dq_cuts(d[4], a.dq_pieces, a.dq_piece), rows = min(a.pack_rows, d[1] - d[2]);
  if (n < 2 || dq_pair(32 * w, a.pack_heads).x >= rows) return;
  const size_t step = (size_t)a.hkv * nz * NW * (D / 4 * 32);
  const f32x4* const from = a.part + (size_t)chunk * a.dq_pieces * step + (((size_t)hk * nz + z) * NW + w) * (D / 4 * 32) + 2 * part * 64 + lane;
  f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
  for (int p0 = 0; p0 < n; p0 += AT_ONCE) {
    f32x4 v[AT_ONCE][2];
#pragma unroll
    for (int i = 0; i < AT_ONCE; ++i) {
      const f32x4* const at = from + min(p0 + i, n - 1) * step;
      v[i][0] = at[0];
      v[i][1] = at[64];
    }
#pragma unroll
    for (int i = 0; i < AT_ONCE; ++i)
      if (p0 + i < n) {
        s0 += v[i][0];
        s1 += v[i][1];
      }
  }
  const int2 p = dq_pair(32 * w + L, a.pack_heads);
  const int g = z * a.pack_heads + p.y;
  if (p.x >= rows || g >= a.G) return;
  uint16_t* const to = a.dq + ((size_t)(d[0] + d[2] + p.x) * a.hq + hk * a.G + g) * D + 16 * part + 4 * H;
  *(u32x2*)to = u32x2{dag_pack_bf2(s0[0] * a.scale, s0[1] * a.scale), dag_pack_bf2(s0[2] * a.scale, s0[3] * a.scale)};
  *(u32x2*)(to + 8) = u32x2{dag_pack_bf2(s1[0] * a.scale, s1[1] * a.scale), dag_pack_bf2(s1[2] * a.scale, s1[3] * a.scale)};
}
template <bool WIDE>
__global__ void __launch_bounds__(512) k_bwd_dq2(BwdArgs a) { dq_ring_body<128, WIDE, false>(a); }
template <bool WIDE>
__global__ void __launch_bounds__(256, 2) k_bwd64_dq(BwdArgs a) { dq_ring_body<64, WIDE, false>(a); }
template <bool PIECES>
__global__ void __launch_bounds__(512) k_nodes_dq2(BwdArgs a) { dq_ring_body<128, false, true, PIECES>(a); }
template <bool PIECES>
__global__ void __launch_bounds__(256, 2) k_nodes64_dq(BwdArgs a) { dq_ring_body<64, false, true, PIECES>(a); }

template <int D, int HG>
int launch_dq(const BwdArgs& a, long total_qtiles, hipStream_t stream) {
  constexpr int sm = 2 * BN * (D + 8) * 2 + BN * 4;
  if (hipFuncSetAttribute((const void*)k_bwd_dq<D, HG>, hipFuncAttributeMaxDynamicSharedMemorySize, sm) != hipSuccess)
    return DAG_ERR_HIP;
  hipLaunchKernelGGL((k_bwd_dq<D, HG>), dim3((unsigned)total_qtiles, (unsigned)a.hkv, (unsigned)((a.G + HG - 1) / HG)),
                     dim3(128 * HG), sm, stream, a);
  DAG_LAUNCH_CHECK();
  return DAG_OK;
}

// Query heads of a KV head in an item of dQ on chunks: all of them, more than eight evenly divided.
int bwd_pack_heads(int G) { return (G + (G + 7) / 8 - 1) / ((G + 7) / 8); }

// Query heads per KV head that the dQ kernel takes one at a time on several query tiles.
int bwd_wide_heads(int G, int head_dim) { return G % (head_dim == 128 ? Dq<128>::NPAIR : Dq<64>::NPAIR); }

// Development switch, read once: DAGATTN_BWD_V1=1 runs the first dQ and dK/dV kernels for every shape.
bool bwd_first_version() {
  static const bool v = [] {
    const char* e = getenv("DAGATTN_BWD_V1");
    return e && e[0] == '1';
  }();
  return v;
}

// At most this many blocks of cut_keys: one for every 128 tokens of a sequence that ends there, one for every border.
int64_t bwd_cut_blocks(int64_t T, int64_t nodes, int64_t ktiles, int64_t n_seqs) { return std::min(ktiles, T / (2 * BN) + nodes + n_seqs); }

template <int D>
int launch_bwd(const BwdArgs& args, const PrefillArgs& p, long total_qtiles, long total_ktiles, hipStream_t stream) {
  BwdArgs a = args;
  constexpr int RPB = 256 / (D / 8), NQ = Dq<D>::NPAIR;  // rows per workgroup of bwd_delta
  const int waves4 = (int)((total_ktiles + 3) / 4);
  const PrepareBlocks pre = {a.runs ? (int)((p.total_nodes + 3) / 4) : 0, (int)((a.total_rows / a.hq + 255) / 256), a.block_start ? a.n_seqs : waves4, (int)((a.total_rows + RPB - 1) / RPB)};
  hipLaunchKernelGGL((k_bwd_delta_tables<D>), dim3((unsigned)(pre.nodes + pre.tokens + pre.weights + pre.delta)), dim3(256), 0, stream, a, p, pre);
  // (without pieces the flags of k_dkv_finish lie where dQ on the block map's tiles reads the words of its rows)
  const bool order_now = a.pieces || a.runs || !a.dkv_stream;
  const OrderBlocks ord = {a.runs ? (int)((a.slots + 3) / 4) : 0,
                           !a.runs && a.dq_narrow < a.G && !bwd_first_version() ? (int)((total_qtiles + 3) / 4) : 0, order_now ? waves4 : 0};
  if (ord.chunks + ord.wide + ord.order > 0)
    hipLaunchKernelGGL((k_bwd_orders<NQ>), dim3((unsigned)(ord.chunks + ord.wide + ord.order)), dim3(256), 0, stream, a, ord);
  DAG_LAUNCH_CHECK();
  int rc;
  if (!bwd_first_version()) {
    constexpr int NPAIR = Dq<D>::NPAIR, sm2 = Dq<D>::NST * Dq<D>::STAGEB;
    const int wide = a.G - a.dq_narrow;
    const bool nodes = a.runs != nullptr;
    a.dq_pieces = 1;
    const int nz = nodes ? (a.G + a.pack_heads - 1) / a.pack_heads : 0;
    const int64_t items = a.slots * a.hkv * nz;
    // (pieces for twice the workgroups that the device holds: about half of the slots have a chunk; sequences of less than 16
    // tiles on average would pay for the launch behind them, 4.5 us, and have next to nothing to share)
    // (Where the chunks alone nearly fill it there is nothing to gain but in chunks that are much longer than the others, as the join of a
    // fork: long sequences of few nodes, and of those the chunks of two DQ_LONG_PIECE.  Forks of 53 to 118 tiles, whole : in pieces
    // 1.03 to 1.26 (a fork of 28 nodes, 7376 tokens, 6 / 2 heads of dimension 128: 507 -> 409 us), of 49 to 51 tiles 0.92 to 0.99; random
    // nodes of 60 to 220 tokens 0.91 to 1.00, 6 x 38 nodes, 4 / 1 heads of dimension 64 76 : 84 us.)
    const int64_t chunks = nodes ? (p.total_tokens / a.pack_rows + p.total_nodes / 2) * a.hkv * nz : 0;
    const int64_t at_once = (int64_t)dag_compute_units() * (D == 128 ? 1 : 2);  // workgroups that run together
    if (at_once < 1) return DAG_ERR_HIP;
    const bool filled = 4 * chunks >= 3 * at_once;
    a.dq_piece = filled ? DQ_LONG_PIECE : DQ_PIECE;
    if (nodes && a.pieces && total_qtiles >= (filled ? 52 : 16) * a.n_seqs && (!filled || p.total_tokens >= 256 * p.total_nodes)) {
      const int64_t fits = (int64_t)a.max_split * a.hkv * (D == 128 ? 1 : 2);
      a.dq_pieces = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(2 * at_once / items, fits / items), DQ_MAX_PIECES));
    }
    auto* const on_chunks = D == 128 ? (a.dq_pieces > 1 ? k_nodes_dq2<true> : k_nodes_dq2<false>) : a.dq_pieces > 1 ? k_nodes64_dq<true> : k_nodes64_dq<false>;
    auto* const one_tile = nodes ? on_chunks : D == 128 ? k_bwd_dq2<false> : k_bwd64_dq<false>;
    auto* const many_tiles = D == 128 ? k_bwd_dq2<true> : k_bwd64_dq<true>;
    if (hipFuncSetAttribute((const void*)one_tile, hipFuncAttributeMaxDynamicSharedMemorySize, sm2) != hipSuccess ||
        hipFuncSetAttribute((const void*)many_tiles, hipFuncAttributeMaxDynamicSharedMemorySize, sm2) != hipSuccess)
      return DAG_ERR_HIP;
    if (nodes) {
      hipLaunchKernelGGL(one_tile, dim3((unsigned)(a.slots * a.dq_pieces), (unsigned)a.hkv, (unsigned)nz), dim3(128 * NPAIR), sm2, stream, a);
      if (a.dq_pieces > 1)
        hipLaunchKernelGGL((k_dq_sum<D>), dim3((unsigned)(items * 2 * NPAIR * (D / 16) / 4)), dim3(256), 0, stream, a, nz);
    } else {
      if (a.dq_narrow > 0)
        hipLaunchKernelGGL(one_tile, dim3((unsigned)total_qtiles, (unsigned)a.hkv, (unsigned)((a.dq_narrow + NPAIR - 1) / NPAIR)), dim3(128 * NPAIR), sm2, stream, a);
      if (wide > 0) {  // the heads left over by the groups of NPAIR take NPAIR query tiles each
        const long groups_bound = std::min(total_qtiles, (total_qtiles + NPAIR - 1) / NPAIR + a.n_seqs);
        hipLaunchKernelGGL(many_tiles, dim3((unsigned)groups_bound, (unsigned)a.hkv, (unsigned)wide), dim3(128 * NPAIR), sm2, stream, a);
      }
    }
    rc = hipGetLastError() == hipSuccess ? DAG_OK : DAG_ERR_HIP;
  } else {
    a.dq_narrow = a.G;
    rc = a.G >= 3 ? launch_dq<D, 4>(a, total_qtiles, stream)
                  : a.G == 2 ? launch_dq<D, 2>(a, total_qtiles, stream) : launch_dq<D, 1>(a, total_qtiles, stream);
  }
  if (rc != DAG_OK) return rc;
  if (!order_now) {
    hipLaunchKernelGGL((k_bwd_orders<NQ>), dim3((unsigned)waves4), dim3(256), 0, stream, a, OrderBlocks{0, 0, waves4});
    DAG_LAUNCH_CHECK();
  }
  if (!bwd_first_version()) {
    constexpr int sm2 = Dkv<D>::NST * Dkv<D>::STAGEB;
    auto* const ring = D == 128 ? (a.dkv_stream ? k_nodes_dkv2 : k_bwd_dkv2) : a.dkv_stream ? k_nodes64_dkv : k_bwd64_dkv;
    if (hipFuncSetAttribute((const void*)ring, hipFuncAttributeMaxDynamicSharedMemorySize, sm2) != hipSuccess)
      return DAG_ERR_HIP;
    const long pairs = a.block_start ? (long)bwd_cut_blocks(p.total_tokens, p.total_nodes, total_ktiles, a.n_seqs) : a.pieces ? (total_ktiles + a.n_seqs) / 2 : total_ktiles;
    hipLaunchKernelGGL(ring, dim3((unsigned)((pairs + a.max_split) * a.hkv)), dim3(256), sm2, stream, a);
    // (it reads K, V, Q and dO once more: not where the gradients have been written over them)
    const size_t q_bytes = (size_t)a.total_rows * D * 2, k_bytes = q_bytes / a.G;
    auto apart = [&](const void* p, size_t p_bytes, const void* out) {
      return (const char*)p + p_bytes <= (const char*)out || (const char*)out + k_bytes <= (const char*)p;
    };
    a.again = a.dkv_stream;
    for (const void* out : {(const void*)a.dk, (const void*)a.dv})
      a.again = a.again && apart(a.q, q_bytes, out) && apart(a.dout, q_bytes, out) && apart(a.k, k_bytes, out) && apart(a.v, k_bytes, out);
    if (a.again || a.pieces)
      hipLaunchKernelGGL(k_dkv_finish<D>, dim3((unsigned)(total_ktiles + (long)(a.max_split / 2) * a.hkv * 4)), dim3(256), 0, stream, a);
  } else {
    constexpr int sm = dkv_smem_bytes<D>();
    if (hipFuncSetAttribute((const void*)k_bwd_dkv<D>, hipFuncAttributeMaxDynamicSharedMemorySize, sm) != hipSuccess)
      return DAG_ERR_HIP;
    hipLaunchKernelGGL((k_bwd_dkv<D>), dim3((unsigned)(total_ktiles * a.hkv)), dim3(256), sm, stream, a);
  }
  DAG_LAUNCH_CHECK();
  return DAG_OK;
}

// ---------------------------------------------------------------------------------------------
// fp32 backward: the accuracy path beside k_prefill_f32 (plain vector arithmetic, exact expf, the
// same 64 x 64 tiles and block map).  Four threads share a row (a query row in k_bwd_dq_f32, a key
// in k_bwd_dkv_f32), each owning a quarter of the head dimension.  Not a performance path.
struct BwdArgsF32 {
  const float *q, *k, *v, *out, *dout, *lse;
  float *dq, *dk, *dv, *delta;
  const int32_t *cu_seqlens, *node_start, *tok_node, *qtile_start, *ktile_start;
  const uint64_t* node_vis;
  const int64_t* block_map_off;
  const uint8_t* block_map;
  int n_seqs, W, hq, hkv, G;
  float scale;
};

__device__ __forceinline__ float quad_sum(float x) {  // over the four threads of a row
  x += __shfl_xor(x, 1);
  x += __shfl_xor(x, 2);
  return x;
}

template <int D>
__global__ void __launch_bounds__(256) k_bwd_dq_f32(BwdArgsF32 a) {
  extern __shared__ float smem_f[];
  float* Ks = smem_f;            // [BN][D]
  float* Vs = smem_f + BN * D;   // [BN][D]
  int* s_node = (int*)(Vs + BN * D);
  constexpr int DP = D / 4;
  const int qt = blockIdx.x, head = blockIdx.y, hk = head / a.G;
  const int b = dag_find_segment(a.qtile_start, a.n_seqs, qt);
  const int cu = a.cu_seqlens[b], T = a.cu_seqlens[b + 1] - cu;
  const int qtl = qt - a.qtile_start[b], KT = (T + BN - 1) / BN;
  const uint8_t* bm = a.block_map + a.block_map_off[b] + (int64_t)qtl * KT;
  const int r = threadIdx.x >> 2, part = threadIdx.x & 3;
  const int i = qtl * BM + r, ic = min(i, T - 1);
  const int ni = a.tok_node[cu + ic];
  const uint64_t* vis_row = a.node_vis + (int64_t)(a.node_start[b] + ni) * a.W;
  const size_t row = (size_t)(cu + ic) * a.hq + head;
  float qr[DP], dor[DP], dq[DP];
  float dl = 0.f;
#pragma unroll
  for (int d = 0; d < DP; ++d) {
    qr[d] = a.q[row * D + part * DP + d];
    dor[d] = a.dout[row * D + part * DP + d];
    dl += dor[d] * a.out[row * D + part * DP + d];
    dq[d] = 0.f;
  }
  dl = quad_sum(dl);
  if (i < T && part == 0) a.delta[row] = dl;  // for the dK / dV kernel
  const float lse = a.lse[row];
  for (int kt = 0; kt < KT; ++kt) {
    const int flag = bm[kt];
    if (flag == 0) continue;
    const int j0 = kt * BN;
    __syncthreads();
    for (int idx = threadIdx.x; idx < BN * (D / 4); idx += 256) {
      const int rr = idx / (D / 4), c4 = idx % (D / 4);
      const size_t g = ((size_t)(cu + min(j0 + rr, T - 1)) * a.hkv + hk) * D + c4 * 4;
      *(f32x4*)(Ks + rr * D + c4 * 4) = *(const f32x4*)(a.k + g);
      *(f32x4*)(Vs + rr * D + c4 * 4) = *(const f32x4*)(a.v + g);
    }
    if (threadIdx.x < BN) s_node[threadIdx.x] = a.tok_node[cu + min(j0 + (int)threadIdx.x, T - 1)];
    __syncthreads();
    const int jn = min(BN, T - j0);
    for (int jj = 0; jj < jn; ++jj) {
      const int j = j0 + jj, nj = s_node[jj];
      const bool ok = flag == 2 || (nj == ni ? j <= i : (bool)((vis_row[nj >> 6] >> (nj & 63)) & 1));
      float s = 0.f, dp = 0.f;
#pragma unroll
      for (int d = 0; d < DP; ++d) {
        s += qr[d] * Ks[jj * D + part * DP + d];
        dp += dor[d] * Vs[jj * D + part * DP + d];
      }
      s = quad_sum(s);
      dp = quad_sum(dp);
      if (ok) {
        const float ds = expf(s * a.scale - lse) * (dp - dl);
#pragma unroll
        for (int d = 0; d < DP; ++d) dq[d] += ds * Ks[jj * D + part * DP + d];
      }
    }
  }
  if (i < T)
#pragma unroll
    for (int d = 0; d < DP; ++d) a.dq[row * D + part * DP + d] = dq[d] * a.scale;
}

template <int D>
__global__ void __launch_bounds__(256) k_bwd_dkv_f32(BwdArgsF32 a) {
  extern __shared__ float smem_f[];
  float* Qs = smem_f;             // [BM][D]
  float* dOs = smem_f + BM * D;   // [BM][D]
  float* s_lse = dOs + BM * D;    // [BM]
  float* s_dl = s_lse + BM;       // [BM]
  int* s_node = (int*)(s_dl + BM);
  constexpr int DP = D / 4;
  const int kt = blockIdx.x, hk = blockIdx.y;
  const int b = dag_find_segment(a.ktile_start, a.n_seqs, kt);
  const int cu = a.cu_seqlens[b], T = a.cu_seqlens[b + 1] - cu;
  const int ktl = kt - a.ktile_start[b];
  const int QT = (T + BM - 1) / BM, KT = (T + BN - 1) / BN;
  const uint8_t* bm = a.block_map + a.block_map_off[b];
  const int nbase = a.node_start[b];
  const int r = threadIdx.x >> 2, part = threadIdx.x & 3;
  const int j = ktl * BN + r, jc = min(j, T - 1);
  const int nj = a.tok_node[cu + jc];
  const size_t krow = (size_t)(cu + jc) * a.hkv + hk;
  float kr[DP], vr[DP], dk[DP], dv[DP];
#pragma unroll
  for (int d = 0; d < DP; ++d) {
    kr[d] = a.k[krow * D + part * DP + d];
    vr[d] = a.v[krow * D + part * DP + d];
    dk[d] = dv[d] = 0.f;
  }
  for (int qt = 0; qt < QT; ++qt) {
    const int flag = bm[(int64_t)qt * KT + ktl];
    if (flag == 0) continue;
    const int r0 = qt * BM;
    for (int g = 0; g < a.G; ++g) {
      const int head = hk * a.G + g;
      __syncthreads();
      for (int idx = threadIdx.x; idx < BM * (D / 4); idx += 256) {
        const int rr = idx / (D / 4), c4 = idx % (D / 4);
        const size_t o = ((size_t)(cu + min(r0 + rr, T - 1)) * a.hq + head) * D + c4 * 4;
        *(f32x4*)(Qs + rr * D + c4 * 4) = *(const f32x4*)(a.q + o);
        *(f32x4*)(dOs + rr * D + c4 * 4) = *(const f32x4*)(a.dout + o);
      }
      if (threadIdx.x < BM) {
        const size_t o = (size_t)(cu + min(r0 + (int)threadIdx.x, T - 1)) * a.hq + head;
        s_lse[threadIdx.x] = a.lse[o];
        s_dl[threadIdx.x] = a.delta[o];
        s_node[threadIdx.x] = a.tok_node[cu + min(r0 + (int)threadIdx.x, T - 1)];
      }
      __syncthreads();
      const int in = min(BM, T - r0);
      for (int ii = 0; ii < in; ++ii) {
        const int i = r0 + ii, ni = s_node[ii];
        bool ok = j < T;
        if (flag != 2 && ok)
          ok = nj == ni ? j <= i : (bool)((a.node_vis[(int64_t)(nbase + ni) * a.W + (nj >> 6)] >> (nj & 63)) & 1);
        float s = 0.f, dp = 0.f;
#pragma unroll
        for (int d = 0; d < DP; ++d) {
          s += kr[d] * Qs[ii * D + part * DP + d];
          dp += vr[d] * dOs[ii * D + part * DP + d];
        }
        s = quad_sum(s);
        dp = quad_sum(dp);
        if (ok) {
          const float p = expf(s * a.scale - s_lse[ii]);
          const float ds = p * (dp - s_dl[ii]);
#pragma unroll
          for (int d = 0; d < DP; ++d) {
            dv[d] += p * dOs[ii * D + part * DP + d];
            dk[d] += ds * Qs[ii * D + part * DP + d];
          }
        }
      }
    }
  }
  if (j < T)
#pragma unroll
    for (int d = 0; d < DP; ++d) {
      a.dk[krow * D + part * DP + d] = dk[d] * a.scale;
      a.dv[krow * D + part * DP + d] = dv[d];
    }
}

template <int D>
int launch_bwd_f32(const BwdArgsF32& a, long total_qtiles, long total_ktiles, hipStream_t stream) {
  const int sm_q = 2 * BN * D * 4 + BN * 4, sm_k = 2 * BM * D * 4 + 3 * BM * 4;
  if (hipFuncSetAttribute((const void*)k_bwd_dq_f32<D>, hipFuncAttributeMaxDynamicSharedMemorySize, sm_q) != hipSuccess ||
      hipFuncSetAttribute((const void*)k_bwd_dkv_f32<D>, hipFuncAttributeMaxDynamicSharedMemorySize, sm_k) != hipSuccess)
    return DAG_ERR_HIP;
  hipLaunchKernelGGL((k_bwd_dq_f32<D>), dim3((unsigned)total_qtiles, (unsigned)a.hq), dim3(256), sm_q, stream, a);
  hipLaunchKernelGGL((k_bwd_dkv_f32<D>), dim3((unsigned)total_ktiles, (unsigned)a.hkv), dim3(256), sm_k, stream, a);
  DAG_LAUNCH_CHECK();
  return DAG_OK;
}

}  // namespace

// Head groupings that leave heads over (G not a multiple of four, at head dimension 64 of two): the tile
// lists of the dQ workgroups that take several query tiles (an int32 and, not used any more, a byte per
// entry of the dense block map, three int32 per query tile).
static size_t bwd_wide_list_bytes(const dag_meta_t* m, int32_t hq, int32_t hkv, int32_t head_dim) {
  if (hq % hkv != 0 || bwd_wide_heads(hq / hkv, head_dim) == 0 || m->sizes.total_tiles < 0) return 0;
  return dag_align_up((size_t)m->sizes.total_tiles * 4, 256) + dag_align_up((size_t)m->sizes.total_tiles, 256) +
         3 * dag_align_up((size_t)(m->sizes.total_qtiles + 1) * 4, 256);
}

// Forward and backward, block map : streams, nodes of 16 / 24 / 32 / 64 / 144 tokens on average: 32 / 8 heads of
// dimension 128 1.00 / 1.02 / 1.02 / 1.06 / 1.08, 16 / 8 heads of dimension 64 1.00 / 1.05 / 1.06 / 1.07 / 1.07.
static bool bwd_dkv_on_stream(const dag_meta_t* m, int32_t hq, int32_t head_dim) {
  return !bwd_first_version() && m->node_tok_start && m->words_per_node <= 2 && m->sizes.total_tokens * hq * head_dim <= (int64_t)UINT32_MAX &&
         m->sizes.total_tokens >= 16 * m->sizes.total_nodes;  // (row offsets are 32-bit)
}

// Pieces of split pairs a KV head (see bwd_order): what an even share of the tiles asks for on 256 compute units (two
// workgroups on each at head dimension 64), or what all tiles of the block map can give.
static int64_t bwd_max_split(const dag_meta_t* m, int32_t hq, int32_t hkv, int32_t head_dim) {
  if (hq % hkv != 0 || !bwd_dkv_on_stream(m, hq, head_dim) || m->sizes.total_tiles < 0) return 0;
  const int64_t G = hq / hkv, most = (m->sizes.total_tiles + m->sizes.total_qtiles) / 2;  // tiles of all pairs
  const int64_t even = ((head_dim == 128 ? 256 : 512) * 2 + hkv - 1) / hkv;
  const int64_t cap = (DKV_MIN_STEPS + G - 1) / G;
  return m->sizes.total_qtiles > cap ? std::min(even, 2 * most / cap) : 0;  // (a pair has as many tiles as its sequence at most)
}
static int64_t bwd_piece_slots(const dag_meta_t* m, int64_t max_split) { return (m->sizes.total_ktiles + m->n_seqs) / 2 + max_split; }
static size_t bwd_piece_bytes(const dag_meta_t* m, int32_t hq, int32_t hkv, int32_t head_dim) {
  const int64_t n = bwd_max_split(m, hq, hkv, head_dim);
  return n == 0 ? 0 : dag_align_up((size_t)bwd_piece_slots(m, n) * 8 + (size_t)n * 4 + 8, 256) + (size_t)n * hkv * (2 * BN) * head_dim * 2 * 4;
}

extern "C" size_t dag_prefill_bwd_workspace_bytes(const dag_meta_t* m, int32_t hq, int32_t hkv, int32_t head_dim) {
  if (!m || hq < 1 || hkv < 1 || head_dim < 1 || m->sizes.total_tokens < 0 || m->sizes.total_qtiles < 0 ||
      m->sizes.total_ktiles < 0)
    return 0;
  // delta and -lse log2(e) [T][hq] fp32 each, weight and launch order of the key tiles, first visibility word per token
  size_t n = 2 * dag_align_up((size_t)m->sizes.total_tokens * hq * 4, 256) +
             2 * dag_align_up((size_t)m->sizes.total_ktiles * 4, 256) +
             dag_align_up((size_t)m->sizes.total_tokens * 8, 256) + 256;
  return n + bwd_wide_list_bytes(m, hq, hkv, head_dim) + bwd_piece_bytes(m, hq, hkv, head_dim);
}

// dQ on query chunks (see launch_d of the forward for where they pay).  Their tables are built in dK, which the
// dQ kernels neither read nor write and the dK / dV kernels, started behind them, overwrite whole.
static bool bwd_dq_on_chunks(const dag_meta_t* m, const BwdArgs& a, int32_t head_dim) {
  const int64_t T = m->sizes.total_tokens, n = m->sizes.total_nodes;
  if (!m->node_tok_start || n < 1 || m->words_per_node > 2 || bwd_first_version()) return false;
  const size_t dk_bytes = (size_t)T * a.hkv * head_dim * 2;
  if (dk_bytes > UINT32_MAX || DAG_SCHED_INTS * 4 + prefill_node_table_bytes(T, n) > dk_bytes) return false;  // (row offsets are 32-bit)
  auto apart = [&](const void* p, size_t bytes) {
    return (const char*)p + bytes <= (const char*)a.dk || (const char*)a.dk + dk_bytes <= (const char*)p;
  };
  const size_t q_bytes = (size_t)a.total_rows * head_dim * 2;
  if (!apart(a.q, q_bytes) || !apart(a.dout, q_bytes) || !apart(a.out, q_bytes) || !apart(a.dq, q_bytes) ||
      !apart(a.k, dk_bytes) || !apart(a.v, dk_bytes) || !apart(a.lse, (size_t)a.total_rows * 4))
    return false;
  // Forward and backward, block map : chunks (of 256 rows of one head to 32 of eight), 64 random nodes of 17 / 24 / 36 / 55 tokens on
  // average, dimension 128: 16 / 8 heads 1.09 / 1.15 / 1.21 / 1.29 (four times, once 1.12 to 1.24), 40 / 8 heads - / 1.23 / 1.28 / 1.37;
  // 80 batches of 2, 3, 5, 6 and 7 heads, nodes of 16 to 62 tokens 0.99 and more; 32 / 8 heads before the heads were
  // packed 1.06 / 1.05 / 1.06 from 24 tokens on, 16 / 8 heads of dimension 64 1.09 / 1.05 / 1.10.
  // One head of dimension 128 fills 256 rows with a node of 16 to 32 tokens: where such items are ten and more for a compute unit and their
  // streams short, chunks cost more than tiles (random nodes of 16 to 30 tokens, sequences of 300 to 1000, 8 to 32 heads 0.86 to
  // 0.96, forks 1.00 to 1.11).  Fewer items 0.92 to 1.56, longer streams 0.92 to 1.11, longer nodes 0.94 to 1.33 (120 batches).
  if (head_dim == 128 && a.G == 1 && T < 32 * n && T < 1000 * (int64_t)a.n_seqs && n * a.hkv >= 2560) return false;
  return T >= 16 * n;
}

extern "C" int dag_attn_prefill_bwd(const dag_meta_t* m, const void* q, const void* k, const void* v, const void* out,
                                    const void* dout, const float* lse, void* dq, void* dk, void* dv, int32_t hq,
                                    int32_t hkv, int32_t head_dim, float softmax_scale, dag_dtype_t dtype, void* ws,
                                    size_t ws_bytes, void* stream) {
  if (!m) return DAG_ERR_NULL;
  if (dtype != DAG_BF16 && dtype != DAG_F32) return DAG_ERR_UNSUPPORTED;
  if (hq < 1 || hkv < 1 || hq % hkv != 0 || (head_dim != 64 && head_dim != 128)) return DAG_ERR_UNSUPPORTED;
  if (m->tile_m != BM || m->tile_n != BN) return DAG_ERR_UNSUPPORTED;
  if (m->n_seqs < 0 || m->sizes.total_tokens < 0 || m->words_per_node < 1) return DAG_ERR_BAD_LEN;
  if (m->n_seqs == 0 || m->sizes.total_tokens == 0) return DAG_OK;
  if (!q || !k || !v || !out || !dout || !lse || !dq || !dk || !dv) return DAG_ERR_NULL;
  if (!m->cu_seqlens || !m->node_start || !m->tok_node || !m->node_vis || !m->qtile_start || !m->ktile_start ||
      !m->block_map_off || !m->block_map || !m->qtile_order || !m->qtile_desc || !m->qtile_col || !m->qtile_flag)
    return DAG_ERR_NULL;
  if (!dag_aligned16(q) || !dag_aligned16(k) || !dag_aligned16(v) || !dag_aligned16(out) || !dag_aligned16(dout) ||
      !dag_aligned16(dq) || !dag_aligned16(dk) || !dag_aligned16(dv))
    return DAG_ERR_ALIGN;
  if (m->sizes.total_tokens * (int64_t)hq > INT32_MAX) return DAG_ERR_UNSUPPORTED;
  if (m->sizes.total_qtiles != m->sizes.total_ktiles) return DAG_ERR_BAD_LEN;  // (both tilings are 64 rows)
  // (a workspace without room for the pieces is taken, too: every pair is then one workgroup's)
  size_t need = dag_prefill_bwd_workspace_bytes(m, hq, hkv, head_dim);
  const size_t piece_bytes = bwd_piece_bytes(m, hq, hkv, head_dim);
  const bool in_pieces = piece_bytes > 0 && ws_bytes >= need;
  need -= piece_bytes;
  // (the lists came later at head dimension 64: a workspace without them is taken, the heads left over then
  // run on one query tile, half of their workgroup idle)
  const bool lists = ws_bytes >= need;
  if (!ws || ws_bytes < need - (head_dim == 64 ? bwd_wide_list_bytes(m, hq, hkv, head_dim) : 0)) return DAG_ERR_WORKSPACE;
  if (dtype == DAG_F32) {
    BwdArgsF32 f;
    f.q = (const float*)q; f.k = (const float*)k; f.v = (const float*)v;
    f.out = (const float*)out; f.dout = (const float*)dout; f.lse = lse;
    f.dq = (float*)dq; f.dk = (float*)dk; f.dv = (float*)dv;
    f.delta = (float*)dag_align_up((size_t)(uintptr_t)ws, 256);
    f.cu_seqlens = m->cu_seqlens; f.node_start = m->node_start; f.tok_node = m->tok_node;
    f.qtile_start = m->qtile_start; f.ktile_start = m->ktile_start;
    f.node_vis = m->node_vis; f.block_map_off = m->block_map_off; f.block_map = m->block_map;
    f.n_seqs = m->n_seqs; f.W = m->words_per_node; f.hq = hq; f.hkv = hkv; f.G = hq / hkv;
    f.scale = softmax_scale;
    hipStream_t s32 = (hipStream_t)stream;
    return head_dim == 128 ? launch_bwd_f32<128>(f, m->sizes.total_qtiles, m->sizes.total_ktiles, s32)
                           : launch_bwd_f32<64>(f, m->sizes.total_qtiles, m->sizes.total_ktiles, s32);
  }
  BwdArgs a;
  a.q = (const uint16_t*)q; a.k = (const uint16_t*)k; a.v = (const uint16_t*)v;
  a.out = (const uint16_t*)out; a.dout = (const uint16_t*)dout;
  a.lse = lse;
  a.dq = (uint16_t*)dq; a.dk = (uint16_t*)dk; a.dv = (uint16_t*)dv;
  a.delta = (float*)dag_align_up((size_t)(uintptr_t)ws, 256);
  a.nlse2 = (float*)((char*)a.delta + dag_align_up((size_t)m->sizes.total_tokens * hq * 4, 256));
  a.kt_weight = (int32_t*)((char*)a.nlse2 + dag_align_up((size_t)m->sizes.total_tokens * hq * 4, 256));
  a.kt_order = a.kt_weight + dag_align_up((size_t)m->sizes.total_ktiles * 4, 256) / 4;
  a.total_ktiles = (int)m->sizes.total_ktiles;
  a.tok_vis0 = (uint64_t*)(a.kt_order + dag_align_up((size_t)m->sizes.total_ktiles * 4, 256) / 4);
  a.wide_col = (int32_t*)((char*)a.tok_vis0 + dag_align_up((size_t)m->sizes.total_tokens * 8, 256));
  a.wide_n = (int32_t*)((char*)a.wide_col + dag_align_up((size_t)m->sizes.total_tiles * 4, 256));
  a.wide_nfast = a.wide_n + dag_align_up((size_t)(m->sizes.total_qtiles + 1) * 4, 256) / 4;
  a.wide_list = a.wide_nfast + dag_align_up((size_t)(m->sizes.total_qtiles + 1) * 4, 256) / 4;
  a.kt_again = (int32_t*)a.tok_vis0;  // (eight bytes a token against four a key tile)
  a.total_qtiles = (int)m->sizes.total_qtiles;
  a.dq_narrow = hq / hkv - (lists ? bwd_wide_heads(hq / hkv, head_dim) : 0);
  a.cu_seqlens = m->cu_seqlens; a.node_start = m->node_start; a.tok_node = m->tok_node;
  a.qtile_start = m->qtile_start; a.ktile_start = m->ktile_start;
  a.qtile_order = m->qtile_order;
  a.qtile_desc = m->qtile_desc; a.qtile_col = m->qtile_col; a.qtile_flag = m->qtile_flag;
  a.node_vis = m->node_vis; a.block_map_off = m->block_map_off; a.block_map = m->block_map;
  a.n_seqs = m->n_seqs; a.W = m->words_per_node; a.hq = hq; a.hkv = hkv; a.G = hq / hkv;
  a.total_rows = (long)m->sizes.total_tokens * hq;
  a.scale = softmax_scale; a.sc = softmax_scale * LOG2E;
  hipStream_t s = (hipStream_t)stream;
  a.node_tok_start = m->node_tok_start;
  a.dkv_stream = bwd_dkv_on_stream(m, hq, head_dim);
  a.pieces = nullptr;
  a.max_split = 0;
  a.again = false;
  if (in_pieces) {
    a.kt_again = a.kt_order;  // (the pieces have their own order)
    a.max_split = (int)bwd_max_split(m, hq, hkv, head_dim);
    char* const at = (char*)a.delta + need - 256;  // (the first 256 bytes of the need are for the alignment of ws)
    a.pieces = (int2*)at;
    a.n_pieces = (int32_t*)(a.pieces + bwd_piece_slots(m, a.max_split));
    a.split_first = a.n_pieces + 2;
    a.part = (f32x4*)(at + piece_bytes - (size_t)a.max_split * hkv * (2 * BN) * head_dim * 2 * 4);
  }
  a.runs = nullptr;
  a.slots = 0;
  a.block_start = nullptr;
  PrefillArgs p = {};
  if (bwd_dq_on_chunks(m, a, head_dim)) {
    p.n_seqs = m->n_seqs; p.W = m->words_per_node;
    p.total_tokens = m->sizes.total_tokens; p.total_nodes = m->sizes.total_nodes;
    p.cu_seqlens = m->cu_seqlens; p.node_start = m->node_start; p.tok_node = m->tok_node; p.node_vis = m->node_vis;
    p.node_tok_start = m->node_tok_start;
    p.sched = (int32_t*)dk;
    p.pack_heads = a.pack_heads = bwd_pack_heads(a.G);
    p.pack_rows = a.pack_rows = 32 * PACK_WAVES(head_dim) / a.pack_heads;
    prefill_node_tables(p, p.sched + DAG_SCHED_INTS);
    a.chunk = p.chunk[DAG_CHUNK_PACK];
    a.slots = chunk_slots(p.total_tokens, p.total_nodes, p.pack_rows);
    a.runs = p.node_runs;
    a.tok_depth = p.tok_depth;
    // Blocks cut at node borders are more than the pairs that the piece list has room for, so it lies behind their first keys in the
    // place of the words that dQ does not read on chunks (eight bytes a token).  Below 4096 tokens the 2 to 4 us of cut_keys
    // are more than forks give back (68 and 118 us: 0.98), and with one head a group a workgroup has as few
    // iterations as it costs (2 x 52 and 5 x 97 random nodes, 2 / 2 heads of dimension 128: 0.96 and 0.98).
    const int64_t blocks = bwd_cut_blocks(p.total_tokens, p.total_nodes, a.total_ktiles, a.n_seqs);
    const size_t start_bytes = dag_align_up((size_t)a.total_ktiles * 4, 8);
    if (a.pieces && a.dkv_stream && a.G >= 2 && p.total_tokens >= 4096 && start_bytes + (size_t)(blocks + a.max_split) * 8 <= (size_t)p.total_tokens * 8) {
      a.block_start = (int32_t*)a.tok_vis0;
      a.pieces = (int2*)((char*)a.tok_vis0 + start_bytes);
    }
  }
  return head_dim == 128 ? launch_bwd<128>(a, p, m->sizes.total_qtiles, m->sizes.total_ktiles, s)
                         : launch_bwd<64>(a, p, m->sizes.total_qtiles, m->sizes.total_ktiles, s);
}
