// Branch-parallel decode over a paged KV cache (paper section 3.2: tokens carry KV-cache
// references; section 4.3 Fork: sibling branches share the prefix KV without copying).
//
// dag_kv_append_rope : store each live branch's new (rotated) key and value into its tail page.
// dag_attn_decode    : cascade attention.  One launch of independent single-wave work items:
//     shared items  (group, kv head, 32-row block, page split): the queries of ALL siblings of the
//                   group (siblings x query heads of the kv head, stacked as MFMA columns) against
//                   a slice of the shared pages -- each shared page is fetched once per group;
//     own items     (branch, kv head, page split): the branch's query heads against its own pages.
//   Every item writes an un-normalised partial (o, m, l); a second launch merges the partials of
//   each (branch, head) by log-sum-exp.  Steps over short contexts are one launch of k_whole_branch.
//
// Pool formats (bf16, 16 tokens per page) are chosen so that global loads land directly in MFMA
// operand layout, fully coalesced, with no LDS staging:
//   K pool [P][hkv][D/8][16][8] : for a fixed 8-wide d-chunk the 16 keys of a page are contiguous;
//                                 one load instruction of a wave reads 2 x 512 contiguous bytes.
//   V pool [P][hkv][D][16]      : for a fixed d the 16 keys of a page are contiguous (the
//                                 contraction dimension of P.V); one load reads 1 KiB contiguous.
// Scores are computed transposed (S^T = K Q^T, 32 keys x 32 query rows per MFMA block) and MFMA
// row i is mapped to key pi(i), so the probabilities come out of the first product already in the
// B-operand layout of the second (O^T = V^T P^T).
#include <stdlib.h>

#include <mutex>
#include <type_traits>

#include "common.h"
#include "decode_plan.h"

namespace {

struct DecodeArgs {
  const int32_t* group_branch_off;
  const int32_t* shared_page_off;
  const int32_t* shared_pages;
  const int32_t* shared_len;
  const int32_t* branch_page_off;
  const int32_t* branch_pages;
  const int32_t* branch_len;
  const uint16_t* q;
  const uint16_t* k_pool;
  const uint16_t* v_pool;
  uint16_t* out;
  float* part_o_a;   // [items_a][32][D]
  float* part_ml_a;  // [items_a][32][2]
  float* part_o_b;   // [items_b][G][D]
  float* part_ml_b;  // [items_b][G][2]
  int n_groups, n_live, hq, hkv, G;
  int rb_max;        // 32-row blocks per (group, kv head)
  int chunk_a, splits_a, chunk_b, splits_b;
  int items_a, items_b;
  int item_base;     // first work item of this launch (k_decode)
  int wide_shared;   // k_decode_wide: workgroups that take shared items (the rest take own pages)
  int wide_first;    // k_decode_wide: workgroups with own pages that are launched before them
  int wide_own;      // k_decode_wide: waves of a workgroup that share an own item
  float sc;          // softmax_scale * log2(e)
  float th;          // how far a score may exceed the reference maximum before it is raised
  float settle;      // k_decode_wide, shared pages: growth of a lane's sum of 16 probabilities from which on the reference is looked after
  float scale;
};

// Decode over lists of KV segments: a segment is a page list with a token count and the set of
// live branches that read it; a branch's context is the union of the segments it reads.
struct SegItem {  // one work item: a slice of a segment's pages against one 32-row block of its readers' rows
  int32_t page_off, len, e0, nrows, row0;
  int32_t p0, place;  // first page of the slice; place of its partial of reader e0
  int32_t nsplit;     // slices of the segment, pages of a slice / 2 in the highest eight bits (unless SegArgs::fixed)
};
static_assert(sizeof(SegItem) == SEG_ITEM_BYTES, "");
struct SegArgs {
  const int32_t* seg_page_off;
  const int32_t* seg_pages;
  const int32_t* seg_len;
  const int32_t* seg_reader_off;
  const int32_t* seg_readers;
  const int32_t* seg_reader_len;  // optional: leading tokens of the segment each reader-list entry sees
  const int32_t* branch_entry_off;
  const int32_t* branch_entries;
  const uint16_t* q;
  const uint16_t* k_pool;
  const uint16_t* v_pool;
  uint16_t* out;
  float* part_o;   // [splits * total_readers][hq][D]: the slices of every reader-list entry one after another
  float* part_ml;  // [splits * total_readers][hq][2]
  SegItem* items;        // [item_cap] compact list of (segment, row block, slice), written by k_seg_plan
  int32_t* totals;       // number of list entries, place behind the last partial, most slices of a segment
  int32_t* entry_first;  // [total_readers] place of the first partial of each reader-list entry (the next one's: behind its last)
  int item_cap;
  int n_segments, n_live, hq, hkv, G;
  int rb_max;      // 32-row blocks per (segment, kv head)
  int chunk, splits, total_readers;  // pages of a slice and slices of a segment that the workspace has room for
  bool fixed;      // slices of `chunk` pages, whatever there is to read
  bool few;        // by the host's bounds the slices have eight pages
  float weight;    // of a page: hkv * D / 128
  float sc, th;
};

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
typedef __attribute__((ext_vector_type(8))) float f32x8;

// MFMA row i (0..31) of a 32-key block -> (page 0/1, slot 0..15): registers 0..7 / 8..15 of the
// transposed score block then hold slots 8H..8H+7 of page 0 / page 1.
__device__ __forceinline__ int key_of_row(int i) {
  const int a = i >> 3, hh = (i >> 2) & 1, c = i & 3;
  return 16 * (a >> 1) + 8 * hh + 4 * (a & 1) + c;
}

template <int D>
struct KVBlock {           // one 32-key block (2 pages) in operand layout
  bf16x8 k[D / 16];        // k[s]: d-chunk 2s+H of key pi(L)
  bf16x8 v[2][D / 32];     // v[page][db]: keys 8H..8H+7 of dimension 32db+L
};

// pgv: page ids of the item's slice, lane i holds page p0 + (i % 64) of the current 64-page window
// (fetched once per window, so that no page-table load sits in front of every K/V load)
template <int D, typename A>
__device__ __forceinline__ void load_block(KVBlock<D>& blk, const A& a, int pgv, int pb_rel, int last_rel,
                                           int hk, int L, int H, int kpage_sel, int kslot) {
  const int pg0 = __builtin_amdgcn_readlane(pgv, pb_rel & 63);
  const int pg1 = __builtin_amdgcn_readlane(pgv, min(pb_rel + 1, last_rel) & 63);
  const size_t kbase0 = ((size_t)pg0 * a.hkv + hk) * (size_t)(D * PAGE);
  const size_t kbase1 = ((size_t)pg1 * a.hkv + hk) * (size_t)(D * PAGE);
  const uint16_t* kp = a.k_pool + (kpage_sel ? kbase1 : kbase0) + kslot * 8 + H * (PAGE * 8);
#pragma unroll
  for (int s = 0; s < D / 16; ++s) blk.k[s] = *(const bf16x8*)(kp + s * (2 * PAGE * 8));
  const uint16_t* vp0 = a.v_pool + kbase0 + L * PAGE + H * 8;
  const uint16_t* vp1 = a.v_pool + kbase1 + L * PAGE + H * 8;
#pragma unroll
  for (int db = 0; db < D / 32; ++db) {
    blk.v[0][db] = *(const bf16x8*)(vp0 + db * 32 * PAGE);
    blk.v[1][db] = *(const bf16x8*)(vp1 + db * 32 * PAGE);
  }
}

// qop(s): the query operand of MFMA step s.  k_decode keeps the operands in LDS, qs[s * 64 + lane]
// (they are needed once per 32-key block; keeping them out of the register file lets two waves
// share a SIMD, which doubles the bytes in flight); k_decode_wide keeps them in registers.
// First phase of a 32-key block: scores against the key operands, online softmax bookkeeping
// (accumulators rescaled when the reference maximum moves), probabilities as the two B operands
// of the second phase.
template <int D, typename QF>
__device__ __forceinline__ void block_scores(const bf16x8 (&kop)[D / 16], QF&& qop, f32x16* O, float& m, float& l,
                                             float sc, float th, int key0, int len, int lim, int H,
                                             bf16x8& pb0, bf16x8& pb1) {
  f32x16 S;
#pragma unroll
  for (int r = 0; r < 16; ++r) S[r] = 0.f;
#pragma unroll
  for (int s = 0; s < D / 16; ++s) S = mfma32(kop[s], qop(s), S);
  if (key0 + 32 > len) {  // len: wave-uniform, the smallest of the rows' limits; lim: this lane's row
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = key0 + 16 * (r >> 3) + 8 * H + (r & 7);
      S[r] = key < lim ? S[r] : -INFINITY;
    }
  }
  float bm = S[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) bm = fmaxf(bm, S[r]);
  bm = fmaxf(bm, __shfl_xor(bm, 32));
  // The reference maximum m is raised only when some row of the wave exceeds it by more than th; the rescale of the accumulators
  // is then rare, and probabilities above one are absorbed exactly by fp32 accumulation and the final division.
  if (__builtin_amdgcn_ballot_w64(bm > m + th) != 0) {
    const float m_new = fmaxf(m, bm);
    if (__builtin_amdgcn_ballot_w64(m > -1e30f) != 0) {  // (the first block finds zeros: what a step of a few blocks loses by the nearer reference)
      const float alpha = __builtin_amdgcn_exp2f((m - m_new) * sc);
      l *= alpha;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[db][r] *= alpha;
    }
    m = m_new;
  }
  const float msc = m * sc;
  f32x8 p0, p1;
  float rowsum = 0.f;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    p0[r] = __builtin_amdgcn_exp2f(fmaf(S[r], sc, -msc));
    p1[r] = __builtin_amdgcn_exp2f(fmaf(S[8 + r], sc, -msc));
    rowsum += p0[r] + p1[r];
  }
  l += rowsum;
  pb0 = __builtin_convertvector(p0, bf16x8);
  pb1 = __builtin_convertvector(p1, bf16x8);
}

// Second phase: O^T += V^T P^T with the value operands of the block's two pages.
template <int D>
__device__ __forceinline__ void block_pv(const bf16x8 (&v0)[D / 32], const bf16x8 (&v1)[D / 32], bf16x8 pb0,
                                         bf16x8 pb1, f32x16* O) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db) {
    O[db] = mfma32(v0[db], pb0, O[db]);
    O[db] = mfma32(v1[db], pb1, O[db]);
  }
}

// Value operands of a block that reaches past the `vlen` tokens its page list holds: the slots
// behind the last token (and the page that a slice with an odd page count reads twice) may hold
// anything, NaN or infinity bit patterns included, and a zero probability does not neutralise
// those in the product, so their elements are cleared.  v0 / v1 hold keys 8 H .. 8 H + 7 of the
// block's first / second page.
template <int D>
__device__ __forceinline__ void clear_unused_values(bf16x8 (&v0)[D / 32], bf16x8 (&v1)[D / 32], int key0, int vlen,
                                                    int H) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {  // 32-bit word w of an operand = keys 8 H + 2 w, 8 H + 2 w + 1 of the page
    const int k0 = key0 + 8 * H + 2 * w, k1 = k0 + 16;
    const uint32_t m0 = (k0 < vlen ? 0x0000ffffu : 0u) | (k0 + 1 < vlen ? 0xffff0000u : 0u);
    const uint32_t m1 = (k1 < vlen ? 0x0000ffffu : 0u) | (k1 + 1 < vlen ? 0xffff0000u : 0u);
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
      u32x4 a = __builtin_bit_cast(u32x4, v0[db]), b = __builtin_bit_cast(u32x4, v1[db]);
      a[w] &= m0;
      b[w] &= m1;
      v0[db] = __builtin_bit_cast(bf16x8, a);
      v1[db] = __builtin_bit_cast(bf16x8, b);
    }
  }
}

// vlen: tokens the page list holds (wave-uniform); len <= vlen: the smallest of the rows' limits.
// The block's value operands are cleared in place where they reach past vlen (the block is dead
// after this call: its registers are refilled by the next load).
template <int D, typename QF>
__device__ __forceinline__ void compute_block(KVBlock<D>& blk, QF&& qop, f32x16* O, float& m, float& l,
                                              float sc, float th, int key0, int len, int lim, int vlen, int H) {
  bf16x8 pb0, pb1;
  block_scores<D>(blk.k, qop, O, m, l, sc, th, key0, len, lim, H, pb0, pb1);
  if (key0 + 32 > vlen) clear_unused_values<D>(blk.v[0], blk.v[1], key0, vlen, H);
  block_pv<D>(blk.v[0], blk.v[1], pb0, pb1, O);
}

// The loop of a single-wave work item: pages [p0, p1) of one page list, 32 keys (two pages) per
// step, the next block's loads in flight while the current one is computed.  `lim` is the number
// of leading tokens of the list that this lane's row sees (keys at or past it are masked), `len`
// the smallest `lim` of the wave, `vlen` the number of tokens the list holds.  Leaves the un-normalised partial
// (O, reference maximum m, row sum l of this lane's half) in registers.
template <int D, typename A, typename QF>
__device__ __forceinline__ void stream_slice(const A& a, const int32_t* pages, int p0, int p1, int len, int lim,
                                             int vlen, int hk, int lane, QF&& qop, f32x16* O, float& m, float& l) {
  const int L = lane & 31, H = lane >> 5;
  const int kr = key_of_row(L);
  const int kpage_sel = kr >> 4, kslot = kr & 15;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) O[db][r] = 0.f;
  m = -1e30f;
  l = 0.f;

  // Page ids in windows of 64 (lane i: page p0 + 64 w + i); a block never straddles a window
  // because windows and blocks both start at even offsets.
  const int np = p1 - p0;
  int pgv = pages[p0 + min(lane, np - 1)];
  asm volatile("" ::"v"(pgv));  // arrived: a wait for it inside the loop would also wait for the K/V loads in flight
  KVBlock<D> b0, b1;
  load_block<D>(b0, a, pgv, 0, np - 1, hk, L, H, kpage_sel, kslot);
  int pb = 0;  // relative to p0
  while (true) {
    if (pb + 2 < np) {
      if (((pb + 2) & 63) == 0) {
        pgv = pages[p0 + min(pb + 2 + lane, np - 1)];
        asm volatile("" ::"v"(pgv));
      }
      load_block<D>(b1, a, pgv, pb + 2, np - 1, hk, L, H, kpage_sel, kslot);
    }
    compute_block<D>(b0, qop, O, m, l, a.sc, a.th, (p0 + pb) * PAGE, len, lim, vlen, H);
    pb += 2;
    if (pb >= np) break;
    if (pb + 2 < np) {
      if (((pb + 2) & 63) == 0) {
        pgv = pages[p0 + min(pb + 2 + lane, np - 1)];
        asm volatile("" ::"v"(pgv));
      }
      load_block<D>(b0, a, pgv, pb + 2, np - 1, hk, L, H, kpage_sel, kslot);
    }
    compute_block<D>(b1, qop, O, m, l, a.sc, a.th, (p0 + pb) * PAGE, len, lim, vlen, H);
    pb += 2;
    if (pb >= np) break;
  }
}

template <int D>
__global__ void __launch_bounds__(64, 2) k_decode(DecodeArgs a) {
  __shared__ bf16x8 qs_all[(D / 16) * 64];
  const int item = blockIdx.x + a.item_base;
  const int lane = threadIdx.x, L = lane & 31, H = lane >> 5;
  const bool is_a = item < a.items_a;
  int hk, split, chunk, len, nrows, row0, branch0;
  const int32_t* pages;
  if (is_a) {
    int x = item;
    split = x % a.splits_a; x /= a.splits_a;
    const int rb = x % a.rb_max; x /= a.rb_max;
    hk = x % a.hkv;
    const int g = x / a.hkv;
    branch0 = a.group_branch_off[g];
    nrows = (a.group_branch_off[g + 1] - branch0) * a.G;
    row0 = rb * 32;
    pages = a.shared_pages + a.shared_page_off[g];
    len = a.shared_len[g];
    chunk = a.chunk_a;
  } else {
    int x = item - a.items_a;
    split = x % a.splits_b; x /= a.splits_b;
    hk = x % a.hkv;
    branch0 = x / a.hkv;
    nrows = a.G;
    row0 = 0;
    pages = a.branch_pages + a.branch_page_off[branch0];
    len = a.branch_len[branch0];
    chunk = a.chunk_b;
  }
  const int npages = (len + PAGE - 1) / PAGE;
  const int p0 = split * chunk, p1 = min(p0 + chunk, npages);
  const int row = row0 + L;
  const bool row_ok = row < nrows;

  float* po;
  float* pml;
  if (is_a) {
    po = a.part_o_a + ((size_t)item * 32 + L) * D;
    pml = a.part_ml_a + ((size_t)item * 32 + L) * 2;
  } else {
    po = a.part_o_b + ((size_t)(item - a.items_a) * a.G + L) * D;
    pml = a.part_ml_b + ((size_t)(item - a.items_a) * a.G + L) * 2;
  }
  if (p0 >= p1 || row0 >= nrows) {  // empty slice: neutral partial
    if (row_ok && H == 0) {
      pml[0] = -1e30f;
      pml[1] = 0.f;
    }
    return;
  }

  const bf16x8* qf = qs_all + lane;
  {
    const int rr = row_ok ? row : 0;
    const int br = branch0 + rr / a.G, head = hk * a.G + rr % a.G;
    const uint16_t* qp = a.q + ((size_t)br * a.hq + head) * D + 8 * H;
#pragma unroll
    for (int s = 0; s < D / 16; ++s) qs_all[s * 64 + lane] = *(const bf16x8*)(qp + 16 * s);
  }
  auto qop = [&](int s) { return qf[s * 64]; };
  f32x16 O[D / 32];
  float m, l;
  stream_slice<D>(a, pages, p0, p1, len, len, len, hk, lane, qop, O, m, l);

  const float l_tot = l + __shfl_xor(l, 32);
  if (row_ok) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        f32x4 o = {O[db][4 * r4], O[db][4 * r4 + 1], O[db][4 * r4 + 2], O[db][4 * r4 + 3]};
        *(f32x4*)(po + 32 * db + 8 * r4 + 4 * H) = o;
      }
    if (H == 0) {
      pml[0] = m;
      pml[1] = l_tot;
    }
  }
}

// Segment form, step 1: the work items.  Segment lengths and reader counts live in device memory,
// so a launch sized by the host bounds would consist mostly of items that find nothing to do, and
// those cost time even when they exit at once (they sit between the real items in the dispatch
// order and hold wave slots while their loads return).  One workgroup therefore writes the compact
// list: for every segment, in the caller's order, its slices x row blocks (exclusive scan of the
// counts), and for every reader-list entry the place of its first partial.
//
// The list also settles how long slices are (rules and figures: SEG_PAGES_16 and what follows it).  What that costs is exchanges between
// the waves: one for what there is to read, and the scan of the counts tells whether the lists have room for slices of that length.  294 segments:
// 6.2 us; with the host's slices, which need neither, 4.8; with an exchange for each length that is tried 7.2.  28 segments: 3.4, 3.1, 3.4.
constexpr int PLAN_THREADS = 1024;
__global__ void __launch_bounds__(PLAN_THREADS) k_seg_plan(SegArgs a) {
  __shared__ uint32_t s_all[2][4][PLAN_THREADS / 64];  // (in turn: a barrier between two exchanges)
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, threads = blockDim.x, room = a.splits * a.total_readers;
  struct Seg {
    int len, e0, nr, npages, rbs;
  };
  auto segment = [&](int s) __attribute__((always_inline)) {
    Seg g = {0, 0, 0, 0, 0};
    if (s < a.n_segments) {
      g.len = max(a.seg_len[s], 0);
      g.e0 = a.seg_reader_off[s];
      g.nr = max(a.seg_reader_off[s + 1] - g.e0, 0);
      g.npages = min((g.len + PAGE - 1) / PAGE, a.chunk * a.splits);
      g.rbs = min((g.nr * a.G + 31) / 32, a.rb_max);
    }
    return g;
  };
  const Seg mine = segment(tid);
  static_assert(PLAN_THREADS == 16 * 64, "");
  int turn = 0;
  auto exchange = [&](uint32_t x) __attribute__((always_inline)) {  // 16 lanes have a value of all waves each: that of lane 0, 1, 2, 3
    uint32_t* const all = &s_all[turn & 1][0][0];
    ++turn;
    if (lane < 4) all[lane * (PLAN_THREADS / 64) + w] = x;
    __syncthreads();
    return (lane & 15) < threads / 64 ? all[lane] : 0u;
  };
  auto of_lane = [](float x, int from) __attribute__((always_inline)) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), from));
  };
  struct Sums {
    float x, y, top;
  };
  auto gather = [&](Sums s) __attribute__((always_inline)) {  // sums over all threads (exact up to 2^24), the maximum of the last value
    s = Sums{dag_wave_sum(s.x), dag_wave_sum(s.y), dag_wave_max(s.top)};
    if (threads > 64) {
      const float v = __uint_as_float(exchange(__float_as_uint(lane == 0 ? s.x : lane == 1 ? s.y : s.top)));
      const float sum = dag_wave_sum<8>(v);
      s = Sums{of_lane(sum, 0), of_lane(sum, 16), of_lane(dag_wave_max<8>(v), 32)};
    }
    return s;
  };
  // slices of a segment of at most 2^k pages (an eighth more of the longer ones), and the pages of them if all are alike and even
  // (a 32-key block never straddles two)
  auto longest_slice = [](int k) __attribute__((always_inline)) { return (1 << k) >= SEG_STRETCH ? 9 << (k - 3) : 1 << k; };
  auto slices_of = [&](int npages, int k) __attribute__((always_inline)) {
    const uint32_t x = (uint32_t)(npages + longest_slice(k) - 1);
    return (int)((1 << k) >= SEG_STRETCH ? (x >> (k - 3)) / 9 : x >> k);
  };
  auto slice_of = [&](int npages, int k) __attribute__((always_inline)) {
    const int n = slices_of(npages, k);
    return n > 0 ? (int)((uint32_t)(npages + n - 1) / (uint32_t)n + 1) & ~1 : 1;
  };
  auto fits = [](float n, int most) { return n < 16777216.f ? n <= (float)most : n * 1.001f < (float)most; };
  const bool at_once = a.n_segments <= threads;
  const int host = 31 - __builtin_clz(a.chunk);  // (of a power of two, unless a.fixed)
  int k = a.few ? 3 : host;
  float longest = (float)(a.chunk * a.splits);
  if (!a.few && !a.fixed) {
    Sums sums = {};
    for (int s = tid; s < a.n_segments; s += threads) {
      const Seg g = s == tid ? mine : segment(s);
      sums.x += (float)g.rbs * (float)g.npages;
      sums.y += (float)g.nr * (float)g.npages;
      sums.top = fmaxf(sums.top, (float)g.npages);
    }
    sums = gather(sums);
    longest = sums.top;
    const float pages = sums.x * a.weight;
    k = pages < (longest <= SEG_SHORT ? SEG_PAGES_16_SHORT : SEG_PAGES_16) ? 3 : pages < SEG_PAGES_32 ? 4 : pages < SEG_PAGES_64 ? 5 : pages < SEG_PAGES_128 ? 6 : 7;
    for (; k < host; ++k) {
      const float one = 1.f / (float)longest_slice(k);
      if (!fits(sums.x * one, a.item_cap) || !fits(sums.y * one, room)) continue;
      if (at_once) break;  // (the places tell)
      Sums n = {};
      for (int s = tid; s < a.n_segments; s += threads) {
        const Seg g = s == tid ? mine : segment(s);
        const float nsp = (float)slices_of(g.npages, k);
        n.x += nsp * (float)g.rbs;
        n.y += nsp * (float)g.nr;
      }
      n = gather(n);
      if (fits(n.x, a.item_cap) && fits(n.y, room)) break;
    }
  }
  int start0 = 0, first0 = 0;  // items and partials of the segments in front
  for (int base = 0; base < a.n_segments; base += threads) {
    const int s = base + tid;
    const Seg g = base == 0 ? mine : segment(s);
    int slice, nsp, cnt, parts, start, first;
    for (;; ++k) {
      slice = a.fixed ? a.chunk : slice_of(g.npages, k);
      nsp = (int)((uint32_t)(g.npages + slice - 1) / (uint32_t)slice);
      cnt = nsp * g.rbs;
      parts = nsp * g.nr;
      start = dag_wave_scan(cnt);
      first = dag_wave_scan(parts);
      int items = __builtin_amdgcn_readlane(start, 63), places = __builtin_amdgcn_readlane(first, 63);
      start += start0 - cnt;
      first += first0 - parts;
      if (threads > 64) {
        const uint32_t v = exchange(lane == 0 ? items : places);
        const int front = dag_wave_sum<8>((lane & 15) < w ? (int)v : 0), sum = dag_wave_sum<8>((int)v);
        start += __builtin_amdgcn_readlane(front, 0);
        first += __builtin_amdgcn_readlane(front, 16);
        items = __builtin_amdgcn_readlane(sum, 0);
        places = __builtin_amdgcn_readlane(sum, 16);
      }
      if (a.few || !at_once || k >= host || ((uint32_t)items <= (uint32_t)a.item_cap && (uint32_t)places <= (uint32_t)room)) {
        start0 += items;
        first0 += places;
        break;
      }
    }
    if (s < a.n_segments) {
      int at = start;
      const int page_off = a.seg_page_off[s], code = a.fixed ? nsp : nsp | slice << 23;
      for (int sp = nsp - 1; sp >= 0; --sp)
        for (int rb = 0; rb < g.rbs; ++rb, ++at)
          if (at < a.item_cap) a.items[at] = SegItem{page_off, g.len, g.e0, g.nr * a.G, rb * 32, sp * slice, first + sp, code};
      for (int e = 0; e < g.nr; ++e) {
        if (g.e0 + e >= 0 && g.e0 + e < a.total_readers) a.entry_first[g.e0 + e] = first + e * nsp;
        if (g.e0 + e == a.total_readers - 1) a.totals[1] = first + (e + 1) * nsp;
      }
      const int end = g.e0 + g.nr;  // (fewer entries listed than announced: the last one's partials end here all the same)
      if (s + 1 == a.n_segments && end >= 0 && end < a.total_readers) a.entry_first[end] = first + parts;
    }
  }
  if (tid == 0) {
    a.totals[0] = min(start0, a.item_cap);
    // most slices of a segment, at least (one of more than 2^24 pages is longer than any pool)
    a.totals[2] = a.fixed || a.few ? a.splits : ((int)longest + (1 << k) - 1) >> k;
  }
}

// Step 2: one wave per (work item, kv head).  Row j * G + g of a segment is query head hk * G + g
// of its j-th reader; the partial of a row goes to the reader's entry in the reader list, which is
// where the combination step looks for it.  The launch covers the host's bound on the list; the
// workgroups past its end exit.
template <int D>
__global__ void __launch_bounds__(64, 2) k_decode_seg(SegArgs a) {
  __shared__ bf16x8 qs_all[(D / 16) * 64];
  const int lane = threadIdx.x, L = lane & 31, H = lane >> 5;
  const int hk = blockIdx.x % a.hkv, idx = blockIdx.x / a.hkv;
  if (idx >= a.totals[0]) return;
  const SegItem it = a.items[idx];
  const int len = it.len, e0 = it.e0, nrows = it.nrows, row0 = it.row0;
  const int npages = min((len + PAGE - 1) / PAGE, a.chunk * a.splits), p0 = it.p0;
  const int slice = a.fixed ? a.chunk : (it.nsplit >> 23) & 0x1fe, nsplit = a.fixed ? it.nsplit : it.nsplit & 0xffffff;
  int p1 = __builtin_amdgcn_readfirstlane(min(p0 + slice, npages));
  if (row0 >= nrows || p0 >= p1) return;  // (never listed)
  const int row = row0 + L;
  const bool row_ok = row < nrows;
  const int rr = row_ok ? row : row0;
  const int entry = e0 + rr / a.G, head = hk * a.G + rr % a.G;
  const int place = it.place + rr / a.G * nsplit;
  const bool store_ok = row_ok && entry < a.total_readers && place < a.splits * a.total_readers;  // (reader lists longer than announced: no partial)
  const size_t pbase = (size_t)place * a.hq + head;
  // per-reader visible prefix of the segment (a token of a node being prefilled sees the node's
  // tokens up to itself): the slice ends at the longest prefix of the wave's rows
  int lim = len, lim_min = len;
  if (a.seg_reader_len) {
    lim = min(max(a.seg_reader_len[entry], 0), len);
    int lim_max = lim;
    lim_min = lim;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      lim_max = max(lim_max, __shfl_xor(lim_max, o));
      lim_min = min(lim_min, __shfl_xor(lim_min, o));
    }
    p1 = min(p1, (lim_max + PAGE - 1) / PAGE);
    if (p0 >= p1) {  // no row of this block sees a token of the slice: neutral partial
      if (store_ok && H == 0) {
        a.part_ml[pbase * 2] = -1e30f;
        a.part_ml[pbase * 2 + 1] = 0.f;
      }
      return;
    }
  }
  const int br = min(max(a.seg_readers[entry], 0), a.n_live - 1);

  const bf16x8* qf = qs_all + lane;
  {
    const uint16_t* qp = a.q + ((size_t)br * a.hq + head) * D + 8 * H;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) qs_all[t * 64 + lane] = *(const bf16x8*)(qp + 16 * t);
  }
  auto qop = [&](int t) { return qf[t * 64]; };
  f32x16 O[D / 32];
  float m, l;
  stream_slice<D>(a, a.seg_pages + it.page_off, p0, p1, lim_min, lim, len, hk, lane, qop, O, m, l);

  const float l_tot = l + __shfl_xor(l, 32);
  if (store_ok) {
    float* po = a.part_o + pbase * D;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        f32x4 o = {O[db][4 * r4], O[db][4 * r4 + 1], O[db][4 * r4 + 2], O[db][4 * r4 + 3]};
        *(f32x4*)(po + 32 * db + 8 * r4 + 4 * H) = o;
      }
    if (H == 0) {
      a.part_ml[pbase * 2] = m;
      a.part_ml[pbase * 2 + 1] = l_tot;
    }
  }
}

// Step 3: one wave per (branch, query head): log-sum-exp combination over the slices of every
// segment the branch reads.  The branch's entries in the reader lists name its partials, which end
// where those of the next entry begin; the lanes fetch the
// (maximum, sum) pairs of up to 64 (entry, split) pairs at once, the wave agrees on the maximum
// and the weights, and the weighted partial outputs are added pair by pair.  A branch without any
// key gets zeros.
template <int D>
__global__ void __launch_bounds__(64) k_decode_seg_merge(SegArgs a) {
  const int r = blockIdx.x / a.hq, head = blockIdx.x % a.hq;
  const int lane = threadIdx.x;
  constexpr int PER = D / 64;  // output elements per lane
  float acc[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] = 0.f;
  float mx = -1e30f, lsum = 0.f;
  const int e0 = a.branch_entry_off[r];
  const int splits = a.splits > 0 ? a.totals[2] : 0;
  const int npairs = (a.branch_entry_off[r + 1] - e0) * splits;
  for (int b = 0; b < npairs; b += 64) {
    const int i = b + lane;
    float ms = -1e30f, ls = 0.f;
    uint32_t base = 0;
    if (i < npairs) {
      const int entry = a.branch_entries[e0 + i / splits];
      int place = -1, behind = -1;  // of this partial, of the entry's last one
      if (entry >= 0 && entry < a.total_readers) {
        place = a.entry_first[entry] + i % splits;
        behind = entry + 1 < a.total_readers ? a.entry_first[entry + 1] : a.totals[1];
      }
      if (place >= 0 && place < min(behind, a.splits * a.total_readers)) {
        base = (uint32_t)((size_t)place * a.hq + head);
        const float2 ml = *(const float2*)(a.part_ml + (size_t)base * 2);
        if (ml.y > 0.f) {
          ms = ml.x;
          ls = ml.y;
        }
      }
    }
    const float mn = fmaxf(mx, dag_wave_max(ms));
    const float keep = __builtin_amdgcn_exp2f((mx - mn) * a.sc);
    const float wgt = ls > 0.f ? __builtin_amdgcn_exp2f((ms - mn) * a.sc) : 0.f;
    lsum = lsum * keep + dag_wave_sum(ls * wgt);
    mx = mn;
#pragma unroll
    for (int t = 0; t < PER; ++t) acc[t] *= keep;
    unsigned long long live = __builtin_amdgcn_ballot_w64(ls > 0.f);
    auto add = [&](auto batch_c) __attribute__((always_inline)) {  // BATCH partials at a time, their loads in flight together
      constexpr int BATCH = decltype(batch_c)::value;
      float w[BATCH], x[BATCH][PER];
      int n_live = 0, j = 0;
#pragma unroll
      for (int n = 0; n < BATCH; ++n) {
        if (live) {
          j = __builtin_ctzll(live);
          live &= live - 1;
          n_live = n + 1;
        }
        w[n] = __shfl(wgt, j);
        const float* o = a.part_o + (size_t)(uint32_t)__shfl((int)base, j) * D + lane * PER;  // (past the last one: that one again)
#pragma unroll
        for (int t = 0; t < PER; ++t) x[n][t] = o[t];
      }
#pragma unroll
      for (int n = 0; n < BATCH; ++n)
#pragma unroll
        for (int t = 0; t < PER; ++t) acc[t] = n < n_live ? fmaf(w[n], x[n][t], acc[t]) : acc[t];
    };
    // (as many as there are: 1024 times two branches with two or three partials take 48.9 us eight at a time, 47.3 so)
    while (live) {
      const int left = __popcll(live);
      if (left <= 2) add(std::integral_constant<int, 2>{});
      else if (left <= 4) add(std::integral_constant<int, 4>{});
      else add(std::integral_constant<int, 8>{});
    }
  }
  const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
  uint16_t* o = a.out + ((size_t)r * a.hq + head) * D + lane * PER;
  if (PER == 2) {
    *(uint32_t*)o = dag_pack_bf2(acc[0] * inv, acc[PER - 1] * inv);
  } else {
    o[0] = (uint16_t)dag_f2bf(acc[0] * inv);
  }
}

// Wide sibling groups (more than 32 stacked query rows per KV head, e.g. 32 siblings x 5 query heads).
//
// Shared items: a workgroup of eight waves per (group, kv head, page slice), a wave per 32-row block, so that the
// shared pages are streamed once per group whatever the number of rows (two row blocks leave four waves to the loads alone; with
// six waves of the form before it 62 such shapes took 1.29 times as long).  The waves read the same K/V tiles of 64
// keys (four pages) from rings in LDS that are filled directly from the pools (a page is the operand image).  Up to
// four row blocks are served by two waves each, one for either half of every tile, with accumulators of
// their own that are put together at the end.
// A wave walks its 32-key units in a pipeline: in one run of slots it takes the scores of unit u, the
// exponentials of unit u - 1 and the P V product of unit u - 2, a slot being one operand read, one MFMA and a share
// of the exponentials; the two products alternate, so that consecutive MFMAs do not depend on each other.
// The reference maximum, that of the first two units, is not looked after before the exponentials: a lane's sum of 16
// probabilities tells afterwards whether a score left the range.
// Own items: (branch, kv head, page slice) in workgroups of the same launch; every wave streams a part of an item's
// pages as k_decode does and the partials are put together in LDS.
// Five and six row blocks: a tile takes as long as the SIMD with the most to do, and four waves with
// two units of a tile each leave the others a unit or none.  Four row blocks have a wave each; the waves
// 4 .. 7 share what is left, one half of every tile each (six) or of every second one (five): 105 -> 99 us.
// 2 groups of 32 siblings x 5 heads on 8 KV heads, 32 K shared and 640 own tokens (436 MB): 128 us with units in
// read - wait - multiply phases by ten waves, 91 us so = 4.8 TB/s; the matrix pipes need 17 us of it.
constexpr int WIDE_RING = 4;         // tiles in the K ring and in the V ring
// dynamic LDS of a launch: the rings, or the query operands and the partials of the own items
inline int wide_lds_bytes(int G, int D, int own) {
  const int rings = 2 * WIDE_RING * WIDE_TILE_PAGES * PAGE * D * 2, bytes = wide_own_bytes(G, D, own);
  return rings > bytes ? rings : bytes;
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {  // s_waitcnt vmcnt(N) only (gfx9 encoding)
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
template <int N>
__device__ __forceinline__ void wait_lgkmcnt() { __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8)); }
// f(integral_constant<int, I>) for I = A .. B - 1, each a separate instantiation
template <int A, int B, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (A < B) {
    f(std::integral_constant<int, A>{});
    static_for<A + 1, B>(f);
  }
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {  // byte address inside LDS of a __shared__ pointer
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// One shared item.  pages: the np pages of the slice, ntok: the tokens they hold; qrow: this lane's query row.
// On return (O, m, l) hold the un-normalised partial of the units this wave took (l of this lane's half of the keys only).
// HALVES 2: units of key half `sub` of every tile.  HALVES 1: all units; parts 2: key half `sub` of every
// tile, parts 4: key half sub % 2 of every second tile from sub / 2 on.
template <int D, int HALVES, typename A>
__device__ __forceinline__ void wide_item(const A& a, unsigned char* smem, const int32_t* pages, int np, int ntok, int hk,
                                          const uint16_t* qrow, int w, int lane, int sub, int parts, bool active, f32x16* O,
                                          float& m, float& l) {
  constexpr int PB = PAGE * D * 2, TB = WIDE_TILE_PAGES * PB;  // bytes of a page, a tile of one pool
  constexpr int KS = D / 16, DB = D / 32, NS = KS + 2 * DB;    // slots of a unit
  constexpr int IP = PB / 1024 / 2;                            // 1 KiB pieces of a page that a wave fetches
  constexpr int LPG = 2 * IP;                                  // a wave's loads per group
  constexpr int LAG = HALVES;                                  // V is read so many tiles behind K
  constexpr int PF = 3, OPR = 4;                               // operand reads in flight ahead, their registers
  const int L = lane & 31, H = lane >> 5;
  unsigned char *const Kring = smem, *const Vring = smem + WIDE_RING * TB;

  const int pg_a = pages[min(lane, np - 1)], pg_b = pages[min(lane + 64, np - 1)];
  bf16x8 qf[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) qf[s] = *(const bf16x8*)(qrow + 8 * H + 16 * s);
  // (arrived: a wait for them further down would also wait for the tiles in flight)
  asm volatile("" ::"v"(pg_a), "v"(pg_b));
#pragma unroll
  for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qf[s]));

  // Group g of the stream: K tile g and V tile g - LAG, in slots g % RING and (g - LAG) % RING of their rings.  Wave w
  // fetches the pieces IP (w % 2) .. of page w / 2 of either tile; what lies outside the slice re-reads a tile
  // of it (never used).  A V piece (32 dimensions x 16 keys) is fetched so that the 16 lanes which read an operand together
  // find it in 256 consecutive bytes: LDS position u of it holds dimension 16 (u / 32) + u % 16, key half (u / 16) % 2.
  const int nt = (np + WIDE_TILE_PAGES - 1) / WIDE_TILE_PAGES, ng = nt + LAG;
  const int F = ntok / (WIDE_TILE_PAGES * PAGE * HALVES) * HALVES;  // tiles in the pipeline
  const uint32_t vsrc = (2 * (16 * (lane / 32) + lane % 16) + (lane / 16) % 2) * 16;
  const unsigned char *p_k = nullptr, *p_v = nullptr;
  unsigned char *p_kl = nullptr, *p_vl = nullptr;
  auto group_setup = [&](int g) __attribute__((always_inline)) {
    auto page = [&](int tile) __attribute__((always_inline)) {
      const int i = min(WIDE_TILE_PAGES * min(max(tile, 0), nt - 1) + w / 2, np - 1);
      const int id = __builtin_amdgcn_readlane(i < 64 ? pg_a : pg_b, i & 63);
      return ((size_t)id * a.hkv + hk) * (size_t)PB + (w % 2) * IP * 1024;
    };
    const uint32_t at = (w / 2) * PB + (w % 2) * IP * 1024;
    p_k = (const unsigned char*)a.k_pool + page(g);
    p_v = (const unsigned char*)a.v_pool + page(g - LAG);
    p_kl = Kring + (g % WIDE_RING) * TB + at;
    p_vl = Vring + ((g + WIDE_RING - LAG) % WIDE_RING) * TB + at;
  };
  auto group_load = [&](auto xc) __attribute__((always_inline)) {
    constexpr int x = decltype(xc)::value;
    const unsigned char* src = x < IP ? p_k + x * 1024 + lane * 16 : p_v + (x - IP) * 1024 + vsrc;
    __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) const void*)src,
                                     (__attribute__((address_space(3))) void*)(x < IP ? p_kl + x * 1024 : p_vl + (x - IP) * 1024), 16, 0, 0);
  };
  auto issue = [&](int g) __attribute__((always_inline)) {
    if (g >= ng) return;
    group_setup(g);
    static_for<0, LPG>(group_load);
  };
  // Group t is there for everybody, and everybody is past what group t - 1 was needed for: the slots of group t + 3 are free.
  auto arrive = [&](int t) __attribute__((always_inline)) {
    if (t + 3 <= ng) wait_vmcnt<2 * LPG>();
    else if (t + 2 <= ng) wait_vmcnt<LPG>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  for (int g = 0; g < 3; ++g) issue(g);

  if (!active) {  // (no rows for this wave: its share of the loads)
    for (int t = 0; t < ng; ++t) {
      arrive(t);
      issue(t + 3);
    }
    return;
  }
  const int kr = key_of_row(L);
  const uint32_t half0 = HALVES == 2 || parts > 1 ? (sub & 1) * 2 * PB : 0;
  const uint32_t koff = lds_addr(Kring) + half0 + (kr >> 4) * PB + H * 256 + (kr & 15) * 16;
  const uint32_t voff = lds_addr(Vring) + half0 + (L / 16) * 512 + H * 256 + (L % 16) * 16;
  auto Ka = [&](int t) __attribute__((always_inline)) { return koff + (uint32_t)(t % WIDE_RING) * TB; };
  auto Va = [&](int t) __attribute__((always_inline)) { return voff + (uint32_t)(t % WIDE_RING) * TB; };

#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) O[db][r] = 0.f;
  m = -1e30f;
  l = 0.f;
  float msc = m * a.sc, limit = a.settle;
  f32x16 SA, SB;
  bf16x8 P0[2], P1[2];

  // The pieces of a unit by themselves (first and last units, the ragged tile): operand reads, wait, products.
  auto scores = [&](uint32_t ka, auto half_c, f32x16& S) __attribute__((always_inline)) {
    constexpr int HF = decltype(half_c)::value;
    bf16x8 kop[KS];
    const uint32_t ka_ = ka;
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(kop[s]) : "v"(ka_), "n"(HF * 2 * PB + s * 512));
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(kop[s]));
#pragma unroll
    for (int r = 0; r < 16; ++r) S[r] = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) S = mfma32(kop[s], qf[s], S);
  };
  auto values = [&](uint32_t va, auto half_c, const bf16x8* P, int key0) __attribute__((always_inline)) {  // key0 + 32 > ntok: ragged
    constexpr int HF = decltype(half_c)::value;
    bf16x8 v0[DB], v1[DB];
    const uint32_t va_ = va;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v0[db]) : "v"(va_), "n"(HF * 2 * PB + db * 1024));
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v1[db]) : "v"(va_), "n"(HF * 2 * PB + PB + db * 1024));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(v0[db]), "+v"(v1[db]));
    if (key0 + 32 > ntok) clear_unused_values<D>(v0, v1, key0, ntok, H);
    block_pv<D>(v0, v1, P[0], P[1], O);
  };
  auto row_max = [&](const f32x16& S) __attribute__((always_inline)) {
    float bm = S[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) bm = fmaxf(bm, S[r]);
    return fmaxf(bm, __shfl_xor(bm, 32));
  };
  auto raise = [&](float bm) __attribute__((always_inline)) {  // the reference maximum to at least bm
    const float m_new = fmaxf(m, bm), alpha = __builtin_amdgcn_exp2f((m - m_new) * a.sc);
    m = m_new;
    msc = m * a.sc;
    l *= alpha;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) O[db][r] *= alpha;
  };
  auto probs = [&](const f32x16& S, bf16x8* P) __attribute__((always_inline)) {
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
      const float pa = __builtin_amdgcn_exp2f(fmaf(S[e], a.sc, -msc)), pb = __builtin_amdgcn_exp2f(fmaf(S[e + 1], a.sc, -msc));
      sum += pa + pb;
      P[e >> 3][e & 7] = (__bf16)pa;
      P[e >> 3][(e & 7) + 1] = (__bf16)pb;
    }
    return sum;
  };
  // Probabilities of S once more, with the reference raised, where they have left the range (what
  // else is under way are scores, which know no reference): a lane's sum of 16 exceeds the one last looked after by a.settle.
  // Scores that are nearly equal make large sums, 16 at most, without leaving anything: such heads would be here in every
  // unit if the sum itself were the measure (K of zeros, 2 x 32 branches over 16,000 tokens, 16 / 4 heads, dimension 64: 32.0 us, so 25.2).
  auto settle = [&](const f32x16& S, bf16x8* P, float& sum) __attribute__((always_inline)) {
    if (__builtin_amdgcn_ballot_w64(!(sum < limit)) == 0) return;
    raise(row_max(S));
    sum = probs(S, P);
    limit = sum + a.settle;
  };
  auto first_part = [&](int t, auto half_c, int key0, bf16x8* P) __attribute__((always_inline)) {  // scores and probabilities
    f32x16 S;
    scores(Ka(t), half_c, S);
    if (key0 + 32 > ntok) {  // masked at the end of the list
#pragma unroll
      for (int r = 0; r < 16; ++r) S[r] = key0 + 16 * (r >> 3) + 8 * H + (r & 7) < ntok ? S[r] : -INFINITY;
    }
    const float bm = row_max(S);
    if (__builtin_amdgcn_ballot_w64(bm > m + a.th) != 0) raise(bm);
    l += probs(S, P);
  };
  auto general = [&](int t, auto half_c, int half) __attribute__((always_inline)) {  // a unit by itself
    bf16x8 P[2];
    const int key0 = t * WIDE_TILE_PAGES * PAGE + 32 * half;
    first_part(t, half_c, key0, P);
    values(Va(t), half_c, P, key0);
  };
  typedef std::integral_constant<int, 0> h0_t;
  typedef std::integral_constant<int, 1> h1_t;

  if constexpr (HALVES == 1) {
    if (parts > 1) {  // the values of a unit a tile behind its scores: the two waves of a SIMD take turns with the matrix pipe
      bool pending = false;
      int key0 = 0;
#pragma unroll 1
      for (int t = 0; t < ng; ++t) {
        arrive(t);
        issue(t + 3);
        if (pending) values(Va(t + WIDE_RING - 1), h0_t{}, P0, key0);
        pending = t < nt && (parts == 2 || (t & 1) == sub >> 1);
        key0 = t * WIDE_TILE_PAGES * PAGE + 32 * (sub & 1);
        if (pending) first_part(t, h0_t{}, key0, P0);
      }
      return;
    }
  }

  // A tile in the steady state: 2 / HALVES units.  Unit u takes scores into SA (u even) or SB.
  auto steady = [&](int t, auto par_c) __attribute__((always_inline)) {
    constexpr int PAR = decltype(par_c)::value, STEPS = 2 / HALVES, NT = STEPS * NS;
    const uint32_t ka = Ka(t), va = Va(t + WIDE_RING - LAG);
    bf16x8 opr[OPR];
    float sum = 0.f, even = 0.f, last = 0.f;
    auto fetch = [&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value, st = i / NS, j = i % NS;
      bf16x8* const op = opr;
      const uint32_t ka_ = ka, va_ = va;
      if constexpr (i < NT) {
        if constexpr (j % 2 == 0) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(op[i % OPR]) : "v"(ka_), "n"(st * 2 * PB + j / 2 * 512));
        else
          asm volatile("ds_read_b128 %0, %1 offset:%2"
                       : "=v"(op[i % OPR])
                       : "v"(va_), "n"(st * 2 * PB + j / 2 / DB * PB + j / 2 % DB * 1024));
      }
    };
    static_for<0, PF>(fetch);
    if (t + 3 < ng) group_setup(t + 3);  // (none left: the last group once more, the same bytes into the same places)
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, NT>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value, st = i / NS, j = i % NS, x = j / 2;
      fetch(std::integral_constant<int, i + PF>{});
      wait_lgkmcnt<(i + PF < NT ? PF : NT - 1 - i)>();
      __builtin_amdgcn_sched_barrier(0);
      constexpr bool odd = (PAR + st) % 2 != 0;
      f32x16& Sn = odd ? SB : SA;
      const f32x16& Sc = odd ? SA : SB;
      bf16x8* const Pp = odd ? P1 : P0;
      bf16x8* const Pc = odd ? P0 : P1;
      if constexpr (j % 2 == 0) {
        if constexpr (j == 0) Sn = mfma32(opr[i % OPR], qf[0], f32x16{});
        else Sn = mfma32(opr[i % OPR], qf[x], Sn);
      } else {
        O[x % DB] = mfma32(opr[i % OPR], Pp[x / DB], O[x % DB]);
      }
      if constexpr (st == STEPS - 1 && j % (NS / LPG) == 1) {  // a load of the group three tiles ahead
        group_load(std::integral_constant<int, j / (NS / LPG)>{});
      }
#pragma unroll
      for (int e = j * 16 / NS; e < (j + 1) * 16 / NS; ++e) {
        const float p = __builtin_amdgcn_exp2f(fmaf(Sc[e], a.sc, -msc));
        sum += last;  // (the one before: its result is there, this one's is not yet)
        last = p;
        asm volatile("" : "+v"(sum));  // keep the running sum
        if (e & 1) {
          Pc[e >> 3][(e & 7) - 1] = (__bf16)even;
          Pc[e >> 3][e & 7] = (__bf16)p;
        } else {
          even = p;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (j == NS - 1) {
        sum += last;
        settle(Sc, Pc, sum);
        l += sum;
        sum = last = 0.f;
      }
    });
  };

  int t = 0;
  if (F > 0) {
    // units 0 and 1
    arrive(0);
    scores(Ka(0), h0_t{}, SA);
    issue(3);
    if constexpr (HALVES == 1) {
      scores(Ka(0), h1_t{}, SB);
    } else {
      arrive(1);
      scores(Ka(1), h0_t{}, SB);
      issue(4);
    }
    raise(fmaxf(row_max(SA), row_max(SB)));  // (of 64 keys: the closer to the row's maximum, the smaller the rounding of its largest probabilities)
    l += probs(SA, P0);
    limit = l + a.settle;
#pragma unroll 1
    for (t = LAG; t < F; t += HALVES) {
      arrive(t);
      steady(t, h0_t{});
      if constexpr (HALVES == 2) {
        arrive(t + 1);
        steady(t + 1, h1_t{});
      }
    }
    // probabilities of the last unit, products of the last two
    arrive(F);
    issue(F + 3);
    values(Va(F - LAG), h0_t{}, P0, 0);
    float sum = probs(SB, P1);
    settle(SB, P1, sum);
    l += sum;
    if constexpr (HALVES == 2) {
      arrive(F + 1);
      values(Va(F - 1), h0_t{}, P1, 0);
    } else {
      values(Va(F - 1), h1_t{}, P1, 0);
    }
    t = F + LAG;
  }
  // what is left, two tiles at most: one that ends inside, and in front of it the odd one of a wave that takes halves
#pragma unroll 1
  for (int g = t; g < ng; ++g) {
    arrive(g);
    issue(g + 3);
  }
#pragma unroll 1
  for (t = F; t < nt; ++t) {
    general(t, h0_t{}, HALVES == 2 ? sub : 0);
    if constexpr (HALVES == 1) general(t, h1_t{}, 1);
  }
}

template <int D>
__global__ void __launch_bounds__(64 * WIDE_WAVES, 2) k_decode_wide(DecodeArgs a) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int L = lane & 31, H = lane >> 5;
  f32x16 O[D / 32];
  float m, l;
  // Workgroups in launch order: a.wide_first with own items, the shared items, the other own items.
  const int first = (int)blockIdx.x - a.wide_first;
  if (first >= 0 && first < a.wide_shared) {
    const bool halves = a.rb_max <= WIDE_WAVES / 2;
    int rb = w % a.rb_max, sub = w / a.rb_max, parts = halves ? 2 : 1;
    if (a.rb_max == 5 || a.rb_max == 6) {
      const int left = a.rb_max - 4;
      rb = w < 4 ? w : 4 + (w - 4) % left;
      sub = w < 4 ? 0 : (w - 4) / left;
      parts = w < 4 ? 1 : 4 / left;
    }
    int x = first;
    const int split = x % a.splits_a; x /= a.splits_a;
    const int hk = x % a.hkv, g = x / a.hkv;
    const int branch0 = a.group_branch_off[g], nrows = (a.group_branch_off[g + 1] - branch0) * a.G;
    const int len = a.shared_len[g], npages = (len + PAGE - 1) / PAGE;
    const int p0 = split * a.chunk_a, p1 = min(p0 + a.chunk_a, npages);
    const int row = 32 * rb + L;
    const bool row_ok = row < nrows, active = sub < parts && 32 * rb < nrows;
    const size_t item = (((size_t)g * a.hkv + hk) * a.rb_max + rb) * a.splits_a + split;
    float* const pml = a.part_ml_a + (item * 32 + L) * 2;
    if (p0 >= p1) {  // empty slice (the same for every wave of the workgroup): neutral partials
      if (row_ok && H == 0 && sub == 0) {
        pml[0] = -1e30f;
        pml[1] = 0.f;
      }
      return;
    }
    const int rr = row_ok ? row : 0;
    const uint16_t* qrow = a.q + (active ? ((size_t)(branch0 + rr / a.G) * a.hq + hk * a.G + rr % a.G) * D : 0);
    const int32_t* pages = a.shared_pages + a.shared_page_off[g] + p0;
    const int np = p1 - p0, ntok = min(len - p0 * PAGE, np * PAGE);
    if (halves) wide_item<D, 2>(a, smem, pages, np, ntok, hk, qrow, w, lane, sub, parts, active, O, m, l);
    else wide_item<D, 1>(a, smem, pages, np, ntok, hk, qrow, w, lane, sub, parts, active, O, m, l);
    int db0 = 0, db1 = D / 32;
    if (halves) {
      // The two waves of a row block exchange halves of their accumulators through the rings (every load has landed, and
      // every wave is past its last operand) and each puts one half of the output dimensions together.
      constexpr int HD = D / 64;  // accumulator blocks of a half
      float* const slots = (float*)smem;
      auto slot = [&](int s2) { return slots + ((size_t)(rb * 2 + s2) * 64 + lane) * (16 * HD + 4); };
      __syncthreads();
      if (active) {
        float* const mine = slot(sub);
#pragma unroll
        for (int db = 0; db < HD; ++db)
#pragma unroll
          for (int r = 0; r < 16; r += 4) {
            const f32x16& give = sub ? O[db] : O[HD + db];
            *(f32x4*)(mine + 16 * db + r) = f32x4{give[r], give[r + 1], give[r + 2], give[r + 3]};
          }
        mine[16 * HD] = m;
        mine[16 * HD + 1] = l;
      }
      __syncthreads();
      if (!active) return;
      const float* const other = slot(1 - sub);
      const float m2 = other[16 * HD], l2 = other[16 * HD + 1], m_new = fmaxf(m, m2);
      const float a1 = __builtin_amdgcn_exp2f((m - m_new) * a.sc), a2 = __builtin_amdgcn_exp2f((m2 - m_new) * a.sc);
      m = m_new;
      l = l * a1 + l2 * a2;
#pragma unroll
      for (int db = 0; db < HD; ++db)
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
          const f32x4 o2 = *(const f32x4*)(other + 16 * db + r);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float own = sub ? O[HD + db][r + e] : O[db][r + e];
            O[db][r + e] = own * a1 + o2[e] * a2;
          }
        }
      db0 = sub ? HD : 0;
      db1 = HD;  // (O[0 ..] hold the wave's half now)
    }
    if (a.rb_max == 5 || a.rb_max == 6) {
      // The waves that share a row block leave their accumulators in the rings and each puts some output dimensions together.
      constexpr int DB = D / 32;
      float* const slots = (float*)smem;
      auto slot = [&](int wave) { return slots + ((size_t)(wave - 4) * 64 + lane) * (16 * DB + 4); };
      __syncthreads();
      if (active && parts > 1) {
        float* const mine = slot(w);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int r = 0; r < 16; r += 4) *(f32x4*)(mine + 16 * db + r) = f32x4{O[db][r], O[db][r + 1], O[db][r + 2], O[db][r + 3]};
        mine[16 * DB] = m;
        mine[16 * DB + 1] = l;
      }
      __syncthreads();
      if (!active) return;
      if (parts > 1) {
        const int left = a.rb_max - 4, first_wave = rb;  // the waves rb, rb + left, ..
        db0 = sub * DB / parts;
        const int n = max((sub + 1) * DB / parts - db0, 0);
        float mx = -1e30f, ls = 0.f;
        for (int p = 0; p < parts; ++p) mx = fmaxf(mx, slot(first_wave + p * left)[16 * DB]);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) O[db][r] = 0.f;
        for (int p = 0; p < parts; ++p) {
          const float* const theirs = slot(first_wave + p * left);
          const float wgt = __builtin_amdgcn_exp2f((theirs[16 * DB] - mx) * a.sc);
          ls += theirs[16 * DB + 1] * wgt;
#pragma unroll
          for (int db = 0; db < DB; ++db)
            if (db < n)
#pragma unroll
              for (int r = 0; r < 16; r += 4) {
                const f32x4 o = *(const f32x4*)(theirs + 16 * (db0 + db) + r);
#pragma unroll
                for (int e = 0; e < 4; ++e) O[db][r + e] += o[e] * wgt;
              }
        }
        m = mx;
        l = ls;
        db1 = n;
      }
    }
    if (!active) return;
    const float l_tot = l + __shfl_xor(l, 32);
    if (!row_ok) return;
    float* const po = a.part_o_a + (item * 32 + L) * D + 32 * db0 + 4 * H;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
      if (db < db1)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *(f32x4*)(po + 32 * db + 8 * r4) = f32x4{O[db][4 * r4], O[db][4 * r4 + 1], O[db][4 * r4 + 2], O[db][4 * r4 + 3]};
    if (H == 0 && sub == 0) {
      pml[0] = m;
      pml[1] = l_tot;
    }
    return;
  }

  // Own pages of a (branch, kv head, slice) for every wide_own waves, in the order of k_decode's own items.
  const int ow = a.wide_own, G = a.G, slot = w / ow, sub = w % ow;
  const int item0 = (first < 0 ? (int)blockIdx.x : (int)blockIdx.x - a.wide_shared) * (WIDE_WAVES / ow), item = min(item0 + slot, a.items_b - 1);
  int x = item;
  const int split = x % a.splits_b; x /= a.splits_b;
  const int hk = x % a.hkv, branch = x / a.hkv;
  const int len = a.branch_len[branch], npages = (len + PAGE - 1) / PAGE;
  const int p0 = split * a.chunk_b, p1 = min(p0 + a.chunk_b, npages);
  const int per = ((max(p1 - p0, 0) + ow - 1) / ow + 1) & ~1;  // pages of a wave (a 32-key block never straddles two)
  const int w0 = p0 + sub * per, w1 = min(w0 + per, p1);
  bf16x8* const qs = (bf16x8*)smem;                                                   // [slot][operand][lane]
  float* const po_lds = (float*)(smem + WIDE_WAVES / ow * (D / 16) * 1024);           // [wave][row][D + 4]
  float* const ml_lds = po_lds + WIDE_WAVES * G * (D + 4);                            // [wave][row][2]
  const bf16x8* const qf = qs + slot * (D / 16) * 64 + lane;
  for (int s = sub; s < D / 16; s += ow)
    qs[(slot * (D / 16) + s) * 64 + lane] = *(const bf16x8*)(a.q + ((size_t)branch * a.hq + hk * G + min(L, G - 1)) * D + 8 * H + 16 * s);
  __syncthreads();
  m = -1e30f;
  float l_tot = 0.f;
  if (w0 < w1) {
    auto qop = [&](int s) { return qf[s * 64]; };
    a.th *= 0.125f;  // (raised by a factor of two: a wave may have a whole slice under the one reference)
    stream_slice<D>(a, a.branch_pages + a.branch_page_off[branch], w0, w1, len, len, len, hk, lane, qop, O, m, l);
    l_tot = l + __shfl_xor(l, 32);
    if (L < G) {
      float* const po = po_lds + (w * G + L) * (D + 4) + 4 * H;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *(f32x4*)(po + 32 * db + 8 * r4) = f32x4{O[db][4 * r4], O[db][4 * r4 + 1], O[db][4 * r4 + 2], O[db][4 * r4 + 3]};
    }
  }
  if (L < G && H == 0) {
    ml_lds[(w * G + L) * 2] = m;
    ml_lds[(w * G + L) * 2 + 1] = l_tot;
  }
  __syncthreads();
  if (item0 + slot >= a.items_b) return;
  const int used = p1 > p0 ? (p1 - p0 + per - 1) / per : 0;
  for (int i = sub * 64 + lane; i < G * D / 4; i += 64 * ow) {
    const int r = i / (D / 4), c = i % (D / 4) * 4;
    float mx = -1e30f, ls = 0.f;
    for (int p = 0; p < used; ++p) mx = fmaxf(mx, ml_lds[((slot * ow + p) * G + r) * 2]);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int p = 0; p < used; ++p) {
      const int at = (slot * ow + p) * G + r;
      const float wgt = __builtin_amdgcn_exp2f((ml_lds[at * 2] - mx) * a.sc);
      const f32x4 o = *(const f32x4*)(po_lds + at * (D + 4) + c);
      ls += ml_lds[at * 2 + 1] * wgt;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += o[e] * wgt;
    }
    *(f32x4*)(a.part_o_b + ((size_t)item * G + r) * D + c) = acc;
    if (c == 0) {
      a.part_ml_b[((size_t)item * G + r) * 2] = mx;
      a.part_ml_b[((size_t)item * G + r) * 2 + 1] = ls;
    }
  }
}

// One wave per (branch, query head): log-sum-exp combination of its partials.  What it costs is the chain
// of dependent loads, so the group is found with one load per lane for every factor of 64 in their number, and the
// outputs of the first partials are on their way together with the maxima and sums.  Up to MERGE_FEW_ROWS rows a lane has four
// output dimensions (PER) of every second partial (every fourth at head dimension 64) and a workgroup four rows: fewer loads in
// the chain.  More rows are more waves than the device holds at once, and what counts is their number of instructions: a lane
// then has the same D / 64 dimensions of every partial, at addresses that the wave computes once, and the partials need no sum over
// lanes.  Few partials, first and second form: dimension 64, 4096 rows 4.2 and 5.1 us, 8192 rows 7.1 and 5.9, 16384 rows 12.6 and 9.1,
// 65536 rows 46 and 33; dimension 128 4.2 and 4.5, 8.0 and 6.8, 12.0 and 10.2, 46 and 38.
constexpr int merge_per(int D, bool few) { return few ? 4 : D / 64; }
constexpr int merge_threads(bool few) { return few ? 256 : 64; }
__device__ __forceinline__ int group_of_branch(const DecodeArgs& a, int r, int lane) {
  int g = 0;  // the last group that starts at or before r, one of the n from g on
  for (int n = a.n_groups; n > 1;) {
    const int step = (n + 63) / 64, at = min(lane * step, n - 1);
    const int before = __popcll(__ballot(lane * step < n && a.group_branch_off[g + at] <= r)) - 1;
    g += max(before, 0) * step;
    n = min(step, n - max(before, 0) * step);
  }
  return g;
}
template <int D, bool FEW>
__global__ void __launch_bounds__(merge_threads(FEW)) k_decode_merge(DecodeArgs a) {
  const int wid = __builtin_amdgcn_readfirstlane(blockIdx.x * (merge_threads(FEW) / 64) + (threadIdx.x >> 6));
  const int r = wid / a.hq, head = wid % a.hq;
  if (r >= a.n_live) return;
  const int hk = head / a.G, j = head % a.G;
  const int lane = threadIdx.x & 63;
  const int g = group_of_branch(a, r, lane);
  const int row = (r - a.group_branch_off[g]) * a.G + j;
  const int rb = row >> 5, rr = row & 31;
  const size_t ia0 = (((size_t)g * a.hkv + hk) * a.rb_max + rb) * a.splits_a;
  const size_t ib0 = ((size_t)r * a.hkv + hk) * a.splits_b;
  constexpr int PER = merge_per(D, FEW), ROW = D / PER, SETS = 64 / ROW;  // lanes to a partial, partials to a load
  typedef __attribute__((ext_vector_type(PER))) float part_t;
  const int set = SETS > 1 ? lane / ROW : 0, c = lane % ROW * PER;
  const int np = a.splits_a + a.splits_b;
  // partial p of this (branch, head): shared split p, then own split p - splits_a
  auto ml_of = [&](int p) {
    return p < a.splits_a ? a.part_ml_a + ((ia0 + p) * 32 + rr) * 2 : a.part_ml_b + ((ib0 + (p - a.splits_a)) * a.G + j) * 2;
  };
  auto o_of = [&](int p) {
    return p < a.splits_a ? a.part_o_a + ((ia0 + p) * 32 + rr) * D : a.part_o_b + ((ib0 + (p - a.splits_a)) * a.G + j) * D;
  };
  part_t acc;
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] = 0.f;
  float lsum = 0.f;
  auto merge = [&](auto batch_c) __attribute__((always_inline)) {  // BATCH loads of SETS partial outputs in flight
    constexpr int BATCH = decltype(batch_c)::value;
    part_t x[BATCH];
    auto fetch = [&](int p0) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < BATCH; ++i) x[i] = *(const part_t*)(o_of(min(p0 + i * SETS + set, np - 1)) + c);
    };
    fetch(0);
    // The reference maximum first (64 partials at a time, one per lane, so that their loads are in
    // flight together), then the weighted sums in the fixed order of the partials: the weights of
    // a group of 64 come from the lanes, and the loads of the partial outputs do not depend on
    // each other (a partial without a visible key has l = 0 and weight 0; what it holds is read
    // and dropped).
    float mx = -1e30f;
    for (int p0 = 0; p0 < np; p0 += 64) {
      const float mv = p0 + lane < np ? ml_of(p0 + lane)[0] : -1e30f;
      mx = fmaxf(mx, mv);
    }
    mx = dag_wave_max(mx);
    for (int p0 = 0; p0 < np; p0 += 64) {
      float wl = 0.f, wgt = 0.f;
      if (p0 + lane < np) {
        const float* ml = ml_of(p0 + lane);
        const float ls = ml[1];
        if (ls > 0.f) {
          wgt = __builtin_amdgcn_exp2f((ml[0] - mx) * a.sc);
          wl = ls * wgt;
        }
      }
      for (int b0 = p0; b0 < min(p0 + 64, np); b0 += BATCH * SETS) {
        if (b0 > 0) fetch(b0);
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {  // (the weight of a partial past the last one is zero)
          const float wi = __shfl(wgt, b0 - p0 + i * SETS + set);
          lsum += __shfl(wl, b0 - p0 + i * SETS + set);
#pragma unroll
          for (int e = 0; e < PER; ++e) acc[e] += wi != 0.f ? wi * x[i][e] : 0.f;
        }
      }
    }
  };
  // (what is read beyond the last partial is that one again)
  if constexpr (FEW) {
    if (np <= SETS) merge(std::integral_constant<int, 1>{});
    else if (np <= 3 * SETS) merge(std::integral_constant<int, 3>{});
    else if (np <= 9 * SETS) merge(std::integral_constant<int, 9>{});
    else merge(std::integral_constant<int, 16>{});
  } else {
    if (np <= 2) merge(std::integral_constant<int, 2>{});
    else if (np <= 4) merge(std::integral_constant<int, 4>{});
    else if (np <= 8) merge(std::integral_constant<int, 8>{});
    else merge(std::integral_constant<int, 16>{});
  }
#pragma unroll
  for (int off = ROW; off < 64; off <<= 1) {
    lsum += __shfl_xor(lsum, off);
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] += __shfl_xor(acc[e], off);
  }
  if (set != 0) return;
  const float inv = 1.f / lsum;
  uint16_t* o = a.out + ((size_t)r * a.hq + head) * D + c;
  if constexpr (PER == 4) *(u32x2*)o = u32x2{dag_pack_bf2(acc[0] * inv, acc[1] * inv), dag_pack_bf2(acc[2] * inv, acc[3] * inv)};
  else if constexpr (PER == 2) *(uint32_t*)o = dag_pack_bf2(acc[0] * inv, acc[1] * inv);
  else *o = (uint16_t)dag_f2bf(acc[0] * inv);
}

// Short contexts: a workgroup takes a (branch, KV head) whole, a wave a slice of the shared or of the own pages, and puts the
// partials together in LDS: no partials in memory and no launch for the merge, which is what these steps consist of (13.0 -> 10.6 us).
// Every branch reads the shared pages for itself.  Eight waves, two a SIMD, because a slice's two blocks take the registers of that.
constexpr int WHOLE_WAVES = 8;
template <int D>
__global__ void __launch_bounds__(64 * WHOLE_WAVES, 2) k_whole_branch(DecodeArgs a) {
  __shared__ bf16x8 qs_all[(D / 16) * 64];
  __shared__ __align__(16) float part[WHOLE_WAVES][WHOLE_ROWS][D + 4];
  __shared__ float part_ml[WHOLE_WAVES][WHOLE_ROWS][2];
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, L = lane & 31, H = lane >> 5;
  const int r = blockIdx.x / a.hkv, hk = blockIdx.x % a.hkv;
  if (w < D / 16) qs_all[w * 64 + lane] = *(const bf16x8*)(a.q + ((size_t)r * a.hq + hk * a.G + min(L, a.G - 1)) * D + 8 * H + 16 * w);
  const int g = group_of_branch(a, r, lane);
  const int len_a = a.splits_a > 0 ? a.shared_len[g] : 0, len_b = a.splits_b > 0 ? a.branch_len[r] : 0;
  const int n_a = min((len_a + PAGE - 1) / PAGE, a.splits_a * a.chunk_a), n_b = min((len_b + PAGE - 1) / PAGE, a.splits_b * a.chunk_b);
  const int blocks_a = (n_a + 1) / 2, blocks_b = (n_b + 1) / 2, blocks = blocks_a + blocks_b;
  const int waves_a = blocks_b <= 0 ? WHOLE_WAVES : blocks_a <= 0 ? 0 : min(max((blocks_a * WHOLE_WAVES + blocks / 2) / blocks, 1), WHOLE_WAVES - 1);
  const bool is_a = w < waves_a;
  const int n = is_a ? n_a : n_b, ways = is_a ? waves_a : WHOLE_WAVES - waves_a, len = is_a ? len_a : len_b;
  const int per = 2 * (((n + 1) / 2 + ways - 1) / ways), p0 = (is_a ? w : w - waves_a) * per, p1 = min(p0 + per, n);
  __syncthreads();
  if (p0 < p1) {
    const int32_t* pages = is_a ? a.shared_pages + a.shared_page_off[g] : a.branch_pages + a.branch_page_off[r];
    const bf16x8* qf = qs_all + lane;
    auto qop = [&](int s) { return qf[s * 64]; };
    f32x16 O[D / 32];
    float m, l;
    stream_slice<D>(a, pages, p0, p1, len, len, len, hk, lane, qop, O, m, l);
    const float l_tot = l + __shfl_xor(l, 32);
    if (L < a.G) {
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4)
          *(f32x4*)&part[w][L][32 * db + 8 * r4 + 4 * H] = f32x4{O[db][4 * r4], O[db][4 * r4 + 1], O[db][4 * r4 + 2], O[db][4 * r4 + 3]};
      if (H == 0) {
        part_ml[w][L][0] = m;
        part_ml[w][L][1] = l_tot;
      }
    }
  } else if (lane < a.G) {
    part_ml[w][lane][0] = -1e30f;
    part_ml[w][lane][1] = 0.f;
  }
  __syncthreads();
  const int j = tid / (D / 4), c = tid % (D / 4) * 4;
  if (j >= a.G) return;
  float mx = -1e30f, lsum = 0.f;
#pragma unroll
  for (int p = 0; p < WHOLE_WAVES; ++p) mx = fmaxf(mx, part_ml[p][j][0]);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < WHOLE_WAVES; ++p) {
    const float lp = part_ml[p][j][1], wgt = lp > 0.f ? __builtin_amdgcn_exp2f((part_ml[p][j][0] - mx) * a.sc) : 0.f;
    const f32x4 o = *(const f32x4*)&part[p][j][c];
    lsum += lp > 0.f ? lp * wgt : 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += wgt != 0.f ? wgt * o[e] : 0.f;
  }
  const float inv = 1.f / lsum;
  *(u32x2*)(a.out + ((size_t)r * a.hq + hk * a.G + j) * D + c) = u32x2{dag_pack_bf2(acc[0] * inv, acc[1] * inv), dag_pack_bf2(acc[2] * inv, acc[3] * inv)};
}

// One block per live branch: rotate the new key at the branch's adaptive position and scatter
// key and value into the pool formats.  The angles depend on the position and the frequency index
// only, so D / 2 threads compute them once (fp64) and the block shares them through LDS.
__global__ void __launch_bounds__(256) k_kv_append(const int32_t* branch_page_off, const int32_t* branch_pages,
                                                   const int32_t* branch_len, const int32_t* branch_pos,
                                                   const uint16_t* k_new, const uint16_t* v_new, uint16_t* k_pool,
                                                   uint16_t* v_pool, int hkv, int D, RopeTheta theta) {
  __shared__ float s_cos[64], s_sin[64];  // D / 2 <= 64 (the entry point admits head_dim 64 and 128 only)
  constexpr int KEEP = 2;                 // a thread's first pairs are on their way while the angles are computed
  const int r = blockIdx.x, half = D / 2, n = hkv * half;
  struct Pair {
    uint16_t k0, k1, v0, v1;
  };
  auto load = [&](int x) __attribute__((always_inline)) {
    const size_t src = ((size_t)r * hkv + x / half) * D + x % half;
    return Pair{k_new[src], k_new[src + half], v_new[src], v_new[src + half]};
  };
  Pair keep[KEEP];
#pragma unroll
  for (int i = 0; i < KEEP; ++i) keep[i] = load(min((int)threadIdx.x + 256 * i, n - 1));
  const int idx = branch_len[r] - 1;
  if (idx < 0) return;
  const int page = branch_pages[branch_page_off[r] + idx / PAGE];
  const int slot = idx % PAGE;
  if ((int)threadIdx.x < half) {
    double sn, cs;
    sincos((double)branch_pos[r] * dag_rope_freq(theta, threadIdx.x, D), &sn, &cs);
    s_cos[threadIdx.x] = (float)cs;
    s_sin[threadIdx.x] = (float)sn;
  }
  __syncthreads();
  auto store = [&](int x, const Pair& p) __attribute__((always_inline)) {
    const int h = x / half, d0 = x % half, d1 = d0 + half;
    const float lo = __uint_as_float((uint32_t)p.k0 << 16), hi = __uint_as_float((uint32_t)p.k1 << 16);
    const float c = s_cos[d0], s = s_sin[d0];  // (the products are rounded alike in k_kv_append_run)
    const size_t pb = ((size_t)page * hkv + h) * (size_t)(D * PAGE);
    k_pool[pb + (size_t)(d0 >> 3) * (PAGE * 8) + slot * 8 + (d0 & 7)] = (uint16_t)dag_f2bf(fmaf(lo, c, -(hi * s)));
    k_pool[pb + (size_t)(d1 >> 3) * (PAGE * 8) + slot * 8 + (d1 & 7)] = (uint16_t)dag_f2bf(fmaf(lo, s, hi * c));
    v_pool[pb + (size_t)d0 * PAGE + slot] = p.v0;
    v_pool[pb + (size_t)d1 * PAGE + slot] = p.v1;
  };
#pragma unroll
  for (int i = 0; i < KEEP; ++i)
    if ((int)threadIdx.x + 256 * i < n) store(threadIdx.x + 256 * i, keep[i]);
  for (int x = threadIdx.x + 256 * KEEP; x < n; x += 256) store(x, load(x));
}

// The same for many entries (the new tokens of prefilled nodes), kRunRows at a time.  Consecutive entries mostly are
// consecutive slots of a page: the angles of an entry serve all heads, keys are rotated and stored in
// 16-byte pieces, and the values of eight entries that fill half a page go out as one 16-byte piece per
// dimension, the others element by element.  32768 entries of 8 heads x 128: 200 -> 58 us aligned, 82 us
// from slot 5 on (the traffic takes 45 us at the rate of a large copy).  Few runs are divided over the
// heads too, to about two workgroups a compute unit.
// Entries from which on: with 8 heads runs of 512 take the same either way, 1024 take 10.3 -> 8.5 us, 4096 26 ->
// 13 to 16.  Entries on pages of their own lose 3 to 7 us up to 4096 (1024: 11.6 -> 15.6 us, 2048: 20.5 -> 23.4,
// 4096: 36.6 -> 42.8) and gain beyond (8192: 189 -> 169).  A descriptor with sibling groups is a decode step, every
// entry the newest token of a branch with pages of its own, and takes this kernel where those gain;
// one without groups lists the tokens of prefilled nodes.
constexpr int kRunRows = 16, kRunThreads = 256;
constexpr int kAppendRunRows = 1024, kAppendRunBranches = 8192;
__global__ void __launch_bounds__(kRunThreads) k_kv_append_run(int n_live, const int32_t* branch_page_off, const int32_t* branch_pages,
                                                       const int32_t* branch_len, const int32_t* branch_pos,
                                                       const uint16_t* k_new, const uint16_t* v_new, uint16_t* k_pool,
                                                       uint16_t* v_pool, int hkv, int D, RopeTheta theta) {
  __shared__ __attribute__((aligned(16))) float s_cos[kRunRows][64], s_sin[kRunRows][64];
  __shared__ int s_page[kRunRows], s_slot[kRunRows], s_whole[kRunRows], s_one[kRunRows], s_wholes, s_ones;  // slot -1: nothing to store
  const int r0 = blockIdx.x * kRunRows, tid = threadIdx.x, half = D / 2;
  const int h0 = (int)blockIdx.y * hkv / (int)gridDim.y, heads = ((int)blockIdx.y + 1) * hkv / (int)gridDim.y - h0;
  if (tid < 64) {  // lane: entry r0 - 7 + lane, so that every unit of eight that reaches into the block is seen
    const int r = r0 - 7 + tid;
    int page = 0, slot = -1;
    if (tid < kRunRows + 14 && r >= 0 && r < n_live) {
      const int idx = branch_len[r] - 1;
      if (idx >= 0) {
        page = branch_pages[branch_page_off[r] + idx / PAGE];
        slot = idx % PAGE;
      }
    }
    // Units of the value stores: eight entries on consecutive slots from a multiple of eight on (the block
    // of the first one stores them), or one entry.
    bool whole = slot >= 0 && slot % 8 == 0;
    for (int e = 1; e < 8; ++e) {
      const int p = __shfl_down(page, e), t = __shfl_down(slot, e);
      whole = whole && p == page && t == slot + e;
    }
    const uint64_t mine = ((1ull << kRunRows) - 1) << 7, below = (1ull << tid) - 1, lead = __ballot(whole);
    const bool covered = (lead & (0x7full << tid >> 7)) != 0;  // by one of the seven entries in front
    const uint64_t wholes = lead & mine, ones = __ballot(slot >= 0 && !whole && !covered) & mine;
    if (wholes >> tid & 1) s_whole[__popcll(wholes & below)] = tid - 7;
    if (ones >> tid & 1) s_one[__popcll(ones & below)] = tid - 7;
    if (mine >> tid & 1) {
      s_page[tid - 7] = page;
      s_slot[tid - 7] = slot;
    }
    if (tid == 0) {
      s_wholes = __popcll(wholes);
      s_ones = __popcll(ones);
    }
  }
  {
    const double freq = dag_rope_freq(theta, tid % half, D);  // (half divides the block)
    for (int i = tid / half; i < kRunRows; i += kRunThreads / half) {
      double sn = 0., cs = 1.;
      if (r0 + i < n_live) sincos((double)branch_pos[r0 + i] * freq, &sn, &cs);
      s_cos[i][tid % half] = (float)cs;
      s_sin[i][tid % half] = (float)sn;
    }
  }
  __syncthreads();
  const int pairs = half / 8;  // 16-byte pieces of half a row
  const bool by_entry = s_wholes > 0;
  for (int x = tid; x < kRunRows * heads * pairs; x += kRunThreads) {
    // entries fastest where they lie on consecutive slots, else pieces of a row
    const int i = by_entry ? x % kRunRows : x / pairs % kRunRows, c = by_entry ? x / kRunRows % pairs : x % pairs;
    const int h = h0 + x / (kRunRows * pairs);
    const int slot = s_slot[i];
    if (slot < 0) continue;
    const uint16_t* src = k_new + ((size_t)(r0 + i) * hkv + h) * D + 8 * c;
    const u32x4 lo = *(const u32x4*)src, hi = *(const u32x4*)(src + half);
    const float *cs = &s_cos[i][8 * c], *sn = &s_sin[i][8 * c];
    u32x4 olo, ohi;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float l0 = dag_bf_lo(lo[w]), l1 = dag_bf_hi(lo[w]), h0 = dag_bf_lo(hi[w]), h1 = dag_bf_hi(hi[w]);
      const float c0 = cs[2 * w], c1 = cs[2 * w + 1], s0 = sn[2 * w], s1 = sn[2 * w + 1];
      olo[w] = dag_f2bf(fmaf(l0, c0, -(h0 * s0))) | dag_f2bf(fmaf(l1, c1, -(h1 * s1))) << 16;
      ohi[w] = dag_f2bf(fmaf(l0, s0, h0 * c0)) | dag_f2bf(fmaf(l1, s1, h1 * c1)) << 16;
    }
    uint16_t* dst = k_pool + ((size_t)s_page[i] * hkv + h) * (size_t)(D * PAGE) + c * (PAGE * 8) + slot * 8;
    *(u32x4*)dst = olo;
    *(u32x4*)(dst + half * PAGE) = ohi;
  }
  // Two dimensions of the values of a head; a thread takes a unit of eight, or up to four single entries.
  const int ny = heads * half, n_wholes = s_wholes, n_ones = s_ones;
  const size_t step = (size_t)hkv * D;
  for (int x = tid; x < (n_wholes + (n_ones + 3) / 4) * ny; x += kRunThreads) {
    const int y = x % ny, g = x / ny, d = 2 * (y % half), h = h0 + y / half;
    const uint16_t* const src = v_new + ((size_t)r0 * hkv + h) * D + d;
    uint16_t* const dst = v_pool + (size_t)h * (D * PAGE) + (size_t)d * PAGE;
    if (g < n_wholes) {
      const int i = s_whole[g];
      uint32_t in[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) in[e] = *(const uint32_t*)(src + (i + e) * step);
      u32x4 even, odd;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        even[w] = (in[2 * w] & 0xffffu) | in[2 * w + 1] << 16;
        odd[w] = in[2 * w] >> 16 | (in[2 * w + 1] & 0xffff0000u);
      }
      uint16_t* const to = dst + (size_t)s_page[i] * step * PAGE + s_slot[i];
      *(u32x4*)to = even;
      *(u32x4*)(to + PAGE) = odd;
    } else {
      uint32_t in[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) in[e] = *(const uint32_t*)(src + s_one[min(4 * (g - n_wholes) + e, n_ones - 1)] * step);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = s_one[min(4 * (g - n_wholes) + e, n_ones - 1)];  // (the last one may be stored again)
        uint16_t* const to = dst + (size_t)s_page[i] * step * PAGE + s_slot[i];
        to[0] = (uint16_t)in[e];
        to[PAGE] = (uint16_t)(in[e] >> 16);
      }
    }
  }
}

// Read from the environment once per process.
int env_int(const char* name) {
  const char* s = getenv(name);
  if (!s || !*s) return 0;
  const int v = atoi(s);
  return v > 0 ? v : 0;
}
const DecodeKnobs& decode_knobs() {
  static const DecodeKnobs k = {env_int("DAGATTN_DECODE_CHUNK_A"), env_int("DAGATTN_DECODE_CHUNK_B"),
                                env_int("DAGATTN_DECODE_CHUNK_SEG")};
  return k;
}

}  // namespace

extern "C" size_t dag_decode_workspace_bytes(const dag_decode_desc_t* desc, int32_t hq, int32_t hkv,
                                             int32_t head_dim) {
  DecodePlan p;
  if (make_plan(desc, hq, hkv, head_dim, decode_knobs(), &p) != DAG_OK) return 0;
  return p.bytes;
}

extern "C" int dag_kv_append_rope(const dag_decode_desc_t* d, const void* k_new, const void* v_new, void* k_pool,
                                  void* v_pool, int32_t hkv, int32_t head_dim, float theta, void* stream_) {
  if (!d) return DAG_ERR_NULL;
  if (d->n_live < 0) return DAG_ERR_BAD_LEN;
  if (d->page_size != PAGE) return DAG_ERR_UNSUPPORTED;
  if (hkv < 1 || (head_dim != 64 && head_dim != 128) || !(theta > 0.f)) return DAG_ERR_UNSUPPORTED;
  if (d->n_live == 0) return DAG_OK;
  if (!k_new || !v_new || !k_pool || !v_pool || !d->branch_page_off || !d->branch_pages || !d->branch_len ||
      !d->branch_pos)
    return DAG_ERR_NULL;
  const int64_t runs = dag_ceil_div(d->n_live, kRunRows), split = dag_ceil_div(512, runs);
  if (d->n_live >= (d->n_groups > 0 ? kAppendRunBranches : kAppendRunRows) && dag_aligned16(k_new) && dag_aligned16(v_new) && dag_aligned16(k_pool) && dag_aligned16(v_pool))
    hipLaunchKernelGGL(k_kv_append_run, dim3((unsigned)runs, (unsigned)(split < hkv ? split : hkv)), dim3(kRunThreads), 0, (hipStream_t)stream_,
                       d->n_live, d->branch_page_off, d->branch_pages, d->branch_len, d->branch_pos,
                       (const uint16_t*)k_new, (const uint16_t*)v_new, (uint16_t*)k_pool, (uint16_t*)v_pool, hkv,
                       head_dim, dag_rope_theta(theta));
  else
    hipLaunchKernelGGL(k_kv_append, dim3(d->n_live), dim3(256), 0, (hipStream_t)stream_, d->branch_page_off,
                     d->branch_pages, d->branch_len, d->branch_pos, (const uint16_t*)k_new, (const uint16_t*)v_new,
                     (uint16_t*)k_pool, (uint16_t*)v_pool, hkv, head_dim, dag_rope_theta(theta));
  DAG_LAUNCH_CHECK();
  return DAG_OK;
}

namespace {

// Scratch of dag_attn_decode_static: the partial results live in this array instead of a caller
// workspace.  Every GPU the library runs on holds its own copy at its own address until the
// process ends; host code never uses the array's name as an address, only what
// hipGetSymbolAddress returned for the current device.
static __device__ __align__(256) unsigned char scratch[DAG_DECODE_STATIC_SCRATCH_BYTES];

int static_scratch(void** out) {
  constexpr int MAX_DEV = 64;
  static void* ptr[MAX_DEV];
  static bool ready[MAX_DEV];
  static std::mutex mu;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEV) return DAG_ERR_HIP;
  std::lock_guard<std::mutex> lock(mu);
  if (!ready[dev]) {  // once per device, with that device current
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DAG_ERR_HIP;
    ptr[dev] = p;
    ready[dev] = true;
  }
  *out = ptr[dev];
  return DAG_OK;
}

// static_ws: the partials go to the library's own scratch array (ws / ws_bytes ignored).
int decode_impl(const dag_decode_desc_t* d, const void* q, const void* k_pool, const void* v_pool, void* out,
                int32_t hq, int32_t hkv, int32_t head_dim, float softmax_scale, void* ws, size_t ws_bytes,
                void* stream_, bool static_ws) {
  DecodePlan p;
  const int rc = make_plan(d, hq, hkv, head_dim, decode_knobs(), &p);
  if (rc != DAG_OK) return rc;
  if (d->n_live == 0) return DAG_OK;
  if (!q || !k_pool || !v_pool || !out || !d->group_branch_off || !d->branch_page_off || !d->branch_pages ||
      !d->branch_len)
    return DAG_ERR_NULL;
  if (d->n_groups < 1) return DAG_ERR_BAD_LEN;
  if (p.items_a > 0 && (!d->shared_page_off || !d->shared_pages || !d->shared_len)) return DAG_ERR_NULL;
  if (p.items_a + p.items_b == 0) return DAG_ERR_BAD_LEN;  // a query needs at least its own token
  if (!dag_aligned16(q) || !dag_aligned16(k_pool) || !dag_aligned16(v_pool) || !dag_aligned16(out))
    return DAG_ERR_ALIGN;
  if (static_ws) {
    if (p.bytes > (size_t)DAG_DECODE_STATIC_SCRATCH_BYTES) return DAG_ERR_WORKSPACE;
    const int rs = static_scratch(&ws);
    if (rs != DAG_OK) return rs;
  } else if (!ws || ws_bytes < p.bytes) {
    return DAG_ERR_WORKSPACE;
  }
  char* base = (char*)dag_align_up((size_t)(uintptr_t)ws, 256);
  DecodeArgs a;
  a.group_branch_off = d->group_branch_off;
  a.shared_page_off = d->shared_page_off;
  a.shared_pages = d->shared_pages;
  a.shared_len = d->shared_len;
  a.branch_page_off = d->branch_page_off;
  a.branch_pages = d->branch_pages;
  a.branch_len = d->branch_len;
  a.q = (const uint16_t*)q;
  a.k_pool = (const uint16_t*)k_pool;
  a.v_pool = (const uint16_t*)v_pool;
  a.out = (uint16_t*)out;
  a.part_o_a = (float*)(base + p.off_o_a);
  a.part_ml_a = (float*)(base + p.off_ml_a);
  a.part_o_b = (float*)(base + p.off_o_b);
  a.part_ml_b = (float*)(base + p.off_ml_b);
  a.n_groups = d->n_groups;
  a.n_live = d->n_live;
  a.hq = hq;
  a.hkv = hkv;
  a.G = hq / hkv;
  a.rb_max = p.rb_max;
  a.chunk_a = p.chunk_a;
  a.splits_a = p.splits_a;
  a.chunk_b = p.chunk_b;
  a.splits_b = p.splits_b;
  a.items_a = p.items_a;
  a.items_b = p.items_b;
  a.scale = softmax_scale;
  a.sc = softmax_scale * 1.4426950408889634f;
  a.th = p.th / a.sc;
  a.settle = p.settle;
  hipStream_t stream = (hipStream_t)stream_;
  a.item_base = 0;
  if (p.whole) {
    if (head_dim == 128) hipLaunchKernelGGL(k_whole_branch<128>, dim3((unsigned)(d->n_live * hkv)), dim3(64 * WHOLE_WAVES), 0, stream, a);
    else hipLaunchKernelGGL(k_whole_branch<64>, dim3((unsigned)(d->n_live * hkv)), dim3(64 * WHOLE_WAVES), 0, stream, a);
    DAG_LAUNCH_CHECK();
    return DAG_OK;
  }
  unsigned items = (unsigned)(p.items_a + p.items_b);
  if (p.wide && p.items_a > 0) {
    // Wide sibling groups: one launch of workgroups with own items, of those that stream a slice of the shared pages
    // once for all rows of a group, and of the other own items.
    const unsigned shared_wgs = (unsigned)(d->n_groups * hkv * p.splits_a);
    const unsigned threads = 64u * WIDE_WAVES;
    const int n_cu = dag_compute_units();
    if (n_cu < 1) return DAG_ERR_HIP;
    a.wide_own = wide_own_waves(p.items_b, n_cu, a.G, head_dim);
    const unsigned own_wgs = (unsigned)dag_ceil_div(p.items_b, WIDE_WAVES / a.wide_own);
    // Half of the compute units start with own pages: an item keeps the memory idle for its first 6 us (lengths, page ids, pages), which all
    // of them at once waste and half of them leave to the others (2 x 32 siblings over 32 K: 9 us of 98).
    a.wide_first = (int)own_wgs < n_cu / 2 ? (int)own_wgs : n_cu / 2;
    const int sm = wide_lds_bytes(a.G, head_dim, a.wide_own);
    a.wide_shared = (int)shared_wgs;
    if (head_dim == 128) {
      if (hipFuncSetAttribute((const void*)k_decode_wide<128>, hipFuncAttributeMaxDynamicSharedMemorySize, sm) != hipSuccess)
        return DAG_ERR_HIP;
      hipLaunchKernelGGL(k_decode_wide<128>, dim3(shared_wgs + own_wgs), dim3(threads), sm, stream, a);
    } else {
      if (hipFuncSetAttribute((const void*)k_decode_wide<64>, hipFuncAttributeMaxDynamicSharedMemorySize, sm) != hipSuccess)
        return DAG_ERR_HIP;
      hipLaunchKernelGGL(k_decode_wide<64>, dim3(shared_wgs + own_wgs), dim3(threads), sm, stream, a);
    }
    DAG_LAUNCH_CHECK();
    items = 0;
  }
  if (items > 0) {
    if (head_dim == 128) hipLaunchKernelGGL(k_decode<128>, dim3(items), dim3(64), 0, stream, a);
    else hipLaunchKernelGGL(k_decode<64>, dim3(items), dim3(64), 0, stream, a);
    DAG_LAUNCH_CHECK();
  }
  const int64_t rows = (int64_t)d->n_live * hq;
  const bool few = rows <= MERGE_FEW_ROWS;
  auto* const merge = head_dim == 128 ? (few ? k_decode_merge<128, true> : k_decode_merge<128, false>)
                                      : few ? k_decode_merge<64, true> : k_decode_merge<64, false>;
  hipLaunchKernelGGL(merge, dim3((unsigned)dag_ceil_div(rows, merge_threads(few) / 64)), dim3(merge_threads(few)), 0, stream, a);
  DAG_LAUNCH_CHECK();
  return DAG_OK;
}

}  // namespace

extern "C" int dag_attn_decode(const dag_decode_desc_t* d, const void* q, const void* k_pool, const void* v_pool,
                               void* out, int32_t hq, int32_t hkv, int32_t head_dim, float softmax_scale, void* ws,
                               size_t ws_bytes, void* stream_) {
  return decode_impl(d, q, k_pool, v_pool, out, hq, hkv, head_dim, softmax_scale, ws, ws_bytes, stream_, false);
}

extern "C" int dag_attn_decode_static(const dag_decode_desc_t* d, const void* q, const void* k_pool,
                                      const void* v_pool, void* out, int32_t hq, int32_t hkv, int32_t head_dim,
                                      float softmax_scale, void* stream_) {
  return decode_impl(d, q, k_pool, v_pool, out, hq, hkv, head_dim, softmax_scale, nullptr, 0, stream_, true);
}

extern "C" size_t dag_decode_segments_workspace_bytes(const dag_decode_seg_desc_t* desc, int32_t hq, int32_t hkv,
                                                      int32_t head_dim) {
  SegPlan p;
  if (make_seg_plan(desc, hq, hkv, head_dim, decode_knobs(), &p) != DAG_OK) return 0;
  return p.bytes;
}

extern "C" int dag_attn_decode_segments(const dag_decode_seg_desc_t* d, const void* q, const void* k_pool,
                                        const void* v_pool, void* out, int32_t hq, int32_t hkv, int32_t head_dim,
                                        float softmax_scale, void* ws, size_t ws_bytes, void* stream_) {
  SegPlan p;
  const int rc = make_seg_plan(d, hq, hkv, head_dim, decode_knobs(), &p);
  if (rc != DAG_OK) return rc;
  if (d->n_live == 0) return DAG_OK;
  if (!q || !k_pool || !v_pool || !out || !d->branch_entry_off || !d->branch_entries) return DAG_ERR_NULL;
  if (d->n_segments > 0 &&
      (!d->seg_page_off || !d->seg_pages || !d->seg_len || !d->seg_reader_off || !d->seg_readers))
    return DAG_ERR_NULL;
  if (!dag_aligned16(q) || !dag_aligned16(k_pool) || !dag_aligned16(v_pool) || !dag_aligned16(out))
    return DAG_ERR_ALIGN;
  if (!ws || ws_bytes < p.bytes) return DAG_ERR_WORKSPACE;
  char* base = (char*)dag_align_up((size_t)(uintptr_t)ws, 256);
  SegArgs a;
  a.seg_page_off = d->seg_page_off;
  a.seg_pages = d->seg_pages;
  a.seg_len = d->seg_len;
  a.seg_reader_off = d->seg_reader_off;
  a.seg_readers = d->seg_readers;
  a.seg_reader_len = d->seg_reader_len;
  a.branch_entry_off = d->branch_entry_off;
  a.branch_entries = d->branch_entries;
  a.q = (const uint16_t*)q;
  a.k_pool = (const uint16_t*)k_pool;
  a.v_pool = (const uint16_t*)v_pool;
  a.out = (uint16_t*)out;
  a.part_o = (float*)(base + p.off_o);
  a.part_ml = (float*)(base + p.off_ml);
  a.items = (SegItem*)(base + p.off_items);
  a.totals = (int32_t*)(base + p.off_total);
  a.entry_first = (int32_t*)(base + p.off_first);
  a.item_cap = (int)p.items;
  a.n_segments = d->n_segments;
  a.n_live = d->n_live;
  a.hq = hq;
  a.hkv = hkv;
  a.G = hq / hkv;
  a.rb_max = p.rb_max;
  a.chunk = p.chunk;
  a.splits = p.splits;
  a.total_readers = d->total_readers;
  a.fixed = decode_knobs().chunk_seg > 0;
  a.weight = (float)hkv * (float)head_dim / 128.f;
  const int64_t most_pages = (int64_t)d->n_segments * p.rb_max * d->max_seg_pages * hkv * head_dim;
  a.few = !a.fixed && p.chunk == 8 && most_pages < (d->max_seg_pages <= SEG_SHORT ? SEG_PAGES_16_SHORT : SEG_PAGES_16) * 128;
  a.sc = softmax_scale * 1.4426950408889634f;
  a.th = ITEM_TH / a.sc;
  hipStream_t stream = (hipStream_t)stream_;
  if (p.items > 0) {
    const int64_t waves = dag_ceil_div(d->n_segments, 64);
    hipLaunchKernelGGL(k_seg_plan, dim3(1), dim3((unsigned)(waves * 64 < PLAN_THREADS ? waves * 64 : PLAN_THREADS)), 0, stream, a);
    DAG_LAUNCH_CHECK();
    const unsigned grid = (unsigned)(p.items * hkv);
    if (head_dim == 128) hipLaunchKernelGGL(k_decode_seg<128>, dim3(grid), dim3(64), 0, stream, a);
    else hipLaunchKernelGGL(k_decode_seg<64>, dim3(grid), dim3(64), 0, stream, a);
    DAG_LAUNCH_CHECK();
  }
  const unsigned nout = (unsigned)(d->n_live * hq);
  if (head_dim == 128) hipLaunchKernelGGL(k_decode_seg_merge<128>, dim3(nout), dim3(64), 0, stream, a);
  else hipLaunchKernelGGL(k_decode_seg_merge<64>, dim3(nout), dim3(64), 0, stream, a);
  DAG_LAUNCH_CHECK();
  return DAG_OK;
}
