// Split rules of the decode steps: host code without HIP, so that the tests can compile it by itself.
#pragma once
#include "dagattn.h"
#include "sizes.h"

constexpr int PAGE = DAG_PAGE_SIZE;

// Single-wave items: log2 of how far a score may exceed the reference maximum.  Probabilities lose less to 16 bits the nearer it is to
// their maximum: error against 64 bits over 80 frontiers 0.99 of that at 8 (at 1 0.95), over 120 decode steps with these slices 0.996 (0.97).
// But at 1 some row of a wave raises its reference in most blocks: 14 x 16 leaves under 4 x 1,791 and 3,991 tokens 50.1 -> 52.3 us, 12
// leaves under 1,729 and 1,156 17.5 -> 18.6; at 3 the times are those at 8.
constexpr float ITEM_TH = 3.f;

constexpr int WIDE_WAVES = 8;          // k_decode_wide: waves of a workgroup, two per SIMD
constexpr int WIDE_MAX_BLOCKS = 8;     // row blocks of a workgroup
constexpr int WIDE_TILE_PAGES = 4;     // of a tile of the pipeline: what a slice has beyond whole ones is a unit by itself
constexpr int WIDE_MAX_PAGES = 128;    // of a shared slice: its page ids sit in two registers
constexpr int WIDE_LDS_BYTES = 160 * 1024;
// LDS of workgroups with own pages: the query operands and the partials of their items
inline int wide_own_bytes(int G, int D, int waves) { return WIDE_WAVES / waves * (D / 16 * 1024) + WIDE_WAVES * G * (D + 6) * 4; }
// Waves to an own item: as many as leave a workgroup for every compute unit (512 items of 40 pages by themselves: eight waves each
// 30.5 us, four 27.9).
inline int wide_own_waves(int64_t items, int units, int G, int D) {
  int waves = WIDE_WAVES;
  while (waves > 1 && items * waves > (int64_t)WIDE_WAVES * units && wide_own_bytes(G, D, waves / 2) <= WIDE_LDS_BYTES) waves /= 2;
  return waves;
}
constexpr int WHOLE_ROWS = 8;          // k_whole_branch: query heads of a KV head
// k_whole_branch takes a (branch, KV head) whole in one workgroup, so that every branch reads the shared pages for itself.  Its lines, from
// 170 steps with up to 8 rows a branch, as fast : items and merge; inside them 0.95 to 1.55, 1.24 on average:
// - 256 workgroups, one a compute unit: between 257 and 360 two take turns, 0.82 to 0.98.
// - pages in a context (a wave walks its slice alone, 1 us a block), and shared ones among them, which items read in longer slices than
//   own ones: branches of one row block above 52 or 41 pages of dimension 128 0.90 to 1.1, above 56 shared ones of 64 0.89 to 1.05.  More
//   row blocks read the shared pages as often when they are items: 64 pages of dimension 128, at 64 below 79 shared ones (0.92).
// - shared pages that pass through more than one L2: workgroups go to the eight dies in turn, so the siblings of a group are on eight of them,
//   on four, two or one if hkv is a multiple of two, four or eight.  What they fetch again, in pages of 128 dimensions (16 groups of 8
//   branches over 560 tokens, 4 / 1 heads: 3920 pages, 11.9 us as items and 15.1 so): above 1500 of one row block 0.77 to 1.04 (once 1.12), above 3000 of more 0.84 to 1.04.
constexpr int WHOLE_GROUPS = 256, WHOLE_DIES = 8;
inline bool whole_branches(int64_t base_w, int64_t base_b, int branches, int hkv, int G, int D, bool one_block, int64_t shared, int64_t own) {
  if (G > WHOLE_ROWS || base_b > WHOLE_GROUPS) return false;
  if (shared + own > (D == 64 ? 96 : one_block ? 52 : 64) || shared > (D == 64 ? (one_block ? 56 : 76) : one_block ? 41 : 64)) return false;
  int64_t dies = WHOLE_DIES;  // a group's workgroups are on
  while (dies > 1 && hkv % (2 * WHOLE_DIES / dies) == 0) dies /= 2;
  if (dies > branches) dies = branches;
  return (dies - 1) * base_w * shared * D <= (one_block ? 1500 : 3000) * 128;
}
// Decode over segments: k_seg_plan settles the slices, because the host knows the longest segment only and takes every other one for as
// long.  Pages of 128 dimensions to be read (once for every row block) and the slices that were fastest over 150 frontiers of 200 to
// 100,000 pages: 8 pages below 2,048, below 4,160 too if no segment has more than 96 (few partials to a branch: 11 x 12 leaves of 249 tokens
// under segments of 90 and 44, 8 heads on one: 17.5 us in slices of 16, 15.4 so), 16 below 9,216, 32 below 32,768, 64 below 81,920, then 128 -- if the
// lists have room for so many, which have the sizes that the host's slices ask for: else twice as long.  5 x 12 leaves under segments of 25 and 174 pages,
// 24 / 4 heads: 60 us with the host's slices, 38 so.  A segment's slices have one length, from 32 pages on an eighth more than that if this
// saves a slice (16 sequences of 254 to 258 | 2 x 126 to 130 | 8 x 63 to 67 pages: 227 -> 212 us); shorter ones are a chain of blocks
// that is all a launch of so few consists of (12 branches over 34, 26 and 20 pages, 32 / 8 heads: slices of 18 pages 15.4 us, of 16 14.3).
constexpr int SEG_PAGES_16 = 2048, SEG_PAGES_16_SHORT = 4160, SEG_SHORT = 96, SEG_PAGES_32 = 9216, SEG_PAGES_64 = 32768, SEG_PAGES_128 = 81920;
constexpr int SEG_STRETCH = 32;
// k_decode_merge: rows (branches x query heads) up to which a wave takes several partials to a load, 16 loads at a time
constexpr int64_t MERGE_FEW_ROWS = 4096;
constexpr size_t SEG_ITEM_BYTES = 32;  // of the list of work items

// Development knobs (pages per decode work item); 0 = not set, the split sizes then follow the shape of the batch.
struct DecodeKnobs {
  int chunk_a, chunk_b, chunk_seg;
};

struct DecodePlan {
  int rb_max, chunk_a, splits_a, chunk_b, splits_b, items_a, items_b;
  bool wide;  // shared items by k_decode_wide (one workgroup per group, kv head and split)
  bool whole;  // no items: k_whole_branch
  float th, settle;  // log2 of how far a score may exceed the reference maximum; DecodeArgs::settle
  size_t off_o_a, off_ml_a, off_o_b, off_ml_b, bytes;
};

// Split sizes: slices as long as the batch allows (every work item pays a start-up latency and
// writes a partial, so fewer and longer items stream better) while still giving the GPU about two
// waves per SIMD; both even so that a 32-key block never straddles a split.
//
// Wide groups, two to WIDE_MAX_BLOCKS row blocks of a KV head.  With little to read the single-wave items take them like any other
// group, every row block reading the shared pages for itself: a workgroup of k_decode_wide costs 5 us before its first tile.  Pages
// of 128 dimensions, shared ones once for each row block: up to 256 in a context, 5632 in all, and 6400 of the branches' own (96
// random shapes, single waves : k_decode_wide below these lines 0.55 to 1.14, 0.87 on average, a step of 2 x 25 branches over 500
// tokens 17.0 -> 12.6 us; above 5632 shared pages up to 2.5, above 256 in a context 1.04 to 1.25, above 6400 own ones 0.9 to 1.37).
constexpr int NARROW_CONTEXT_PAGES = 256, NARROW_PAGES = 5632, NARROW_OWN_PAGES = 6400;

// What is left: a compute unit has room for one workgroup of k_decode_wide, and each slice leaves 32 rows of sums that the merge
// reads, so the shared pages get WIDE_GROUPS workgroups and the own ones 256, in slices of one length.  At head dimension 64, where a
// page takes its time in exponentials and not in memory, the shared pages get a workgroup for every unit if their slices are longer
// than WIDE_LONG_64 pages (WIDE_LONG_64_TALL where a wave has a row block for itself) and the own pages are not the greater part.  If
// that is more than one for each unit, the last workgroups with own pages begin when the first end: where two of them in a row
// take a quarter longer than a shared one, the shared pages get as many as fit beside them (12 groups of 14 siblings over 3,849 shared and
// 1,181 own tokens, five heads on one: 30.6 us, with 128 workgroups 39.5, with those of the shorter slices 45.1).  The times are those
// that fit the measured steps best, in units of 0.05 us: 5 us and half a microsecond a page of a wave with own pages, 6 us and 0.35 (0.25 at dimension 64)
// a page of a workgroup with shared ones.  Slices of eight pages become 16 where there are more than 64 of them or twice as many own
// pages as shared ones: fewer partials.  If the longest slices there are still make more than WIDE_GROUPS workgroups, they are as
// short as a workgroup for every unit makes them (12 groups of 19 over 11,129 tokens, 8 / 2 heads: 77 -> 66 us), and the
// shorter slices stay where their workgroups have room at once and these do not (29 siblings over 936 and 574 tokens, 48 / 8 heads: 29.8 -> 25.6).
// A quarter longer at most where the merge has a round less to go (31 siblings over 19,910 and 125 tokens, 8 / 2 heads of dimension 64: 65 partials 19.2 us,
// 54 17.6; 200 shapes 1.002 times as fast, 0.97 at least).
// Whole tiles: half a tile more (2 groups of 10 over 6,598 and 969 tokens, 12 / 2 heads: slices of 14 pages 21.3 us, of 16 19.7; 180 shapes
// 1.005 times as fast, 0.98 at least).
// 180 random shapes against the slices that `bytes` is for: dimension 64 1.11 times as fast on average (0.91 to 1.42), 128 1.15
// (0.99 to 1.55); with a hundred workgroups and 16 pages at least everywhere 1.04 (0.79 to 1.37) and 1.11 (0.85 to 1.43).
// Longer slices have fewer references, and probabilities lose less to 16 bits the nearer the reference is to their maximum, so where
// slices get longer it follows the maximum: always in single waves, in k_decode_wide when the sum of 16 probabilities grows by 3 (2.5 at
// dimension 128): error against 64 bits over these shapes, with : without longer slices, 0.996 and 1.000 on average, 0.96 to 1.05;
// by 4 1.002 and 1.011, by 1024 as elsewhere 1.014 and 1.021.
// The workspace keeps the size of the shorter slices: buffers sized by an earlier library stay as good as they were.
constexpr int WIDE_UNITS = 256, WIDE_GROUPS = 128, WIDE_BESIDE = 48, WIDE_LONG_64 = 64, WIDE_LONG_64_TALL = 42;

inline int make_plan(const dag_decode_desc_t* d, int hq, int hkv, int D, const DecodeKnobs& knobs, DecodePlan* p) {
  if (!d) return DAG_ERR_NULL;
  if (d->n_groups < 0 || d->n_live < 0 || d->max_shared_pages < 0 || d->max_branch_pages < 0 || d->max_group_size < 0)
    return DAG_ERR_BAD_LEN;
  if (d->page_size != PAGE) return DAG_ERR_UNSUPPORTED;
  if (hq < 1 || hkv < 1 || hq % hkv != 0 || hq / hkv > 32) return DAG_ERR_UNSUPPORTED;
  if (D != 64 && D != 128) return DAG_ERR_UNSUPPORTED;
  const int G = hq / hkv, shared = d->max_shared_pages, own = d->max_branch_pages;
  p->rb_max = (int)dag_ceil_div((int64_t)d->max_group_size * G, 32);
  if (p->rb_max < 1) p->rb_max = 1;
  const int64_t base_w = (int64_t)d->n_groups * hkv, base_a = base_w * p->rb_max, base_b = (int64_t)d->n_live * hkv;
  const bool wide = p->rb_max >= 2 && p->rb_max <= WIDE_MAX_BLOCKS;
  auto lay_out = [&](int ca, int cb) {
    p->chunk_a = ca;
    p->chunk_b = cb;
    p->splits_a = (int)dag_ceil_div(shared, ca);
    p->splits_b = (int)dag_ceil_div(own, cb);
    const int64_t ia = base_a * p->splits_a, ib = base_b * p->splits_b;
    if (ia + ib > INT32_MAX) return DAG_ERR_UNSUPPORTED;
    p->items_a = (int)ia;
    p->items_b = (int)ib;
    size_t off = 0;
    p->off_o_a = off;  off += dag_align_up((size_t)ia * 32 * D * 4, 256);
    p->off_ml_a = off; off += dag_align_up((size_t)ia * 32 * 2 * 4, 256);
    p->off_o_b = off;  off += dag_align_up((size_t)ib * G * D * 4, 256);
    p->off_ml_b = off; off += dag_align_up((size_t)ib * G * 2 * 4, 256);
    p->bytes = off + 256;
    return DAG_OK;
  };
  auto even = [](int64_t c) { return (int)(c + (c & 1)); };
  auto halved = [](int c, int least, int64_t base, int pages, int64_t want) {  // until there are `want` workgroups or waves
    while (c > least && base * dag_ceil_div(pages, c) < want) c /= 2;
    return c;
  };
  auto longer = [&](int pages, int c) {  // an eighth more (two pages at least) where it saves a slice
    const int64_t n = dag_ceil_div(pages, c + (c / 8 > 2 ? c / 8 : 2));
    return n > 0 && n < dag_ceil_div(pages, c) ? even(dag_ceil_div(pages, n)) : c;
  };
  int ca = knobs.chunk_a ? even(knobs.chunk_a) : halved(128, 8, wide ? base_w : base_a, shared, wide ? 256 : 512);
  int cb = knobs.chunk_b ? even(knobs.chunk_b) : halved(64, 4, base_b, own, wide ? 512 : 1024);
  if (wide && ca > WIDE_MAX_PAGES) ca = WIDE_MAX_PAGES;
  const int rc = lay_out(ca, cb);
  if (rc != DAG_OK) return rc;
  const size_t bytes = p->bytes;  // (what follows has at most as many items of either kind)
  p->wide = wide && base_w > 0 && shared > 0 &&
            (shared > NARROW_CONTEXT_PAGES || base_a * shared * D > NARROW_PAGES * 128 || base_b * own * D > NARROW_OWN_PAGES * 128);
  p->th = 8.f;
  p->settle = 1024.f;
  const int round = (int64_t)d->n_live * hq > MERGE_FEW_ROWS ? 16 : D == 128 ? 32 : 64;  // partials that the merge takes at a time
  if (!p->wide) {
    // Single waves: a slice takes a microsecond for two of its pages, so longer ones pay where the merge goes round once less (509 shared and
    // 43 own pages of one sequence, 75 partials and 59: 17.2 -> 15.4 us; 92 and 81, 33 and 24: 13.1 -> 12.0; where it does not, slices of ten
    // pages for eight and six for four cost up to a tenth: 94 and 16, 14.9 us for 14.5), and a last slice of an eighth of the others,
    // which is a partial as large as any, where they have 16 pages or more (91 and 18 pages of 117 branches, 16 / 8 heads: 61.4 -> 53.7;
    // slices that are merely fewer: 0.97 to 1.01).
    if (!knobs.chunk_a) ca = halved(128, 8, base_a, shared, 512);
    auto rounds = [&](int xa, int xb) { return dag_ceil_div(dag_ceil_div(shared, xa) + dag_ceil_div(own, xb), round); };
    auto joined = [&](int pages, int c) { return c >= 16 && pages > c && pages % c > 0 && pages % c <= c / 8 ? even(dag_ceil_div(pages, pages / c)) : c; };
    const int la = longer(shared, ca), lb = longer(own, cb);
    const bool merged = rounds(knobs.chunk_a ? ca : la, knobs.chunk_b ? cb : lb) < rounds(ca, cb);
    if (!knobs.chunk_a) ca = merged ? la : joined(shared, ca);
    if (!knobs.chunk_b) cb = merged ? lb : joined(own, cb);
    p->th = wide ? 0.f : ITEM_TH;
    lay_out(ca, cb);
  } else if (!knobs.chunk_a && !knobs.chunk_b) {
    int lb = longer(own, halved(64, 4, base_b, own, 256));
    if (lb < cb) lb = cb;
    if (own > lb) lb = even(dag_ceil_div(own, dag_ceil_div(own, lb)));  // of one length
    const int64_t items = base_b * dag_ceil_div(own, lb);
    const int waves = wide_own_waves(items, WIDE_UNITS, G, D);
    const int64_t beside = WIDE_UNITS - dag_ceil_div(items, WIDE_WAVES / waves);
    const int64_t own_time = 100 + 10 * dag_ceil_div(own < lb ? own : lb, waves);
    auto slice = [&](int64_t groups) {  // of that many workgroups
      const int64_t c = dag_ceil_div(shared, base_w < groups ? groups / base_w : 1);
      return c < WIDE_MAX_PAGES ? even(c) : WIDE_MAX_PAGES;
    };
    int la = slice(WIDE_GROUPS);
    if (D == 64 && la > (p->rb_max <= WIDE_WAVES / 2 ? WIDE_LONG_64 : WIDE_LONG_64_TALL) && base_b * own < base_w * shared) la = slice(WIDE_UNITS);
    if (base_w * dag_ceil_div(shared, la) > WIDE_GROUPS) la = slice(WIDE_UNITS);
    const int64_t shared_time = 120 + (D == 64 ? 5 : 7) * (int64_t)la;
    if (base_w * dag_ceil_div(shared, la) > beside && 8 * own_time > 5 * shared_time && beside >= WIDE_BESIDE) la = slice(beside);
    if (la < 16 && (dag_ceil_div(shared, 8) > 64 || base_b * own >= 2 * base_w * shared)) la = 16;
    auto tiles = [](int64_t c) { return (c + WIDE_TILE_PAGES - 1) / WIDE_TILE_PAGES * WIDE_TILE_PAGES; };
    const int64_t own_slices = dag_ceil_div(own, lb), room = (dag_ceil_div(shared, la) + own_slices - 1) / round * round - own_slices;
    const int64_t fewer = room > 0 ? tiles(dag_ceil_div(shared, room)) : 0;  // pages of slices with which the merge goes round once less
    if (fewer > la && fewer <= la + la / 4 && fewer <= WIDE_MAX_PAGES) la = (int)fewer;
    if (la > 8) la = (int)tiles(la);
    if (la < ca) la = ca;
    auto together = [&](int xa, int xb) {
      const int64_t n = base_b * dag_ceil_div(own, xb);
      return base_w * dag_ceil_div(shared, xa) + dag_ceil_div(n, WIDE_WAVES / wide_own_waves(n, WIDE_UNITS, G, D)) <= WIDE_UNITS;
    };
    if (together(ca, cb) && !together(la, lb)) {
      la = ca;
      lb = cb;
    }
    if ((la < shared ? la : shared) > (ca < shared ? ca : shared)) p->settle = D == 64 ? 3.f : 2.5f;
    if (la > ca || lb != cb) p->th = 0.f;
    lay_out(la, lb);
  }
  p->bytes = bytes;
  p->whole = !knobs.chunk_a && !knobs.chunk_b && whole_branches(base_w, base_b, d->max_group_size, hkv, G, D, p->rb_max == 1, shared, own);
  if (p->whole) p->th = 0.f;
  return DAG_OK;
}

struct SegPlan {
  int rb_max, chunk, splits;
  long items;  // bound on the work items (per kv head)
  size_t off_o, off_ml, off_items, off_total, off_first, bytes;
};

// What the lists have room for: one split size for all segments (their lengths live in device memory), as long as possible while the
// launch still has about a thousand items if every segment were the longest one.  k_seg_plan settles the slices that are taken.
inline int make_seg_plan(const dag_decode_seg_desc_t* d, int hq, int hkv, int D, const DecodeKnobs& knobs, SegPlan* p) {
  if (!d) return DAG_ERR_NULL;
  if (d->n_live < 0 || d->n_segments < 0 || d->max_seg_pages < 0 || d->max_readers < 0 || d->total_readers < 0)
    return DAG_ERR_BAD_LEN;
  if (d->page_size != PAGE) return DAG_ERR_UNSUPPORTED;
  if (hq < 1 || hkv < 1 || hq % hkv != 0 || hq / hkv > 32) return DAG_ERR_UNSUPPORTED;
  if (D != 64 && D != 128) return DAG_ERR_UNSUPPORTED;
  const int G = hq / hkv;
  p->rb_max = (int)dag_ceil_div((int64_t)d->max_readers * G, 32);
  if (p->rb_max < 1) p->rb_max = 1;
  const int knob = knobs.chunk_seg;
  int c = knob ? knob : 128;
  c += c & 1;
  const int64_t base = (int64_t)d->n_segments * hkv * p->rb_max;
  if (!knob)
    while (c > 8 && base * dag_ceil_div(d->max_seg_pages, c) < 1024) c /= 2;
  p->chunk = c;
  p->splits = d->max_seg_pages > 0 ? (int)dag_ceil_div(d->max_seg_pages, c) : 0;
  const int64_t items = (int64_t)d->n_segments * p->rb_max * p->splits;
  if (items * hkv > INT32_MAX) return DAG_ERR_UNSUPPORTED;
  p->items = (long)items;
  size_t off = 0;
  const size_t rows = (size_t)p->splits * (size_t)d->total_readers * hq;
  if (rows > (size_t)INT32_MAX) return DAG_ERR_UNSUPPORTED;
  p->off_o = off;  off += dag_align_up(rows * D * 4, 256);
  p->off_ml = off; off += dag_align_up(rows * 2 * 4, 256);
  p->off_items = off;  off += dag_align_up((size_t)items * SEG_ITEM_BYTES, 256);
  p->off_total = off;  off += 256;
  p->off_first = off; off += dag_align_up((size_t)d->total_readers * 4, 256);
  p->bytes = off + 256;
  return DAG_OK;
}
