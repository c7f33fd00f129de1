// Split rules of the decode steps: host code without HIP, so that the tests can compile it by itself.
#pragma once
#include "dagattn.h"
#include "sizes.h"

constexpr int PAGE = DAG_PAGE_SIZE;

// Single-wave items: log2 of how far a score may exceed the reference maximum.  Probabilities lose less to 16 bits the nearer it is to
// their maximum: error against 64 bits over 100 shapes 0.95 of that at 8, and the time of the largest steps the same (at 0: 0.93, and 0.2 %).
constexpr float ITEM_TH = 1.f;

constexpr int WIDE_MAX_BLOCKS = 8;     // k_decode_wide: row blocks of a workgroup
constexpr int WIDE_MAX_PAGES = 128;    // of a shared slice: its page ids sit in two registers
constexpr int WHOLE_ROWS = 8;          // k_whole_branch: query heads of a KV head
// Up to these pages in a context (a wave walks its slice alone, 1 us a block) and workgroups (one a compute unit: two take turns);
// 88 random steps with up to 8 rows a branch: inside 1.02 to 1.40 times as fast as items and merge; above 64 pages of dimension 128
// 0.99 to 1.16, above 110 0.66 to 0.92, between 257 and 360 workgroups 0.82 to 0.98, above that 0.68 to 1.25.
constexpr int WHOLE_PAGES_128 = 64, WHOLE_PAGES_64 = 96, WHOLE_GROUPS = 256;
constexpr int SEG_PAGES_16 = 2048, SEG_PAGES_32 = 9216, SEG_PAGES_64 = 32768, SEG_PAGES_128 = 65536;
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
// What is left takes slices that make a hundred workgroups with shared pages and 256 with own ones, not 256 and 512:
// each slice leaves 32 rows of sums that the merge reads (a group of 22 branches over 13,072 tokens, four KV heads: 103 slices of 8
// pages 32.4 us, 26 of 32 pages 20.2; 135 random shapes of both kinds 1.09 times as fast, four of them 3 to 7 % slower).
// Longer slices have fewer references, and probabilities lose less to 16 bits the nearer the reference is to their maximum, so where
// slices get longer it follows the maximum: always in single waves, in k_decode_wide when the sum of 16 probabilities grows by 2.5
// (error against 64 bits, 110 shapes, with : without longer slices 0.997 on average, 0.95 to 1.05; by 4 1.006, by 1024 as elsewhere 1.017).
// The workspace keeps the size of the shorter slices: buffers sized by an earlier library stay as good as they were.
constexpr int NARROW_CONTEXT_PAGES = 256, NARROW_PAGES = 5632, NARROW_OWN_PAGES = 6400;
inline int make_plan(const dag_decode_desc_t* d, int hq, int hkv, int D, const DecodeKnobs& knobs, DecodePlan* p) {
  if (!d) return DAG_ERR_NULL;
  if (d->n_groups < 0 || d->n_live < 0 || d->max_shared_pages < 0 || d->max_branch_pages < 0 || d->max_group_size < 0)
    return DAG_ERR_BAD_LEN;
  if (d->page_size != PAGE) return DAG_ERR_UNSUPPORTED;
  if (hq < 1 || hkv < 1 || hq % hkv != 0 || hq / hkv > 32) return DAG_ERR_UNSUPPORTED;
  if (D != 64 && D != 128) return DAG_ERR_UNSUPPORTED;
  const int G = hq / hkv;
  p->rb_max = (int)dag_ceil_div((int64_t)d->max_group_size * G, 32);
  if (p->rb_max < 1) p->rb_max = 1;
  const int64_t base_a = (int64_t)d->n_groups * hkv * p->rb_max;
  const int64_t base_b = (int64_t)d->n_live * hkv;
  p->wide = p->rb_max >= 2 && p->rb_max <= WIDE_MAX_BLOCKS;
  p->th = p->wide ? 8.f : ITEM_TH;
  p->settle = 1024.f;
  // Slices of at least `least` pages, halved until there are `shared` / `own` workgroups or waves.  An eighth more than that
  // (`longer`; two pages at least) where it saves a slice: a context of 65 pages was one of 64 and one of a page, which is a partial as
  // large as any (60 random steps 1.02 times as fast, one sequence of 509 shared and 43 own pages 17.2 -> 15.4 us).
  auto slices = [&](bool wide, int64_t shared, int least, int64_t own, bool longer) {
    int ca = knobs.chunk_a ? knobs.chunk_a : 128, cb = knobs.chunk_b ? knobs.chunk_b : 64;
    ca += ca & 1;
    cb += cb & 1;
    if (p->wide && ca > WIDE_MAX_PAGES) ca = WIDE_MAX_PAGES;
    const int64_t base = wide ? (int64_t)d->n_groups * hkv : base_a;
    if (!knobs.chunk_a)
      while (ca > least && base * dag_ceil_div(d->max_shared_pages, ca) < shared) ca /= 2;
    if (!knobs.chunk_b)
      while (cb > 4 && base_b * dag_ceil_div(d->max_branch_pages, cb) < own) cb /= 2;
    auto stretch = [&](int pages, int c, int most) {
      const int more = c + (c / 8 > 2 ? c / 8 : 2), longest = more < most ? more : most, n = (int)dag_ceil_div(pages, longest);
      return n > 0 && n < dag_ceil_div(pages, c) ? ((pages + n - 1) / n + 1) & ~1 : c;
    };
    if (longer && !knobs.chunk_a) ca = stretch(d->max_shared_pages, ca, p->wide ? WIDE_MAX_PAGES : INT32_MAX);
    if (longer && !knobs.chunk_b) cb = stretch(d->max_branch_pages, cb, INT32_MAX);
    p->splits_a = d->max_shared_pages > 0 ? (int)dag_ceil_div(d->max_shared_pages, ca) : 0;
    p->splits_b = d->max_branch_pages > 0 ? (int)dag_ceil_div(d->max_branch_pages, cb) : 0;
    if (wide && !knobs.chunk_a && p->splits_a > 1) {  // slices of one length, unless that is more rounds of workgroups
      const int same = ((d->max_shared_pages + p->splits_a - 1) / p->splits_a + 1) & ~1;
      if (dag_ceil_div(base * p->splits_a, 256) * same <= dag_ceil_div(base * (p->splits_a - 1), 256) * ca) ca = same;
    }
    p->chunk_a = ca;
    p->chunk_b = cb;
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
  const int rc = slices(p->wide, p->wide ? 256 : 512, 8, p->wide ? 512 : 1024, false);
  if (rc != DAG_OK) return rc;
  const size_t bytes = p->bytes;  // (what follows has at most as many items of either kind)
  const int shorter_a = p->chunk_a, shorter_b = p->chunk_b;
  if (!p->wide) {
    slices(false, 512, 8, 1024, true);
  } else if (d->max_shared_pages <= NARROW_CONTEXT_PAGES && base_a * d->max_shared_pages * D <= NARROW_PAGES * 128 &&
      base_b * d->max_branch_pages * D <= NARROW_OWN_PAGES * 128) {
    slices(false, 512, 8, 512, true);
    p->wide = false;
    p->th = 0.f;
  } else {
    slices(true, 100, 16, 256, true);
    auto length = [](int pages, int c) { return pages < c ? pages : c; };
    if (length(d->max_shared_pages, p->chunk_a) > length(d->max_shared_pages, shorter_a)) p->settle = 2.5f;
    if (p->chunk_a > shorter_a || p->chunk_b > shorter_b) p->th = 0.f;
  }
  p->bytes = bytes;
  p->whole = G <= WHOLE_ROWS && !knobs.chunk_a && !knobs.chunk_b && base_b <= WHOLE_GROUPS &&
             (int64_t)d->max_shared_pages + d->max_branch_pages <= (D == 128 ? WHOLE_PAGES_128 : WHOLE_PAGES_64);
  if (p->whole) p->th = 0.f;
  return DAG_OK;
}

struct SegPlan {
  int rb_max, chunk, splits;
  long items;  // bound on the work items (per kv head)
  size_t off_o, off_ml, off_items, off_total, off_first, bytes;
};

// One split size for all segments (their lengths live in device memory): as long as possible
// while the launch still has about a thousand items if every segment were the longest one.
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
