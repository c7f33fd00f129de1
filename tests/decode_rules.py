"""The split rules of the decode steps as the library has them: csrc/decode_plan.h compiled for the host, so that a test can state
the route of each of its cases and a changed rule cannot take the case elsewhere unnoticed."""
import atexit
import ctypes as C
import functools
import os
import shutil
import subprocess
import tempfile
from types import SimpleNamespace

from paper_2602_07529_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "decode_plan.h"
extern "C" int decode_rules(const dag_decode_desc_t* d, int hq, int hkv, int D, const int* knobs, double* out) {
  DecodePlan p{};
  const int rc = make_plan(d, hq, hkv, D, DecodeKnobs{knobs[0], knobs[1], knobs[2]}, &p);
  const double v[] = {(double)p.rb_max, (double)p.chunk_a, (double)p.splits_a, (double)p.chunk_b, (double)p.splits_b, (double)p.wide,
                      (double)p.whole, p.th, p.settle, (double)p.bytes};
  for (int i = 0; i < 10; ++i) out[i] = v[i];
  return rc;
}
extern "C" int segment_rules(const dag_decode_seg_desc_t* d, int hq, int hkv, int D, const int* knobs, double* out) {
  SegPlan p{};
  const int rc = make_seg_plan(d, hq, hkv, D, DecodeKnobs{knobs[0], knobs[1], knobs[2]}, &p);
  const double v[] = {(double)p.rb_max, (double)p.chunk, (double)p.splits, (double)p.items, (double)p.off_items, (double)p.off_total,
                      (double)p.bytes};
  for (int i = 0; i < 7; ++i) out[i] = v[i];
  return rc;
}
"""


@functools.lru_cache(maxsize=None)
def _lib():
    folder = tempfile.mkdtemp()
    atexit.register(shutil.rmtree, folder, ignore_errors=True)
    src, so = os.path.join(folder, "rules.cpp"), os.path.join(folder, "rules.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(ROOT, "paper_2602_07529_amd", "csrc"), src, "-o", so], check=True)
    return C.CDLL(so)


def _call(fn, names, desc, hq, hkv, d, knobs):
    out, k = (C.c_double * len(names))(), (C.c_int * 3)(*knobs)
    rc = fn(C.byref(desc), hq, hkv, d, k, out)
    plan = SimpleNamespace(rc=rc, **{n: (v if n in ("th", "settle") else int(v)) for n, v in zip(names, out)})
    return plan


def decode(desc, hq, hkv, d, knobs=(0, 0, 0)):
    """Plan of dag_attn_decode for a dag_decode_desc_t; `route`: 'whole' (k_whole_branch), 'wide' (k_decode_wide) or 'items' (k_decode)."""
    names = ("rb_max", "chunk_a", "splits_a", "chunk_b", "splits_b", "wide", "whole", "th", "settle", "bytes")
    plan = _call(_lib().decode_rules, names, desc, hq, hkv, d, knobs)
    plan.route = "whole" if plan.whole else "wide" if plan.wide and plan.splits_a else "items"
    return plan


def step(groups, branches, shared_pages, own_pages, hq, hkv, d, **kw):
    """The same for `groups` groups of `branches` branches with these numbers of pages."""
    return decode(B.dag_decode_desc_t(groups, groups * branches, 16, shared_pages, own_pages, branches, *([0x1000] * 8)), hq, hkv, d, **kw)


def segments(desc, hq, hkv, d, knobs=(0, 0, 0)):
    """What the host settles for dag_attn_decode_segments."""
    return _call(_lib().segment_rules, ("rb_max", "chunk", "splits", "items", "off_items", "off_total", "bytes"), desc, hq, hkv, d, knobs)


def listed_slices(plan, ws):
    """{(first page-list position, first page): pages} of the work items that k_seg_plan left in a workspace (a uint8 array of the host)."""
    n = int(ws[plan.off_total:plan.off_total + 4].view("int32")[0])
    items = ws[plan.off_items:plan.off_items + 32 * n].view("int32").reshape(n, 8)
    return {(int(i[0]), int(i[5])): int(i[7]) >> 23 & 0x1fe for i in items}
