"""GPU: dag_kv_append_rope over many entries at once against the same entries a few at a time (the one-entry
kernel, itself checked against the oracle): pools bit for bit, slots nobody stores to included."""
import numpy as np
import pytest
import torch

from paper_2602_07529_amd import binding as B
from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu


def _desc(page, length, pos):
    n, none = len(page), np.zeros(1, np.int32)
    return B.DecodeDesc(dict(n_groups=0, n_live=n, page_size=16, group_branch_off=none, shared_page_off=none,
                             shared_pages=none, shared_len=none, branch_page_off=np.arange(n + 1), branch_pages=page,
                             branch_len=length, branch_pos=pos), DEV)


# runs: tokens of consecutive slots, each run on pages of its own from a slot of its own on; 1: nothing but single entries
@pytest.mark.parametrize("hkv,d", [(8, 128), (1, 64), (3, 64), (2, 128)])
@pytest.mark.parametrize("runs", [[(0, 1024)], [(5, 1030)], [(8, 8), (0, 7), (15, 18), (3, 1000)], [(7, 1)] * 1040,
                                  [(b % 16, b % 37 + 1) for b in range(64)]])
def test_append_many_entries(runs, hkv, d):
    rng = np.random.Generator(np.random.PCG64(11 * hkv + d + len(runs)))
    slots = [(b, first + i) for b, (first, n) in enumerate(runs) for i in range(n)]
    pages_of = np.cumsum([0] + [-(-(first + n) // 16) for first, n in runs])
    perm = rng.permutation(int(pages_of[-1]) + 2)
    page = np.asarray([perm[pages_of[b] + s // 16] for b, s in slots], np.int32)
    length = np.asarray([s % 16 + 1 for _, s in slots], np.int32)
    length[rng.integers(0, len(slots), 3)] = 0   # an entry without a token stores nothing
    pos = rng.integers(0, 60000, len(slots)).astype(np.int32)
    n = len(slots)
    assert n >= 1024
    gen = torch.Generator(device=DEV).manual_seed(d)
    k_new, v_new = (torch.randn((n, hkv, d), generator=gen, device=DEV).bfloat16() for _ in range(2))
    pools = [torch.full((len(perm), hkv, d * 16), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(4)]
    B.dag_kv_append_rope(_desc(page, length, pos), k_new, v_new, pools[0], pools[1], 5e5)
    for i in range(0, n, 100):
        part = slice(i, min(i + 100, n))
        B.dag_kv_append_rope(_desc(page[part], length[part], pos[part]), k_new[part], v_new[part], pools[2], pools[3], 5e5)
    torch.cuda.synchronize()
    assert torch.equal(pools[0].view(torch.int16), pools[2].view(torch.int16))
    assert torch.equal(pools[1].view(torch.int16), pools[3].view(torch.int16))


# a decode step's descriptor (sibling groups, a page of its own for every branch) around the sizes where the kernel changes
@pytest.mark.parametrize("n", [1024, 8191, 8192])
def test_append_of_a_decode_step(n):
    hkv, d = 2, 64
    rng = np.random.Generator(np.random.PCG64(n))
    page, length = rng.permutation(n).astype(np.int32), rng.integers(0, 17, n).astype(np.int32)
    pos = rng.integers(0, 60000, n).astype(np.int32)
    gen = torch.Generator(device=DEV).manual_seed(n)
    k_new, v_new = (torch.randn((n, hkv, d), generator=gen, device=DEV).bfloat16() for _ in range(2))
    pools = [torch.full((n, hkv, d * 16), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(4)]
    none = np.zeros(1, np.int32)
    step = B.DecodeDesc(dict(n_groups=1, n_live=n, page_size=16, group_branch_off=np.asarray([0, n]), shared_page_off=np.zeros(2, np.int32),
                             shared_pages=none, shared_len=none, branch_page_off=np.arange(n + 1), branch_pages=page,
                             branch_len=length, branch_pos=pos), DEV)
    B.dag_kv_append_rope(step, k_new, v_new, pools[0], pools[1], 5e5)
    for i in range(0, n, 1000):
        part = slice(i, min(i + 1000, n))
        B.dag_kv_append_rope(_desc(page[part], length[part], pos[part]), k_new[part], v_new[part], pools[2], pools[3], 5e5)
    torch.cuda.synchronize()
    assert torch.equal(pools[0].view(torch.int16), pools[2].view(torch.int16))
    assert torch.equal(pools[1].view(torch.int16), pools[3].view(torch.int16))


# pointers that are not on 16 bytes (the others are taken 16 bytes at a time)
def test_append_of_many_unaligned_entries():
    n, hkv, d = 1030, 2, 64
    page, length = (np.arange(n) // 16).astype(np.int32), (np.arange(n) % 16 + 1).astype(np.int32)
    pos = np.arange(n).astype(np.int32)
    gen = torch.Generator(device=DEV).manual_seed(3)
    k_new, v_new = (torch.randn(n * hkv * d + 1, generator=gen, device=DEV).bfloat16() for _ in range(2))
    n_pages = int(page.max()) + 1
    pools = [torch.zeros((n_pages, hkv, d * 16), dtype=torch.bfloat16, device=DEV) for _ in range(4)]
    odd = [x[1:].view(n, hkv, d) for x in (k_new, v_new)]
    assert odd[0].data_ptr() % 16 == 2
    B.dag_kv_append_rope(_desc(page, length, pos), *odd, pools[0], pools[1], 5e5)
    B.dag_kv_append_rope(_desc(page, length, pos), odd[0].clone(), odd[1].clone(), pools[2], pools[3], 5e5)
    torch.cuda.synchronize()
    assert torch.equal(pools[0], pools[2]) and torch.equal(pools[1], pools[3])
