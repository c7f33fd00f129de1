"""GPU: a key has the same angles whether dag_rope_qk or dag_kv_append_rope rotates it.  The key (1, .., 1, 0, .., 0) becomes the
cosines and sines themselves; at positions of up to 2^31 - 1 a frequency that is off by its last bit moves them by up to 2^-22,
which 16 bits show in a few of the millions compared."""
import numpy as np
import pytest
import torch

from paper_2602_07529_amd import binding as B
from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu


# 1000 entries: the kernel of one entry each; 20,000: that of runs
@pytest.mark.parametrize("n", [1000, 20000])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("theta", [0.5, 2.0, 10000.0, 500000.0, float("inf")])
def test_append_and_rope_agree(n, d, theta):
    rng = np.random.Generator(np.random.PCG64(n + d))
    pos = np.concatenate([rng.integers(0, 2 ** 31, n - 4), [0, 1, 2 ** 31 - 2, 2 ** 31 - 1]]).astype(np.int32)
    hkv, pages = 2, -(-n // 16)
    k = torch.zeros(n, hkv, d, dtype=torch.bfloat16, device=DEV)
    k[:, :, :d // 2] = 1.0
    dd = B.DecodeDesc(dict(n_groups=0, n_live=n, page_size=16, group_branch_off=[0], shared_page_off=[0], shared_pages=[0], shared_len=[0],
                           branch_page_off=np.arange(n + 1), branch_pages=np.arange(n) // 16, branch_len=np.arange(n) % 16 + 1, branch_pos=pos), DEV)
    k_pool = torch.zeros(pages, hkv, d // 8, 16, 8, dtype=torch.bfloat16, device=DEV)
    v_pool = torch.zeros(pages, hkv, d, 16, dtype=torch.bfloat16, device=DEV)
    B.dag_kv_append_rope(dd, k, torch.zeros_like(k), k_pool, v_pool, theta)
    got = k_pool.permute(0, 3, 1, 2, 4).reshape(pages * 16, hkv, d)[:n]
    for dtype in (torch.float32, torch.bfloat16):
        want = k.to(dtype)
        B.dag_rope_qk(torch.from_numpy(pos).to(DEV), None, want, theta)
        torch.cuda.synchronize()
        assert torch.isfinite(want.float()).all()
        assert torch.equal(got, want.to(torch.bfloat16)), "%d of %d differ" % ((got != want.to(torch.bfloat16)).sum(), got.numel())
