"""GPU parity of the two cuts of the fp32 prefill kernel (row blocks side by side; the key tiles of a
row block divided over four waves), both chosen by the number of (query tile, head) pairs."""
import numpy as np
import pytest
import torch

from workloads import dags
from tests.gpu_util import check_close, oracle_prefill, run_prefill

pytestmark = pytest.mark.gpu


# query tiles of the batch below: 1 + 1 + 5 + 3 + 2 = 12, so 48 heads reach 512 workgroups and 12 do not
@pytest.mark.parametrize("hq,hkv,d", [(12, 4, 64), (6, 3, 128), (48, 4, 64), (48, 2, 128)])
def test_fp32_row_blocks_and_key_splits(hq, hkv, d):
    rng = np.random.Generator(np.random.PCG64(4400 + hq + d))
    dag_list = [dags.linear_chain([1]),                                                  # one row: three of four splits are empty
                dags.linear_chain([64]),
                dags.fork_join(130, [33, 64, 17], 30),                                   # ragged last tile, masked tiles
                dags.random_dag(rng, n_nodes=70, depth=6, len_lo=1, len_hi=4)[:2],       # two visibility words
                dags.linear_chain([49, 16])]                                             # ends inside a 16-row block
    T = int(sum(int(np.sum(L)) for L, _ in dag_list))
    q, k, v = dags.make_qkv(71 + d, T, hq, hkv, d, 1.0, torch.float32)
    out, lse, _, _, _ = run_prefill(dag_list, q, k, v, 1e4, want_lse=True)
    ref, ref_lse, _ = oracle_prefill(dag_list, q, k, v, 1e4)
    check_close(out, ref, torch.float32, "out")
    assert np.abs(lse.cpu().double().numpy() - ref_lse).max() < 1e-4
