"""GPU: paged prefill whose rows of tiles are cut into pieces, and whose items take one or two heads, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, check_close
from tests.test_gpu_prefill_paged import _gpu_prefill_paged, _multilevel

pytestmark = pytest.mark.gpu


def _check(st, hq, hkv, d):
    out, lse = _gpu_prefill_paged(st, hq, hkv, d, want_lse=True)
    ref = orc.attn_decode_segments(st["desc"], dags.to_f64(st["q"]), dags.to_f64(st["k_pool"]), dags.to_f64(st["v_pool"]))
    check_close(out, ref, torch.bfloat16, "paged prefill out")
    assert torch.isfinite(lse).all()
    return out, lse


# contexts just long enough for pieces, of many pieces, pieces of masked tiles alone (77 new tokens behind full pages), and
# a workspace without room for them: the same row sums, from one piece
@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 128), (5, 1, 64), (2, 2, 128), (8, 1, 64)])
@pytest.mark.parametrize("lens,new", [([1470, 80], 77), ([1472, 64], 64), ([3000, 700], 700), ([5000, 33, 1], 1)])
def test_pieces_of_a_row_of_tiles(lens, new, hq, hkv, d, monkeypatch):
    dag = dags.linear_chain(lens)
    st = dags.decode_segments_state(8100 + hq + new, [dag], [[len(lens) - 1]], hq, hkv, d, kv_scale=0.7, q_scale=0.7, new_tokens=[[new]])
    pd = B.PagedPrefillDesc(st["paged"], DEV)
    slots, nt_max = -(-pd.c.max_new // 64), -(-pd.c.max_ctx_pages // 4)
    small = 4 * (128 + 64 + slots * (17 + 8 * nt_max)) + 256
    assert nt_max >= 24 and B.dag_prefill_paged_workspace_bytes(pd) > small
    out, lse = _check(st, hq, hkv, d)
    monkeypatch.setattr(B, "dag_prefill_paged_workspace_bytes", lambda desc: small)
    out1, lse1 = _check(st, hq, hkv, d)
    # sums of the same bf16 probabilities, which a reference maximum of its own in every piece rounds anew (2^-9 each)
    assert (lse - lse1).abs().max() < 2 ** -9
    assert (out.float() - out1.float()).abs().max() < 2 ** -6 * out1.float().abs().max()


# more items of four heads than compute units: one head on 256 rows, two on 128
@pytest.mark.parametrize("hq,hkv,d", [(8, 8, 128), (16, 8, 128), (40, 8, 128), (8, 8, 64), (16, 8, 64)])
def test_items_of_fewer_heads(hq, hkv, d):
    dag_list = [_multilevel(12)] * 4
    assert 4 * 3 * 3 * hkv * -(-hq // hkv // 4) > 256
    st = dags.decode_segments_state(8200 + hq + d, dag_list, [[8, 6, 4]] * 4, hq, hkv, d, kv_scale=0.7, q_scale=0.7,
                                    new_tokens=[[150, 64, 1], [130, 223, 12], [1, 65, 12], [153, 84, 7]])
    _check(st, hq, hkv, d)
