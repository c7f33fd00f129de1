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


def _check(st, hq, hkv, d, rows=slice(None)):
    out, lse = _gpu_prefill_paged(st, hq, hkv, d, want_lse=True)
    ref = orc.attn_decode_segments(st["desc"], dags.to_f64(st["q"]), dags.to_f64(st["k_pool"]), dags.to_f64(st["v_pool"]),
                                   branches=range(st["q"].shape[0])[rows] if isinstance(rows, slice) else rows)
    check_close(out[rows], ref[rows], torch.bfloat16, "paged prefill out")
    assert torch.isfinite(lse).all()
    return out, lse


# contexts just long enough for pieces, of many pieces, pieces of masked tiles alone (77 new tokens behind full pages), and
# a workspace without room for them: the same row sums, from one piece
@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 128), (5, 1, 64), (2, 2, 128), (8, 1, 64)])
@pytest.mark.parametrize("lens,new", [([1470, 80], 77), ([1472, 64], 64), ([3000, 700], 700), ([5000, 33, 1], 1)])
def test_pieces_of_a_row_of_tiles(lens, new, hq, hkv, d, monkeypatch):
    dag = dags.linear_chain(lens)
    st = dags.decode_segments_state(8100 + hq + new, [dag], [[len(lens) - 1]], hq, hkv, d, kv_scale=0.7, q_scale=0.7, new_tokens=[[new]])
    _check_pieces(st, hq, hkv, d, monkeypatch)


# more items of four heads than compute units, so few of one head on 256 rows that these are cut: two and three pieces, nodes that
# end inside a wave's 32 rows, the last rows of a node by themselves, contexts of different lengths.  (Items of two heads are at
# least half as many as those of four, more than half of the compute units: they are never cut.)
@pytest.mark.parametrize("hq,hkv,d,new", [(8, 8, 128, [300, 290, 300, 257, 300, 31, 300, 1]), (8, 8, 64, [300, 290, 300, 257, 300, 31, 300, 1]),
                                          (8, 8, 128, [700, 513, 650]), (16, 16, 64, [256, 256, 130, 1, 256])])
def test_pieces_of_items_of_one_head(hq, hkv, d, new, monkeypatch):
    dag_list = [dags.linear_chain([1500 + 37 * i, n + 5]) for i, n in enumerate(new)]
    st = dags.decode_segments_state(8150 + hq + len(new), dag_list, [[1]] * len(new), hq, hkv, d, kv_scale=0.7, q_scale=0.7,
                                    new_tokens=[[n] for n in new])
    items = lambda rows: len(new) * -(-max(new) // rows) * hkv  # noqa: E731
    assert items(64) > 256 and items(256) <= 128
    first = np.cumsum([0] + new)
    rows = np.concatenate([first[:-1], first[1:] - 1, [255, 256, 31, 32, 127, 128], np.random.default_rng(hq).integers(0, first[-1], 40)])
    _check_pieces(st, hq, hkv, d, monkeypatch, np.unique(rows))  # (against the oracle; the two runs are compared whole)


def _check_pieces(st, hq, hkv, d, monkeypatch, rows=slice(None)):
    pd = B.PagedPrefillDesc(st["paged"], DEV)
    slots, nt_max = pd.c.n_nodes * -(-pd.c.max_new // 64), -(-pd.c.max_ctx_pages // 4)
    small = 4 * (128 + 64 + slots * (17 + 8 * nt_max)) + 256
    assert nt_max >= 24 and B.dag_prefill_paged_workspace_bytes(pd) > small
    out, lse = _check(st, hq, hkv, d, rows)
    monkeypatch.setattr(B, "dag_prefill_paged_workspace_bytes", lambda desc: small)
    out1, lse1 = _check(st, hq, hkv, d, rows)
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
