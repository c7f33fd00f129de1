"""GPU parity of the bf16 prefill and its backward on the routes that the rules of the dispatch choose between.  Every case
states its route and computes the rule on the host, so that a changed threshold cannot move it to
another kernel unnoticed."""
import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, build_meta, check_close, oracle_prefill, run_prefill
from tests.test_gpu_prefill_bwd import check_close as check_grad

pytestmark = pytest.mark.gpu


def _sizes(dag_list):
    return int(sum(int(np.sum(L)) for L, _ in dag_list)), sum(len(L) for L, _ in dag_list), max(a.shape[1] for _, a in dag_list)


def _on_chunks(dag_list, hq, hkv, d):
    T, n, words = _sizes(dag_list)
    return words <= 2 and T * hkv * 2 * d < 2 ** 32 and T >= (32 if d == 128 and hq // hkv % 2 else 16) * n


def _heads_per_item_of_a_small_batch(dag_list, hq, hkv, d):
    T, n, _ = _sizes(dag_list)
    items, g, units = (T // 64 + n) * hkv, hq // hkv, torch.cuda.get_device_properties(0).multi_processor_count
    return 0 if d == 64 and g < 3 else 1 if items * g <= units else 2 if items * ((g + 1) // 2) <= units else 0


def _check(dag_list, hq, hkv, d, seed, rows_per_seq=None):
    T = _sizes(dag_list)[0]
    q, k, v = dags.make_qkv(seed, T, hq, hkv, d, 0.5, torch.bfloat16)
    out, lse, _, _, _ = run_prefill(dag_list, q, k, v, 5e5, want_lse=True)
    ref, ref_lse, rows = oracle_prefill(dag_list, q, k, v, 5e5, rows_per_seq=rows_per_seq, seed=seed)
    check_close(out[rows], ref[rows], torch.bfloat16, "out")
    assert np.abs(lse.cpu().double().numpy()[rows] - ref_lse[rows]).max() < 2e-2


# the block map's tiles: three visibility words (with nodes of many tiles, so that rows have long runs of FULL tiles), then
# one and two words with short nodes beside a long one; four-head items, 256-row tiles, both
@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 128), (4, 4, 128), (4, 2, 128), (5, 1, 128), (6, 1, 128),
                                      (4, 1, 64), (2, 2, 64), (4, 2, 64), (5, 1, 64), (6, 1, 64)])
@pytest.mark.parametrize("n_nodes", [150, 100, 40])
def test_block_map_route(n_nodes, hq, hkv, d):
    rng = np.random.Generator(np.random.PCG64(5100 + n_nodes))
    L, anc = dags.random_dag(rng, n_nodes=n_nodes, depth=6, len_lo=1, len_hi=9)[:2]
    L[0] = 700 if n_nodes == 150 else 130
    if n_nodes == 150:
        L[[3, 40, 90]] = 400, 333, 250
    dag_list = [(L, anc), dags.fork_join(70, [3] * (n_nodes // 4), 9)]
    assert not _on_chunks(dag_list, hq, hkv, d)
    _check(dag_list, hq, hkv, d, 5200 + n_nodes + hq, rows_per_seq=200)


# query chunks: batches that leave compute units idle take one or two heads an item, the others the items of the head split
@pytest.mark.parametrize("copies,heads_per_item", [(1, 1), (6, 2), (40, 0)])
@pytest.mark.parametrize("hq,hkv,d", [(5, 1, 128), (8, 1, 128), (5, 1, 64), (8, 1, 64)])
def test_chunk_route(copies, heads_per_item, hq, hkv, d):
    dag_list = [dags.fork_join(130, [40, 64, 33], 50)] * copies
    assert _on_chunks(dag_list, hq, hkv, d)
    got = _heads_per_item_of_a_small_batch(dag_list, hq, hkv, d)
    assert got == heads_per_item
    _check(dag_list, hq, hkv, d, 5300 + copies + hq)


# gradients on the memory of the inputs they belong to, and dK on the forward's output: the tables of the query chunks,
# which are built in dK, have no place there
@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 128), (5, 1, 128), (2, 1, 64), (3, 1, 64)])
@pytest.mark.parametrize("where", ["inputs", "out"])
def test_backward_with_gradients_on_the_inputs(hq, hkv, d, where):
    dag_list = [dags.fork_join(130, [80, 64, 73, 150, 83], 70), dags.linear_chain([130, 190])]
    T, n, _ = _sizes(dag_list)
    assert T >= 64 * n   # (chunks where nothing overlaps)
    q, k, v = (x.to(DEV) for x in dags.make_qkv(5400 + hq, T, hq, hkv, d, 0.7, torch.bfloat16))
    dout = dags.make_qkv(5401 + hq, T, hq, hkv, d, 1.0, torch.bfloat16)[0].to(DEV)
    _, meta = build_meta(dag_list, hq, hkv, d, torch.bfloat16)
    out, lse = torch.empty_like(q), torch.empty(T, hq, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, q, k, v, out, lse)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    B.dag_attn_prefill_bwd(meta, q, k, v, out, dout, lse, dq, dk, dv)
    dq2, k2, v2 = torch.empty_like(q), k.clone(), v.clone()
    dk2 = out.flatten()[:k.numel()].view_as(k) if where == "out" else k2
    B.dag_attn_prefill_bwd(meta, q, k2, v2, out, dout, lse, dq2, dk2, v2)
    assert torch.equal(dk2, dk) and torch.equal(v2, dv)
    check_grad(dq2, dq.cpu().double().numpy(), torch.bfloat16, "dq")   # (other order of the keys)


def test_row_offsets_beyond_32_bits():
    """More than 4 GiB of K, and as many elements of Q: the row offsets of chunks and streams are 32-bit, the block
    map's tiles take the call.  The first and the last sequence, one KV head."""
    hq, hkv, d, n_seqs, n = 32, 16, 128, 640, 1650
    dag_list = [dags.linear_chain([1000, 650])] * n_seqs
    T = n_seqs * n
    assert T * hkv * 2 * d >= 2 ** 32 and T * hq * d >= 2 ** 32 and T * hq < 2 ** 31
    gen = torch.Generator(device=DEV).manual_seed(1)
    draw = lambda h: torch.empty((T, h, d), dtype=torch.bfloat16, device=DEV).normal_(0., 0.5, generator=gen)
    q, dout, k, v = draw(hq), draw(hq), draw(hkv), draw(hkv)
    _, meta = build_meta(dag_list, hq, hkv, d, torch.bfloat16)
    out, lse = torch.empty_like(q), torch.empty(T, hq, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, q, k, v, out, lse)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    B.dag_attn_prefill_bwd(meta, q, k, v, out, dout, lse, dq, dk, dv)
    torch.cuda.synchronize()
    f64 = lambda x, heads: x[:, heads].float().cpu().double().numpy()
    for t0, kv in ((0, 0), (T - n, hkv - 1)):
        sl, heads = slice(t0, t0 + n), slice(kv * 2, kv * 2 + 2)
        args = f64(q[sl], heads), f64(k[sl], slice(kv, kv + 1)), f64(v[sl], slice(kv, kv + 1))
        ref, _ = orc.attn_prefill(*args, *dag_list[0])
        check_close(out[sl][:, heads], ref, torch.bfloat16, "out")
        grads = orc.attn_prefill_bwd(*args, f64(dout[sl], heads), *dag_list[0])
        for name, g, h, r in (("dq", dq, heads, grads[0]), ("dk", dk, slice(kv, kv + 1), grads[1]), ("dv", dv, slice(kv, kv + 1), grads[2])):
            check_grad(g[sl][:, h], r, torch.bfloat16, name)
    del q, dout, k, v, out, dq, dk, dv, meta
    torch.cuda.empty_cache()
