"""GPU parity of the bf16 prefill on query chunks (rows cut at the borders of groups of siblings, keys
streamed in the order of the node's visible tokens), and static checks of its generated code."""
import os

import numpy as np
import pytest
import torch

from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, build_meta, check_close, oracle_prefill, run_prefill
from tests.test_asm_lds_reads import HIPCC, _assembly, _conflicts_of_kernel, _kernels


def _check(dag_list, hq, hkv, d, seed):
    T = int(sum(int(np.sum(L)) for L, _ in dag_list))
    q, k, v = dags.make_qkv(seed, T, hq, hkv, d, 0.5, torch.bfloat16)
    out, lse, _, _, _ = run_prefill(dag_list, q, k, v, 5e5, want_lse=True)
    ref, ref_lse, _ = oracle_prefill(dag_list, q, k, v, 5e5)
    check_close(out, ref, torch.bfloat16, "out")
    assert np.abs(lse.cpu().double().numpy() - ref_lse).max() < 2e-2


# every head split: items of four heads, pairs, single heads (the one- and two-head items of batches that leave compute
# units idle: tests/test_gpu_prefill_routes.py)
@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 128), (2, 1, 128), (1, 1, 128), (7, 1, 128), (10, 2, 128),
                                      (4, 1, 64), (2, 1, 64), (1, 1, 64), (7, 1, 64), (12, 2, 64)])
def test_chunks_every_head_split(hq, hkv, d):
    rng = np.random.Generator(np.random.PCG64(8800 + hq + d))
    dag_list = [dags.fork_join(130, [40, 64, 3, 150, 63], 70),        # five siblings cut into chunks across their borders
                dags.fork_join(64, [64, 64], 64),                     # nothing but whole tiles
                dags.linear_chain([1]), dags.linear_chain([65, 190, 257]),
                dags.random_dag(rng, n_nodes=20, depth=5, len_lo=1, len_hi=80)[:2]]
    _check(dag_list, hq, hkv, d, 8900 + hq + d)


# the last node of one visibility word, and lists of runs over two words (alternating ancestors: one run per node)
@pytest.mark.gpu
@pytest.mark.parametrize("n_nodes", [63, 64, 65, 127, 128])
def test_chunks_many_nodes_and_runs(n_nodes):
    rng = np.random.Generator(np.random.PCG64(8700 + n_nodes))
    alternating = [[u for u in range(v) if u % 2 == v % 2] for v in range(n_nodes)]
    dag_list = [(np.asarray(rng.integers(4, 40, n_nodes), dtype=np.int32), dags.bits_from_sets(alternating)),
                dags.random_dag(rng, n_nodes=n_nodes, depth=6, len_lo=10, len_hi=40)[:2]]
    _check(dag_list, 4, 1, 128, 8600 + n_nodes)


# a prompt that starts at an offset: its positions are shifted in place, the mask stays what it was
@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 128), (3, 1, 64)])
def test_mask_does_not_depend_on_the_positions(hq, hkv, d):
    dag_list = [dags.fork_join(130, [40, 64, 33, 150, 63], 70), dags.linear_chain([65, 190])]
    T = int(sum(int(np.sum(L)) for L, _ in dag_list))
    q, k, v = (x.to(DEV) for x in dags.make_qkv(8500 + d, T, hq, hkv, d, 0.5, torch.bfloat16))
    dout = dags.make_qkv(8501 + d, T, hq, hkv, d, 1.0, torch.bfloat16)[0].to(DEV)
    results = []
    for shift in (0, 1000):
        _, meta = build_meta(dag_list, hq, hkv, d, torch.bfloat16)
        meta.t["pos_ids"] += shift
        meta.t["node_pos_start"] += shift // 2
        out, lse = torch.empty_like(q), torch.empty(T, hq, dtype=torch.float32, device=DEV)
        B.dag_attn_prefill(meta, q, k, v, out, lse)
        grads = [torch.empty_like(x) for x in (q, k, v)]
        B.dag_attn_prefill_bwd(meta, q, k, v, out, dout, lse, *grads)
        results.append([out, lse] + grads)
    for x, y in zip(*results):
        assert torch.equal(x, y)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_generated_code_of_the_chunk_kernels(tmp_path):
    seen = 0
    for name, lines in _kernels(_assembly("prefill_bf16", tmp_path), "k_prefill_nodes"):
        _, bad = _conflicts_of_kernel(lines)
        assert not bad, "%s: %s" % (name, bad[:3])
        assert not any("scratch_" in l for l in lines), name
        seen += 1
    assert seen == 9
