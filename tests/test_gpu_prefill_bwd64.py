"""GPU parity of the pipelined backward kernels at head dimension 64, and of the masked tiles of
sequences with more than one visibility word per node at both head dimensions; static checks of the
generated code of the kernels for head dimension 64."""
import os

import numpy as np
import pytest
import torch

from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.test_asm_lds_reads import HIPCC, _assembly, _conflicts_of_kernel, _kernels, _run
from tests.test_gpu_prefill_bwd import _check_against_oracle, _forward_backward


def _ragged(rng):
    return [dags.fork_join(300, [100, 64, 37, 5], 70),                                # 1 to 9 query tiles, ragged ends
            dags.random_dag(rng, n_nodes=20, depth=4, len_lo=1, len_hi=60)[:2],
            dags.linear_chain([1]), dags.linear_chain([64]), dags.linear_chain([65, 190]),
            dags.fork_join(256, [64, 64], 64)]                                        # tile-aligned nodes: FULL tiles only


# one head on two query tiles; pairs of heads; both; more pairs than one workgroup takes
@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv", [(1, 1), (2, 1), (3, 1), (4, 2), (10, 2), (8, 1)])
def test_bwd_head_dim_64_head_groupings(hq, hkv):
    dag_list = _ragged(np.random.Generator(np.random.PCG64(6400 + hq)))
    inputs, grads = _forward_backward(dag_list, hq, hkv, 64, 6500 + hq)
    _check_against_oracle(dag_list, inputs, grads)


# nodes long enough for query chunks, lists of runs over one and two visibility words
@pytest.mark.gpu
@pytest.mark.parametrize("n_nodes,hq,hkv,d", [(20, 5, 1, 128), (64, 4, 1, 64), (65, 3, 1, 64), (100, 6, 1, 128), (128, 2, 1, 64)])
def test_bwd_on_chunks_and_streams(n_nodes, hq, hkv, d):
    rng = np.random.Generator(np.random.PCG64(6800 + n_nodes))
    alternating = [[u for u in range(v) if u % 2 == v % 2] for v in range(n_nodes)]
    dag_list = [(np.asarray(rng.integers(17, 30, n_nodes), dtype=np.int32), dags.bits_from_sets(alternating)),
                dags.random_dag(rng, n_nodes=n_nodes, depth=6, len_lo=10, len_hi=50)[:2],
                dags.fork_join(130, [40, 64, 3, 150, 63], 70)]
    inputs, grads = _forward_backward(dag_list, hq, hkv, d, 6900 + n_nodes)
    _check_against_oracle(dag_list, inputs, grads)


# a workspace without room for the tile lists of left-over heads is still taken
@pytest.mark.gpu
@pytest.mark.parametrize("hq,hkv", [(1, 1), (5, 1), (6, 2)])
def test_bwd_head_dim_64_without_tile_lists(hq, hkv, monkeypatch):
    dag_list = _ragged(np.random.Generator(np.random.PCG64(6450 + hq)))
    call = B.dag_attn_prefill_bwd

    def with_small_workspace(meta, q, *args, **kw):
        up = lambda n: -(-n // 256) * 256  # noqa: E731
        m = meta.sizes
        n = 2 * up(m.total_tokens * hq * 4) + 2 * up(m.total_ktiles * 4) + up(m.total_tokens * 8) + 256
        assert n < B.dag_prefill_bwd_workspace_bytes(meta, hq, hkv, 64)
        call(meta, q, *args, workspace=torch.empty(n, dtype=torch.uint8, device=q.device), **kw)

    monkeypatch.setattr(B, "dag_attn_prefill_bwd", with_small_workspace)
    inputs, grads = _forward_backward(dag_list, hq, hkv, 64, 6550 + hq)
    _check_against_oracle(dag_list, inputs, grads)


# 65 to 128 nodes keep two words per lane, more fetch the word they need
@pytest.mark.gpu
@pytest.mark.parametrize("n_nodes,hq,hkv,d", [(64, 2, 1, 64), (65, 2, 1, 64), (128, 3, 1, 64), (129, 2, 1, 64),
                                              (128, 5, 1, 128), (129, 4, 1, 128), (200, 1, 1, 128)])
def test_bwd_visibility_words(n_nodes, hq, hkv, d):
    rng = np.random.Generator(np.random.PCG64(6600 + n_nodes))
    dag_list = [dags.random_dag(rng, n_nodes=n_nodes, depth=7, len_lo=1, len_hi=6)[:2], dags.fork_join(90, [30] * 3, 20)]
    inputs, grads = _forward_backward(dag_list, hq, hkv, d, 6700 + n_nodes + hq)
    _check_against_oracle(dag_list, inputs, grads)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_generated_code_of_the_chunk_kernels(tmp_path):
    seen = 0
    for name, lines in _kernels(_assembly("prefill_bwd", tmp_path), "k_nodes"):
        _, bad = _conflicts_of_kernel(lines)
        assert not bad, "%s: %s" % (name, bad[:3])
        assert not any("scratch_" in l for l in lines), name
        seen += 1
    assert seen == 6


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_generated_code_of_the_head_dim_64_kernels(tmp_path):
    """No instruction touches a register whose LDS read may be in flight; a pipelined iteration (one
    without masks, one with) is one straight-line block: 16 row operands and 16 (dQ: 8) transposed
    ones of two reads each, in dK/dV also 8 groups of row data of two reads."""
    want = {"k_bwd64_dkv": ([64, 64], 32), "k_bwd64_dq": ([32, 32], 24)}
    seen = 0
    for name, lines in _kernels(_assembly("prefill_bwd", tmp_path), "k_bwd64_"):
        blocks, bad = _conflicts_of_kernel(lines)
        assert not bad, "%s: %s" % (name, bad[:3])
        assert not any("scratch_" in l for l in lines), name
        reads, mfmas = next(v for k, v in want.items() if k in name)
        found = []
        for b in blocks:
            if sum(1 for l in b["insts"] if l.startswith("v_mfma")) >= mfmas:
                assert not _run(b["insts"], [])[0], name
                found.append(sum(1 for l in b["insts"] if l.startswith("ds_read")))
        assert sorted(found) == reads, "%s: %s" % (name, found)
        seen += 1
    assert seen == 3
