"""GPU parity of the bf16 prefill whose items hold all heads of a group (row-major pairs of rows and heads), and static checks of its
generated code.  The batches are so large that none takes the one- and two-head items of small ones."""
import os

import numpy as np
import pytest
import torch

from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, build_meta, check_close, launched_kernels, oracle_prefill, run_prefill
from tests.test_asm_lds_reads import HIPCC, _assembly, _conflicts_of_kernel, _kernels
from tests.test_gpu_prefill_routes import _heads_per_item_of_a_small_batch, _on_chunks, _sizes


def _packed(dag_list, hq, hkv, d):
    g = hq // hkv
    return _on_chunks(dag_list, hq, hkv, d) and _heads_per_item_of_a_small_batch(dag_list, hq, hkv, d) == 0 and g not in ((1, 2) if d == 64 else (1, 2, 4))


def _check(dag_list, hq, hkv, d, seed, rows_per_seq):
    q, k, v = dags.make_qkv(seed, _sizes(dag_list)[0], hq, hkv, d, 0.5, torch.bfloat16)
    out, lse, _, _, _ = run_prefill(dag_list, q, k, v, 5e5, want_lse=True)
    ref, ref_lse, rows = oracle_prefill(dag_list, q, k, v, 5e5, rows_per_seq=rows_per_seq, seed=seed)
    check_close(out[rows], ref[rows], torch.bfloat16, "out")
    assert np.abs(lse.cpu().double().numpy()[rows] - ref_lse[rows]).max() < 2e-2


# groups of 3 to 8 heads (85 to 16 rows a chunk, with pairs that belong to no row), more than eight divided evenly and with a
# head to spare (9 = 5 + 4, 11 = 6 + 5, 17 = 3 x 6 - 1), four at head dimension 64
@pytest.mark.gpu
@pytest.mark.parametrize("g", [3, 4, 5, 6, 7, 8, 9, 11, 16, 17])
@pytest.mark.parametrize("d", [64, 128])
def test_every_group(g, d):
    hkv = 2
    rng = np.random.Generator(np.random.PCG64(9100 + g))
    dag_list = [dags.fork_join(130, [40, 64, 3, 150, 63], 70), dags.linear_chain([1]), dags.linear_chain([65, 190, 257]),
                dags.random_dag(rng, n_nodes=100, depth=6, len_lo=10, len_hi=80)[:2]] * 4
    assert _packed(dag_list, g * hkv, hkv, d) == (g != 4 or d == 64)
    _check(dag_list, g * hkv, hkv, d, 9200 + g + d, 80)


# contexts of 16,384 tokens and more, and twelve items of four heads for every compute unit: heads of dimension 64 in fours on 64 rows
@pytest.mark.gpu
@pytest.mark.parametrize("tokens,four", [(16300, False), (24600, True)])
def test_long_contexts_of_small_heads(tokens, four):
    hq, hkv, d = 32, 8, 64
    dag_list = [dags.fork_join(tokens - 700, [200, 150, 250], 100)]
    T = _sizes(dag_list)[0]
    units = torch.cuda.get_device_properties(0).multi_processor_count
    assert _packed(dag_list, hq, hkv, d) and (T >= 16384 and T // 64 * hkv >= 12 * units) == four
    _check(dag_list, hq, hkv, d, 9300 + tokens, 40)


# a workspace prepared for a group that packs other heads, or none: the table is built again where it is of other rows
@pytest.mark.gpu
@pytest.mark.parametrize("order", [(5, 6, 5), (4, 8, 3), (8, 16, 8), (7, 1, 7)])
@pytest.mark.parametrize("d", [64, 128])
def test_prepared_for_another_group(order, d):
    hkv = 2
    dag_list = [dags.fork_join(130, [40, 64, 33, 150, 63], 70)] * 30
    T = _sizes(dag_list)[0]
    first, rest = order[0], order[1:]
    _, meta = build_meta(dag_list, first * hkv, hkv, d, torch.bfloat16)
    v = dags.make_qkv(9400, T, hkv, hkv, d, 0.5, torch.bfloat16)[2].to(DEV)
    ws = torch.zeros(B.dag_prefill_workspace_bytes(meta, hkv, d, B.DAG_BF16), dtype=torch.uint8, device=DEV)
    B.dag_prefill_prepare_v(meta, v, first * hkv, workspace=ws)
    for g in rest + rest:
        q, k, _ = (x.to(DEV) for x in dags.make_qkv(9410 + g, T, g * hkv, hkv, d, 0.5, torch.bfloat16))
        ref, out = torch.empty_like(q), torch.empty_like(q)
        B.dag_attn_prefill(meta, q, k, v, ref)
        B.dag_attn_prefill(meta, q, k, v, out, workspace=ws, prepared=True)
        assert torch.equal(out, ref)


# few nodes and slots: the tables come from the kernel that keeps their counts and descriptors in LDS, so that nothing but the ordered
# table is in the workspace.  The same group, twice, another one in between, and behind a combined call.
@pytest.mark.gpu
@pytest.mark.parametrize("g,other,d", [(5, 8, 128), (8, 3, 128), (3, 5, 128), (6, 7, 128), (4, 8, 64), (5, 3, 64), (8, 4, 64)])
@pytest.mark.parametrize("lengths", [[700, 200, 150, 256, 188, 170], [400, 64, 90, 130, 150, 33, 256, 120, 75, 80, 100, 166]])
def test_prepared_for_few_nodes(g, other, d, lengths):
    hkv = 8
    dag_list = [dags.fork_join(lengths[0], lengths[1:-1], lengths[-1])]
    T, nodes = _sizes(dag_list)[:2]
    assert T == 1664 and nodes == len(lengths) <= 64
    _, meta = build_meta(dag_list, hkv, hkv, d, torch.bfloat16)
    v = dags.make_qkv(9420, T, hkv, hkv, d, 0.5, torch.bfloat16)[2].to(DEV)
    calls = {}
    for x in (g, other):
        assert _packed(dag_list, x * hkv, hkv, d) and T // ((256 if d == 128 else 128) // x) + nodes <= 128
        q, k, _ = (t.to(DEV) for t in dags.make_qkv(9421 + x, T, x * hkv, hkv, d, 0.5, torch.bfloat16))
        ref = torch.empty_like(q)
        B.dag_attn_prefill(meta, q, k, v, ref)
        calls[x] = q, k, ref
    ws = torch.ones(B.dag_prefill_workspace_bytes(meta, hkv, d, B.DAG_BF16), dtype=torch.uint8, device=DEV)

    def prepared(x):
        q, k, ref = calls[x]
        out = torch.zeros_like(q)
        B.dag_attn_prefill(meta, q, k, v, out, workspace=ws, prepared=True)
        assert torch.equal(out, ref)

    B.dag_prefill_prepare_v(meta, v, g * hkv, workspace=ws)
    for x in (g, g, other, other, g):
        prepared(x)
    ws.fill_(1)
    B.dag_attn_prefill(meta, calls[g][0], calls[g][1], v, torch.empty_like(calls[g][0]), workspace=ws)
    for x in (g, g, other):
        prepared(x)


# a prepared call is the attention kernel, with packed heads behind a look at their table
@pytest.mark.gpu
@pytest.mark.parametrize("g,d,copies", [(5, 128, 30), (8, 128, 4), (4, 64, 30), (4, 128, 30), (2, 64, 30), (5, 128, 1)])
def test_launches_of_a_prepared_call(g, d, copies):
    hkv = 2
    dag_list = [dags.fork_join(130, [40, 64, 33, 150, 63], 70)] * copies
    q, k, v = (t.to(DEV) for t in dags.make_qkv(9430, _sizes(dag_list)[0], g * hkv, hkv, d, 0.5, torch.bfloat16))
    _, meta = build_meta(dag_list, g * hkv, hkv, d, torch.bfloat16)
    ws = torch.zeros(B.dag_prefill_workspace_bytes(meta, hkv, d, B.DAG_BF16), dtype=torch.uint8, device=DEV)
    B.dag_prefill_prepare_v(meta, v, g * hkv, workspace=ws)
    out = torch.empty_like(q)
    names = launched_kernels(lambda: B.dag_attn_prefill(meta, q, k, v, out, workspace=ws, prepared=True))
    want = ["k_pack_tables", "k_prefill_packed"] if _packed(dag_list, g * hkv, hkv, d) else ["k_prefill_nodes"]
    assert len(names) == len(want) and all(w in n for w, n in zip(want, names)), names


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_generated_code_of_the_packed_kernels(tmp_path):
    seen = 0
    for name, lines in _kernels(_assembly("prefill_bf16", tmp_path), "k_prefill_packed"):
        _, bad = _conflicts_of_kernel(lines)
        assert not bad, "%s: %s" % (name, bad[:3])
        assert not any("scratch_" in l for l in lines), name
        seen += 1
    assert seen >= 2
