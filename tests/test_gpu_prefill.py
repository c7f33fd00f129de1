"""GPU parity: dag_attn_prefill (through the C ABI) against the fp64 oracle, element by element."""
import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, check_close, oracle_prefill, run_prefill

pytestmark = pytest.mark.gpu


def _run_and_check(dag_list, hq, hkv, d, dtype, scale, theta, seed, rows_per_seq=None, want_lse=True):
    T = int(sum(int(np.sum(L)) for L, _ in dag_list))
    q, k, v = dags.make_qkv(seed, T, hq, hkv, d, scale, dtype)
    out, lse, meta, _, _ = run_prefill(dag_list, q, k, v, theta, want_lse=want_lse)
    ref, ref_lse, rows = oracle_prefill(dag_list, q, k, v, theta, rows_per_seq=rows_per_seq, seed=seed)
    res = check_close(out[rows], ref[rows], dtype, "prefill out")
    if want_lse:
        l = lse.cpu().double().numpy()[rows]
        assert np.abs(l - ref_lse[rows]).max() < (1e-4 if dtype == torch.float32 else 2e-2)
    return res


def test_config1_tiny_fork_join_fp32():
    c = dags.config(0)
    dag_list = dags.config_dags(c)
    max_abs, rel = _run_and_check(dag_list, c["hq"], c["hkv"], c["d"], torch.float32, c["scale"], c["theta"], c["seed"])
    assert max_abs < 1e-4


@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 128), (8, 2, 64), (5, 1, 128), (2, 1, 128), (6, 3, 64),
                                      (3, 3, 128), (1, 1, 64), (8, 1, 128), (5, 1, 64), (3, 1, 128), (6, 1, 64),
                                      (14, 2, 128)])
def test_bf16_small_dags_every_kernel_variant(hq, hkv, d):
    rng = np.random.Generator(np.random.PCG64(1000 + hq * 10 + d))
    dag_list = [dags.fork_join(100, [37, 64, 5], 70),               # ragged everywhere
                dags.random_dag(rng, n_nodes=14, depth=4, len_lo=1, len_hi=45)[:2],
                dags.linear_chain([1]),
                dags.linear_chain([200])]
    _run_and_check(dag_list, hq, hkv, d, torch.bfloat16, 0.5, 5e5, 2000 + hq + d)


def test_fp32_ragged_and_gqa_and_d128():
    rng = np.random.Generator(np.random.PCG64(9))
    dag_list = [dags.fork_join(70, [33, 64], 31), dags.random_dag(rng, n_nodes=10, depth=4, len_lo=1, len_hi=30)[:2]]
    _run_and_check(dag_list, 4, 2, 128, torch.float32, 1.0, 1e4, 31)
    _run_and_check(dag_list, 3, 1, 64, torch.float32, 1.0, 1e4, 32)


def test_bf16_more_than_64_nodes():
    rng = np.random.Generator(np.random.PCG64(78))
    L, anc, _, _ = dags.random_dag(rng, n_nodes=90, depth=6, len_lo=1, len_hi=12)
    _run_and_check([(L, anc)], 4, 1, 128, torch.bfloat16, 0.5, 5e5, 33)


def test_bf16_linear_chain_is_causal_attention_of_the_library_kind():
    # independent of the oracle: compare with torch's fp32 SDPA on the GPU-rotated inputs
    dag_list = [dags.linear_chain([50, 150, 56])]
    q, k, v = dags.make_qkv(41, 256, 8, 2, 128, 0.5, torch.bfloat16)
    out, _, _, qd, kd = run_prefill(dag_list, q, k, v, 5e5)
    qf = qd.float().permute(1, 0, 2)[None].cpu()
    kf = kd.float().permute(1, 0, 2)[None].repeat_interleave(4, dim=1).cpu()
    vf = v.float().permute(1, 0, 2)[None].repeat_interleave(4, dim=1)
    ref = torch.nn.functional.scaled_dot_product_attention(qf, kf, vf, is_causal=True)[0].permute(1, 0, 2)
    check_close(out, ref.double().numpy(), torch.bfloat16, "vs sdpa")


def test_config2_llama_shape_full_size_sampled_rows():
    c = dags.config(1)
    dag_list = dags.config_dags(c)
    _run_and_check(dag_list, c["hq"], c["hkv"], c["d"], torch.bfloat16, c["scale"], c["theta"], c["seed"],
                   rows_per_seq=96)


def test_config4_random_multilevel_full_size_sampled_rows():
    c = dags.config(3)
    dag_list = dags.config_dags(c)
    _run_and_check(dag_list, c["hq"], c["hkv"], c["d"], torch.bfloat16, c["scale"], c["theta"], c["seed"],
                   rows_per_seq=64)


@pytest.mark.parametrize("hq,hkv,d", [(5, 1, 128), (6, 1, 128), (2, 2, 64), (9, 1, 64)])
def test_left_over_heads_on_256_row_tiles_ragged_multilevel_dags(hq, hkv, d):
    """Head groups of 5, 6, 1 and 9 (one or two heads beside the four-head items, or alone) on
    sequences of 1 to 19 query tiles whose lengths leave a ragged 256-row tile; sampled rows of every
    sequence and every head.  The group of 5 runs on the block map's tiles, the rows of its
    256-row tiles over the key tiles derived from the 64 x 64 block map on the device (mixed SKIP / FULL
    / PARTIAL quartets, fully hidden 32-row blocks inside a visited tile); the others run on query chunks
    (tests/test_gpu_prefill_routes.py has every group on either route)."""
    rng = np.random.Generator(np.random.PCG64(4000 + hq + d))
    dag_list = [dags.random_dag(rng, n_nodes=40, depth=5, len_lo=1, len_hi=60)[:2],
                dags.fork_join(517, [64, 190, 3], 131),
                dags.linear_chain([1]),
                dags.random_dag(rng, n_nodes=70, depth=6, len_lo=3, len_hi=30)[:2],   # two visibility words
                dags.linear_chain([255]), dags.linear_chain([257])]
    _run_and_check(dag_list, hq, hkv, d, torch.bfloat16, 0.5, 5e5, 4100 + hq + d, rows_per_seq=80)


def test_config5_head_shape_reduced_length_sampled_rows():
    """Benchmark config 5's head configuration (40 query / 8 KV heads, G = 5) on its DAG shape at an
    eighth of the length (2 x 6272 tokens: prefix 4096 -> 32 branches x 64 -> join 128): both
    launches of the head split at many tiles per row."""
    c = dags.config(4)
    dag_list = [dags.fork_join(4096, [64] * 32, 128)] * 2
    _run_and_check(dag_list, c["hq"], c["hkv"], c["d"], torch.bfloat16, c["scale"], c["theta"], c["seed"] + 9,
                   rows_per_seq=48)


def test_config2_one_sequence_every_row_of_one_kv_group():
    c = dags.config(1)
    dag_list = dags.config_dags(c)[:1]
    T = 4608
    q, k, v = dags.make_qkv(c["seed"] + 100, T, c["hq"], c["hkv"], c["d"], c["scale"], torch.bfloat16)
    out, _, _, _, _ = run_prefill(dag_list, q, k, v, c["theta"])
    heads = [4, 5, 6, 7]
    ref, _, _ = oracle_prefill(dag_list, q, k, v, c["theta"], heads=heads)
    check_close(out[:, heads], ref[:, heads], torch.bfloat16, "config2 all rows, kv group 1")


def test_prefill_is_deterministic_run_to_run():
    dag_list = [dags.fork_join(300, [100, 90], 50)]
    q, k, v = dags.make_qkv(51, 540, 8, 2, 128, 0.5, torch.bfloat16)
    o1, _, _, _, _ = run_prefill(dag_list, q, k, v, 5e5)
    o2, _, _, _, _ = run_prefill(dag_list, q, k, v, 5e5)
    assert torch.equal(o1, o2)


def test_prepare_v_then_prepared_attention_equals_the_combined_call():
    """The two halves of dag_attn_prefill, launched separately, give the bits the combined call
    gives (and therefore the oracle's values), with a caller-provided workspace."""
    from tests.gpu_util import build_meta
    dag_list = [dags.fork_join(130, [70, 33], 40), dags.linear_chain([77])]
    T = int(sum(int(np.sum(L)) for L, _ in dag_list))
    q, k, v = dags.make_qkv(77, T, 8, 2, 128, 0.5, torch.bfloat16)
    _, meta = build_meta(dag_list, 8, 2, 128, torch.bfloat16)
    qd, kd, vd = q.to(DEV).clone(), k.to(DEV).clone(), v.to(DEV)
    B.dag_rope_qk(meta.get("pos_ids"), qd, kd, 5e5)
    o1, o2 = torch.empty_like(qd), torch.zeros_like(qd)
    B.dag_attn_prefill(meta, qd, kd, vd, o1)
    ws = torch.zeros(B.dag_prefill_workspace_bytes(meta, 2, 128, B.DAG_BF16), dtype=torch.uint8, device=DEV)
    B.dag_prefill_prepare_v(meta, vd, 8, workspace=ws)
    B.dag_attn_prefill(meta, qd, kd, vd, o2, workspace=ws, prepared=True)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2)
    ref, _, rows = oracle_prefill(dag_list, q, k, v, 5e5)
    check_close(o2[rows], ref[rows], torch.bfloat16, "prepared prefill")


def test_repeated_launches_on_one_workspace_hand_out_every_item_once():
    """The attention kernel hands its work items out through counters in the workspace and leaves
    them zeroed: three launches in a row after one prepare_v (more items than compute units, so
    the counters are really used) all give the bits of the first one, which match the oracle; a
    workspace filled with ones beforehand shows that prepare_v is what zeroes the counters."""
    from tests.gpu_util import build_meta
    dag_list = [dags.fork_join(1024, [256] * 6, 320), dags.fork_join(700, [130, 260, 90], 200)]
    T = int(sum(int(np.sum(L)) for L, _ in dag_list))
    hq, hkv, d = 32, 8, 128
    q, k, v = dags.make_qkv(91, T, hq, hkv, d, 0.5, torch.bfloat16)
    _, meta = build_meta(dag_list, hq, hkv, d, torch.bfloat16)
    n_items = meta.sizes.total_qtiles * hkv
    assert n_items > 2 * torch.cuda.get_device_properties(0).multi_processor_count
    qd, kd, vd = q.to(DEV).clone(), k.to(DEV).clone(), v.to(DEV)
    B.dag_rope_qk(meta.get("pos_ids"), qd, kd, 5e5)
    ws = torch.full((B.dag_prefill_workspace_bytes(meta, hkv, d, B.DAG_BF16),), 1, dtype=torch.uint8, device=DEV)
    B.dag_prefill_prepare_v(meta, vd, hq, workspace=ws)
    outs = [torch.zeros_like(qd) for _ in range(3)]
    for o in outs:
        B.dag_attn_prefill(meta, qd, kd, vd, o, workspace=ws, prepared=True)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    ref, _, rows = oracle_prefill(dag_list, q, k, v, 5e5, rows_per_seq=96, seed=5)
    check_close(outs[2][rows], ref[rows], torch.bfloat16, "repeated prepared prefill")


def test_config5_qwen_shape_full_size_sampled_rows():
    """Benchmark config 5 prefill at full size (2 x 50,176 tokens, 40 query heads in groups of 5):
    sampled rows against the oracle, which gets only those query rows (compact mode)."""
    c = dags.config(4)
    dag_list = dags.config_dags(c)
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    T = int(sum(int(np.sum(L)) for L, _ in dag_list))
    q, k, v = dags.make_qkv(c["seed"], T, hq, hkv, d, c["scale"], torch.bfloat16)
    out, _, meta, _, _ = run_prefill(dag_list, q, k, v, c["theta"])
    assert int(meta.get("useful_pairs").sum().item()) == 2 * 1128817152
    rng = np.random.Generator(np.random.PCG64(c["seed"]))
    t0 = 0
    for L, anc in dag_list:
        Tb = int(np.sum(L))
        _, pos = orc.token_meta(L, anc)
        # first / last rows, the rows around the fork and the join, and a seeded sample
        edges = [0, 1, 32767, 32768, 32768 + 511, 32768 + 512, 32768 + 32 * 512 - 1, 32768 + 32 * 512, Tb - 1]
        rows = np.unique(np.concatenate([edges, rng.choice(Tb, size=16, replace=False)]))
        ks = orc.rope(dags.to_f64(k[t0:t0 + Tb]), pos, c["theta"])
        qs = orc.rope(dags.to_f64(q[t0:t0 + Tb][rows]), pos[rows], c["theta"])
        ref, _ = orc.attn_prefill(qs, ks, dags.to_f64(v[t0:t0 + Tb]), L, anc, rows=rows, compact=True)
        check_close(out[t0 + rows], ref, torch.bfloat16, "config 5 prefill")
        t0 += Tb
    # whole tiles of the first sequence inside the branches: the 256 rows of one
    # tile of the left-over heads (the fifth head of two KV groups), the 64 rows of one tile of a four-head item
    L, anc = dag_list[0]
    Tb = int(np.sum(L))
    _, pos = orc.token_meta(L, anc)
    ks = orc.rope(dags.to_f64(k[:Tb]), pos, c["theta"])
    for first, n_rows, heads in ((32768 + 3 * 512 - 256, 256, [4, 39]), (32768 + 9 * 512, 64, [10, 11, 12, 13])):
        rows = np.arange(first, first + n_rows)
        qs = orc.rope(dags.to_f64(q[:Tb][rows]), pos[rows], c["theta"])
        ref, _ = orc.attn_prefill(qs, ks, dags.to_f64(v[:Tb]), L, anc, rows=rows, heads=heads, compact=True)
        check_close(out[rows][:, heads], ref[:, heads], torch.bfloat16, "config 5 prefill, whole tile at row %d" % first)


def test_config4_one_sequence_every_row_of_one_kv_group():
    """Benchmark config 4 (random multi-level DAGs, half of the visited tiles PARTIAL): the whole
    batch runs on the GPU; every row of one sequence, the four query heads of one KV group,
    against the oracle."""
    c = dags.config(3)
    dag_list = dags.config_dags(c)
    T = int(sum(int(np.sum(L)) for L, _ in dag_list))
    q, k, v = dags.make_qkv(c["seed"] + 200, T, c["hq"], c["hkv"], c["d"], c["scale"], torch.bfloat16)
    out, lse, meta, _, _ = run_prefill(dag_list, q, k, v, c["theta"], want_lse=True)
    t0 = int(sum(int(np.sum(L)) for L, _ in dag_list[:5]))
    L, anc = dag_list[5]
    Tb = int(np.sum(L))
    heads = [8, 9, 10, 11]
    sl = slice(t0, t0 + Tb)
    ref, ref_lse, _ = oracle_prefill([(L, anc)], q[sl], k[sl], v[sl], c["theta"], heads=heads)
    check_close(out[sl][:, heads], ref[:, heads], torch.bfloat16, "config 4, sequence 5, kv group 2")
    assert np.abs(lse[sl][:, heads].cpu().double().numpy() - ref_lse[:, heads]).max() < 2e-2


def test_bf16_two_visibility_words_many_tiles():
    """More than 64 nodes (two visibility words per node) at several thousand tokens, on query chunks with lists of
    runs over two words (the block map's tiles with two and three words: tests/test_gpu_prefill_routes.py)."""
    rng = np.random.Generator(np.random.PCG64(177))
    L, anc, _, _ = dags.random_dag(rng, n_nodes=100, depth=7, len_lo=16, len_hi=80)
    assert anc.shape[1] == 2 and int(np.sum(L)) >= 4000
    _run_and_check([(L, anc), dags.fork_join(300, [70, 41], 90)], 8, 2, 128, torch.bfloat16, 0.5, 5e5, 178)
