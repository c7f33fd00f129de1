"""GPU: what Eq. 3 hides from a row does not reach it, also where it is Inf or NaN and shares a key tile with
what the row sees.  The rows that do not see such a token are compared with the oracle on clean inputs; the
rows that see one are not numbers."""
import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, TOL, build_meta, oracle_prefill

pytestmark = pytest.mark.gpu


def _batch(seed):
    """Siblings that share key tiles, nodes that start and end inside a tile, rows in front of a bad token of their
    own node; and the bad tokens: a whole branch, single tokens, the last token of a sequence."""
    rng = np.random.Generator(np.random.PCG64(seed))
    dag_list = [dags.fork_join(64, [32, 32, 32, 32], 40), dags.fork_join(130, [40, 64, 33, 150, 63], 70),
                dags.random_dag(rng, n_nodes=24, depth=5, len_lo=20, len_hi=90)[:2], dags.linear_chain([200, 77])]
    at = np.cumsum([0] + [int(np.sum(L)) for L, _ in dag_list])
    bad = list(range(64, 96)) + [at[0] + 64 + 32 + 17]                 # first branch of the first sequence, a token of the second
    bad += [at[1] + 130 + 40 + 63, at[1] + 130 + 40 + 64 + 5]          # two branches of the second
    bad += [at[2] + int(np.sum(dag_list[2][0])) // 2, at[3] + 150, at[4] - 1]
    return dag_list, np.asarray(bad), int(at[-1])


def _sees_bad(dag_list, bad, T):
    out, t0 = np.zeros(T, dtype=bool), 0
    for L, anc in dag_list:
        Tb = int(np.sum(L))
        here = bad[(bad >= t0) & (bad < t0 + Tb)] - t0
        out[t0:t0 + Tb] = orc.explicit_mask(L, anc)[:, here].any(axis=1)
        t0 += Tb
    return out


def _spoil(v, bad):
    v = v.clone()
    for x, t in enumerate(bad):
        v[t] = (float("nan"), float("inf"), float("-inf"))[x % 3]
    return v


def _check(got, ref, rows, tol):
    g, r = got.cpu().double().numpy()[rows], ref[rows]
    assert np.isfinite(g).all(), "%d rows lost" % int((~np.isfinite(g)).reshape(len(g), -1).any(axis=1).sum())
    scale = max(1.0, float(np.abs(r).max()))
    assert np.abs(g - r).max() <= tol[0] * scale and np.linalg.norm(g - r) <= tol[1] * np.linalg.norm(r)


# fp32: both cuts of the work; bf16: every launch shape on query chunks (nodes of 16 tokens and more)
@pytest.mark.parametrize("hq,hkv,d,dtype", [(2, 1, 64, torch.float32), (3, 1, 128, torch.float32), (24, 2, 64, torch.float32),
                                            (24, 4, 128, torch.float32), (4, 1, 128, torch.bfloat16), (7, 1, 128, torch.bfloat16),
                                            (56, 8, 128, torch.bfloat16), (7, 1, 64, torch.bfloat16), (56, 8, 64, torch.bfloat16)])
def test_hidden_values(hq, hkv, d, dtype):
    dag_list, bad, T = _batch(hq + d)
    q, k, v = dags.make_qkv(60 + hq, T, hq, hkv, d, 0.5 if dtype == torch.bfloat16 else 1.0, dtype)
    ref, ref_lse, _ = oracle_prefill(dag_list, q, k, v, 1e4)
    _, meta = build_meta(dag_list, hq, hkv, d, dtype)
    qd, kd, vd = q.to(DEV).clone(), k.to(DEV).clone(), _spoil(v, bad).to(DEV)
    B.dag_rope_qk(meta.get("pos_ids"), qd, kd, 1e4)
    out, lse = torch.empty_like(qd), torch.empty(T, hq, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, qd, kd, vd, out, lse)
    sees = _sees_bad(dag_list, bad, T)
    assert not torch.isfinite(out[torch.from_numpy(sees).to(DEV)].float()).any(dim=-1).any()
    _check(out, ref, ~sees, TOL[dtype])
    assert np.abs(lse.cpu().double().numpy() - ref_lse).max() < (1e-4 if dtype == torch.float32 else 2e-2)


# dQ with one and two visibility words, on query chunks (first two) and on the block map's tiles (shorter nodes)
@pytest.mark.parametrize("hq,hkv,d,n_nodes,longest", [(2, 1, 64, 24, 90), (4, 1, 128, 70, 60), (3, 1, 64, 40, 14), (4, 1, 128, 100, 14)])
def test_hidden_values_backward_dq(hq, hkv, d, n_nodes, longest):
    rng = np.random.Generator(np.random.PCG64(700 + n_nodes))
    dag_list = [dags.random_dag(rng, n_nodes=n_nodes, depth=5, len_lo=longest // 2, len_hi=longest)[:2]]
    T = int(np.sum(dag_list[0][0]))
    bad = np.asarray([T // 3, T // 2, T - 1])
    q, k, v = dags.make_qkv(80 + hq, T, hq, hkv, d, 0.7, torch.bfloat16)
    dout = dags.make_qkv(81 + hq, T, hq, hkv, d, 1.0, torch.bfloat16)[0]
    _, meta = build_meta(dag_list, hq, hkv, d, torch.bfloat16)
    qd, kd, dod = q.to(DEV), k.to(DEV), dout.to(DEV)
    vd = v.to(DEV)
    out, lse = torch.empty_like(qd), torch.empty(T, hq, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, qd, kd, vd, out, lse)
    dq, dk, dv = torch.empty_like(qd), torch.empty_like(kd), torch.empty_like(kd)
    B.dag_attn_prefill_bwd(meta, qd, kd, _spoil(v, bad).to(DEV), out, dod, lse, dq, dk, dv)
    ref = orc.attn_prefill_bwd(dags.to_f64(q), dags.to_f64(k), dags.to_f64(v), dags.to_f64(dout), *dag_list[0])[0]
    _check(dq, ref, ~_sees_bad(dag_list, bad, T), TOL[torch.bfloat16])


# a branch and the last token of another one hold nothing but Inf and NaN, in every input: the siblings' gradients, and those
# of the tokens in front of the fork for the rows' part, are what they are without them
@pytest.mark.parametrize("hq,hkv,d", [(2, 1, 64), (3, 1, 64), (4, 1, 128), (5, 1, 128)])
@pytest.mark.parametrize("prefix,branches", [(128, [64, 64, 64, 64]), (77, [40, 100, 64, 90, 130]),
                                             (2000, [64, 40, 100, 64])])  # (the last: chunks of 33 key tiles, shared by five workgroups)
def test_hidden_tokens_backward(prefix, branches, hq, hkv, d):
    dag_list = [dags.fork_join(prefix, branches, None), dags.linear_chain([200, 77])]
    L, anc = dag_list[0]
    T = int(sum(int(np.sum(x)) for x, _ in dag_list))
    start = prefix + branches[0]
    bad = np.concatenate([np.arange(start, start + branches[1]), [prefix + sum(branches[:3]) - 1]])
    q, k, v = dags.make_qkv(90 + hq, T, hq, hkv, d, 0.7, torch.bfloat16)
    dout = dags.make_qkv(91 + hq, T, hq, hkv, d, 1.0, torch.bfloat16)[0]
    _, meta = build_meta(dag_list, hq, hkv, d, torch.bfloat16)
    qd, kd, vd, dod = (_spoil(x, bad).to(DEV) for x in (q, k, v, dout))
    out, lse = torch.empty_like(qd), torch.empty(T, hq, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, qd, kd, vd, out, lse)
    dq, dk, dv = torch.empty_like(qd), torch.empty_like(kd), torch.empty_like(vd)
    B.dag_attn_prefill_bwd(meta, qd, kd, vd, out, dod, lse, dq, dk, dv)
    ref, t0 = [], 0
    for x, y in dag_list:
        sl = slice(t0, t0 + int(np.sum(x)))
        ref.append(orc.attn_prefill_bwd(*(dags.to_f64(z[sl]) for z in (q, k, v, dout)), x, y))
        t0 = sl.stop
    dq_ref, dk_ref, dv_ref = (np.concatenate(z) for z in zip(*ref))
    lost_rows = _sees_bad(dag_list, bad, T)                 # (a bad row sees itself)
    lost_keys, n = np.zeros(T, dtype=bool), int(np.sum(L))
    lost_keys[:n] = orc.explicit_mask(L, anc)[lost_rows[:n]].any(axis=0)
    assert not lost_keys.all() and lost_keys[:prefix].all()
    _check(dq, dq_ref, ~lost_rows, TOL[torch.bfloat16])
    _check(dk, dk_ref, ~lost_keys, TOL[torch.bfloat16])
    _check(dv, dv_ref, ~lost_keys, TOL[torch.bfloat16])
    assert not torch.isfinite(dv[:prefix].float()).all(dim=-1).any()
