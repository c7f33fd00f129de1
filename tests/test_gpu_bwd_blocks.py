"""GPU: dK / dV on blocks of keys that are cut at node borders, against the fp64 oracle: blocks of one node and of several, of 64 to
128 keys and shorter ones at the end, sequences that keep blocks of 128 beside others, one and two visibility words."""
import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, build_meta
from tests.test_gpu_bwd_pieces import _without_pieces
from tests.test_gpu_prefill_bwd import _check_against_oracle, _forward_backward, check_close

pytestmark = pytest.mark.gpu


def _dags(name):
    rng = np.random.Generator(np.random.PCG64(8100))
    return {
        # blocks that end at borders (64, 127, 128 and 129 keys a node), a last block of 63 keys, beside a chain that keeps blocks of 128
        "edges": [dags.linear_chain([64, 65, 127, 128, 129, 1, 63, 192] * 3 + [1]), dags.fork_join(700, [128, 64, 129, 127, 1] * 2, 63),
                  dags.linear_chain([133])],
        "words": [dags.random_dag(rng, n_nodes=70, depth=6, len_lo=10, len_hi=90)[:2], dags.random_dag(rng, n_nodes=30, depth=5, len_lo=20, len_hi=160)[:2]],
        # siblings of about 100 tokens, for which blocks of 128 keys cost less, beside one that is cut
        "even": [dags.fork_join(484, [106, 95, 100, 111] * 3, 30), dags.random_dag(rng, n_nodes=40, depth=5, len_lo=30, len_hi=150)[:2], dags.linear_chain([700])],
    }[name]


def _blocks(L, anc, g):
    """The rule of cut_keys: (first keys of the blocks, whether they are cut at borders), which they are where their streams cost 3 % less
    than those of blocks of 128 keys."""
    L = [int(x) for x in L]
    n, starts = len(L), [int(x) for x in np.cumsum([0] + L)]
    T = starts[-1]
    sees = np.zeros((n, n), dtype=bool)
    for v in range(n):
        sees[v, [u for u in range(n) if int(anc[v][u >> 6]) >> (u & 63) & 1]] = sees[v, v] = True
    node = np.repeat(np.arange(n), L)
    costs, keys = [], [[], []]
    for cut in (False, True):
        key0, cost = 0, 0.0
        while key0 < T:
            keys[cut].append(key0)
            ends = [b for b in starts if key0 + 64 <= b <= key0 + 128]
            key1 = T if T <= key0 + 128 else ends[-1] if cut and ends else key0 + 128
            u0, u1 = node[key0], node[key1 - 1]
            rows = starts[u0] - key0 + sum(L[v] for v in range(n) if sees[v, u0:u1 + 1].any())
            sure = sum(starts[u1 + 1] - key1 if v == u1 else L[v] for v in range(n) if sees[v, u0:u1 + 1].all())
            cost += g * (1.25 * (-(-rows // 64)) - 0.25 * (sure // 64)) + 8
            key0 = key1
        costs.append(cost)
    cut = not costs[0] < 1.03 * costs[1]
    return keys[cut], cut


def _is_cut(L, anc, g):
    return _blocks(L, anc, g)[1]


def _key_tables(meta, ws, hq):
    """What a call has left of its blocks in the workspace: (weights, first keys), a slot for every 64 keys of a sequence."""
    up = lambda n: -(-n // 256) * 256  # noqa: E731
    rows, tiles = up(meta.sizes.total_tokens * hq * 4), meta.sizes.total_ktiles
    skip = -ws.data_ptr() % 256
    at = lambda o: ws[skip + o:skip + o + 4 * tiles].view(torch.int32).cpu().numpy()  # noqa: E731
    return at(2 * rows), at(2 * rows + 2 * up(4 * tiles))


@pytest.mark.parametrize("name,cut", [("edges", [False, True, False]), ("words", [True, True]), ("even", [False, True, False])])
@pytest.mark.parametrize("hq,hkv,d", [(2, 1, 64), (8, 2, 64), (4, 2, 128), (5, 1, 128)])
def test_dkv_blocks(name, cut, hq, hkv, d, monkeypatch):
    dag_list = _dags(name)
    assert sum(int(np.sum(L)) for L, _ in dag_list) >= 4096
    blocks = [_blocks(L, anc, hq // hkv) for L, anc in dag_list]
    assert [c for _, c in blocks] == cut
    _, meta = build_meta(dag_list, hq, hkv, d, torch.bfloat16)
    ws = torch.zeros(B.dag_prefill_bwd_workspace_bytes(meta, hq, hkv, d), dtype=torch.uint8, device=DEV)
    call = B.dag_attn_prefill_bwd
    monkeypatch.setattr(B, "dag_attn_prefill_bwd", lambda *args, **kw: call(*args, workspace=ws, **kw))
    inputs, grads = _forward_backward(dag_list, hq, hkv, d, 8200 + hq)
    first = _key_tables(meta, ws, hq)[1]
    for (L, _), (keys, _) in zip(dag_list, blocks):   # (slots without a block hold the end of the sequence)
        T = int(np.sum(L))
        slots, first = first[:-(-T // 64)], first[-(-T // 64):]
        assert slots.tolist() == keys + [T] * (len(slots) - len(keys))
    _check_against_oracle(dag_list, inputs, grads)


@pytest.mark.parametrize("hq,hkv,d", [(2, 1, 64), (3, 1, 128)])
def test_hidden_keys_behind_a_short_block(hq, hkv, d):
    """A branch whose rows are Inf, next to blocks of fewer than 128 keys: the lanes of those blocks without a key of their own take part
    in the tiles without masks and must not reach anything that is stored."""
    L, anc = dag = dags.fork_join(300, [128, 64, 129, 127, 193] * 7, 63)
    T = int(np.sum(L))
    assert T >= 4096 and _is_cut(L, anc, hq // hkv)
    q, k, v = dags.make_qkv(8300, T, hq, hkv, d, 0.7, torch.bfloat16)
    dout = dags.make_qkv(8301, T, hq, hkv, d, 1.0, torch.bfloat16)[0]
    ref = orc.attn_prefill_bwd(*(dags.to_f64(x) for x in (q, k, v, dout)), L, anc)
    _, meta = build_meta([dag], hq, hkv, d, torch.bfloat16)
    out, lse = torch.empty_like(q, device=DEV), torch.empty(T, hq, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, q.to(DEV), k.to(DEV), v.to(DEV), out, lse)
    bad = slice(428, 492)  # the second branch
    qd, dod = q.to(DEV), dout.to(DEV)
    qd[bad], dod[bad] = float("inf"), float("inf")
    dq, dk, dv = torch.empty_like(qd), torch.empty(T, hkv, d, dtype=torch.bfloat16, device=DEV), torch.empty(T, hkv, d, dtype=torch.bfloat16, device=DEV)
    B.dag_attn_prefill_bwd(meta, qd, k.to(DEV), v.to(DEV), out, dod, lse, dq, dk, dv)
    torch.cuda.synchronize()
    for sl in (slice(300, 428), slice(492, T)):
        check_close(dk[sl], ref[1][sl], torch.bfloat16, "dk")
        check_close(dv[sl], ref[2][sl], torch.bfloat16, "dv")
    assert not torch.isfinite(dv[:300].float()).all(dim=-1).any()


def test_a_sequence_of_more_blocks_than_there_is_room_for():
    """Over 1024 key tiles: the sequence keeps blocks of 128, beside one that is cut.  Against the call without room for pieces, which has
    no blocks."""
    hq, hkv, d = 2, 1, 64
    long, short = dags.fork_join(40, [600] * 110, 30), dags.fork_join(700, [128, 64, 129, 127, 1] * 2, 63)
    keys, cut = _blocks(*short, hq // hkv)
    T = [int(np.sum(L)) for L, _ in (long, short)]
    assert T[0] > 1024 * 64 and cut
    q, k, v, dout = (x.to(DEV) for x in (*dags.make_qkv(8400, sum(T), hq, hkv, d, 0.7, torch.bfloat16), dags.make_qkv(8401, sum(T), hq, hkv, d, 1.0, torch.bfloat16)[0]))
    _, meta = build_meta([long, short], hq, hkv, d, torch.bfloat16)
    out, lse = torch.empty_like(q), torch.empty(sum(T), hq, dtype=torch.float32, device=DEV)
    B.dag_attn_prefill(meta, q, k, v, out, lse)
    grads = []
    for size in (_without_pieces(meta, hq, hkv, d), B.dag_prefill_bwd_workspace_bytes(meta, hq, hkv, d)):
        ws = torch.zeros(size, dtype=torch.uint8, device=DEV)
        grads.append((torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)))
        B.dag_attn_prefill_bwd(meta, q, k, v, out, dout, lse, *grads[-1], workspace=ws)
    first = _key_tables(meta, ws, hq)[1].tolist()
    slots = [-(-t // 64) for t in T]
    even = list(range(0, T[0], 128))
    assert first[:slots[0]] == even + [T[0]] * (slots[0] - len(even))
    assert first[slots[0]:] == keys + [T[1]] * (slots[1] - len(keys))
    for a, b in zip(*grads):   # (fp32 sums in another order, half a unit of bf16 each: 2^-9)
        assert torch.isfinite(b.float()).all() and float((a.double() - b.double()).norm()) <= 4e-3 * float(a.double().norm())
