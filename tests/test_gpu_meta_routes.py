"""GPU parity of dag_build_meta where its launches change: one workgroup for a small batch, the node table as
a kernel argument or as copies.  Integer tables, bit-exact."""
import numpy as np
import pytest

from workloads import dags
from tests.gpu_util import assert_meta_equal, oracle_meta
from tests.test_gpu_meta import _build_with_tiles

pytestmark = pytest.mark.gpu


def _random(seed, n, lo, hi):
    rng = np.random.Generator(np.random.PCG64(seed))
    return dags.random_dag(rng, n_nodes=n, depth=5, len_lo=lo, len_hi=hi)[:2]


# 2048 = 32 x 64 tokens is the largest one-workgroup batch with tiles of 64
@pytest.mark.parametrize("name,make", [
    ("one token", lambda: [dags.linear_chain([1])]),
    ("32 tiles", lambda: [dags.fork_join(512, [256] * 5, 256)]),
    ("33 tiles", lambda: [dags.fork_join(512, [256] * 5, 257)]),
    ("64 sequences", lambda: [dags.linear_chain([b % 3 + 1]) for b in range(64)]),
    ("65 sequences", lambda: [dags.linear_chain([b % 3 + 1]) for b in range(65)]),
    ("three sequences", lambda: [_random(1, 64, 1, 20), dags.linear_chain([5, 7]), _random(2, 63, 1, 20)]),
    ("two words", lambda: [_random(3, 130, 1, 9), dags.linear_chain([4])]),
    ("largest argument", lambda: [dags.linear_chain([b + 1]) for b in range(8)] + [_random(4, 64, 1, 3)] * 4),
    ("copies", lambda: [_random(5, 64, 20, 60)] * 6),
])
def test_meta_routes(name, make):
    dag_list = make()
    for tm, tn in ((64, 64), (5, 3)) if sum(int(np.sum(L)) for L, _ in dag_list) < 700 else ((64, 64),):
        assert_meta_equal(_build_with_tiles(dag_list, tm, tn), oracle_meta(dag_list, tm, tn))


@pytest.mark.parametrize("nodes", [296, 297, 298, 299])
def test_meta_table_around_the_argument_limit(nodes):
    dag_list = [dags.linear_chain([1] * 60), _random(nodes, 60, 1, 4), _random(nodes + 1, 60, 1, 4),
                _random(nodes + 2, 60, 1, 4), _random(nodes + 3, nodes - 240, 1, 4)]
    assert_meta_equal(_build_with_tiles(dag_list, 64, 64), oracle_meta(dag_list, 64, 64))
