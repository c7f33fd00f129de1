"""GPU: dQ on query chunks, whose items hold all heads of a group as row-major (row, head) pairs, against the fp64 oracle: groups with pairs
that belong to no row or no head, waves without rows, items of more than eight heads, tiles shared out over several workgroups."""
import numpy as np
import pytest

from workloads import dags
from tests.test_gpu_prefill_bwd import _check_against_oracle, _forward_backward

pytestmark = pytest.mark.gpu


def _dags(name):
    rng = np.random.Generator(np.random.PCG64(8400))
    return {
        # remainders of every chunk size (256 to 16 rows), one token, two visibility words
        "batch": [dags.fork_join(130, [40, 64, 3, 150, 63], 70), dags.linear_chain([1]), dags.linear_chain([65, 190, 257]),
                  dags.random_dag(rng, n_nodes=70, depth=6, len_lo=10, len_hi=40)[:2]],
        # few chunks of many tiles: pieces
        "pieces": [dags.fork_join(1100, [70, 33], 51)],
    }[name]


@pytest.mark.parametrize("name", ["batch", "pieces"])
@pytest.mark.parametrize("g", [1, 2, 3, 4, 5, 7, 8, 9, 17])
@pytest.mark.parametrize("d", [64, 128])
def test_every_group(name, g, d):
    hkv = 2 if name == "batch" and g < 9 else 1
    dag_list = _dags(name)
    inputs, grads = _forward_backward(dag_list, g * hkv, hkv, d, 8500 + g + d)
    _check_against_oracle(dag_list, inputs, grads)
