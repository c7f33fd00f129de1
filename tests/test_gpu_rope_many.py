"""GPU parity of dag_rope_qk where sixteen tokens share a block: few heads, many tokens, a ragged last block."""
import numpy as np
import pytest
import torch

from oracle import dag_oracle as orc
from paper_2602_07529_amd import binding as B
from workloads import dags
from tests.gpu_util import DEV, check_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [8192, 8193, 8207])
@pytest.mark.parametrize("hq,hkv,d,dtype", [(1, 1, 64, torch.bfloat16), (5, 1, 128, torch.bfloat16), (6, 2, 128, torch.bfloat16), (3, 1, 96, torch.bfloat16), (2, 1, 64, torch.float32)])
def test_many_tokens_of_few_heads(T, hq, hkv, d, dtype):
    q, k, _ = dags.make_qkv(13, T, hq, hkv, d, 1.0, dtype)
    pos = np.random.Generator(np.random.PCG64(4)).integers(0, 60000, size=T).astype(np.int32)
    qd, kd = q.to(DEV).clone(), k.to(DEV).clone()
    B.dag_rope_qk(torch.from_numpy(pos).to(DEV), qd, kd, 5e5)
    torch.cuda.synchronize()
    check_close(qd, orc.rope(dags.to_f64(q), pos, 5e5), dtype, "q")
    check_close(kd, orc.rope(dags.to_f64(k), pos, 5e5), dtype, "k")
