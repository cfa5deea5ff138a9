"""LOAD's re-layout: more tensors than one launch describes, every filter form, channel counts beside the chunks it works in."""
import pytest

from gpu_common import TOL, Case, rel_err_per_sample
from oracle import topology as T
from test_gpu_parity import check_all_ops, check_head

pytestmark = pytest.mark.gpu
O = T.Op


def net(chain):
    ops = [O(T.CONV, 3, 32, 3, 3, 1, 1, 1, -1, -1), O(T.CONV, 32, 96, 3, 3, 1, 1, 1, -1, 0), O(T.CONV, 96, 32, 5, 5, 1, 2, 1, -1, 1),
           O(T.CONV, 32, 160, 1, 1, 1, 0, 1, -1, 2), O(T.CONV, 160, 32, 2, 2, 1, 0, 1, -1, 3)]
    for _ in range(chain):
        ops.append(O(T.CONV, 32, 32, 1, 1, 1, 0, 0, -1, 4))
    ops += [O(T.CONV, 32, 256, 3, 3, 2, 1, 1, -1, len(ops) - 1), O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, len(ops)),
            O(T.FC, 256, 7, 1, 1, 1, 0, 0, -1, len(ops) + 1), O(T.SOFTMAX, 7, 7, 0, 0, 1, 0, 0, -1, len(ops) + 2)]
    return ops


@pytest.mark.parametrize("chain,dtype", [(0, "fp16"), (0, "bf16"), (53, "fp16"), (54, "fp16")])   # 7, 60 and 61 tensors
def test_packed_weights(chain, dtype):
    from paper_2006_02464_amd.runner import Worker
    wk = Worker(workspace_bytes=256 << 20, io_bytes=16 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        case = Case(net(chain), 14, seed=4, dtype=dtype, dist="uniform")
        wk.ctx.set_debug_keep(True)
        mid = wk.ctx.model_define(case.ops, 3, 14, 14, batch_sizes=(2,), dtype=dtype)
        wk.load(mid, case.blob)
        x = case.images(0, 2)
        probs, logits, _ = wk.infer(mid, x, classes=7)
        outs, _, gpu = check_all_ops(wk, case, mid, 2, x)
        check_head(case, gpu[-1], logits, probs)
        assert rel_err_per_sample(logits, outs[-2]).max() <= TOL
    finally:
        wk.close()
