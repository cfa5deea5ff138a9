"""A densely connected layer, 1x1 to 128 channels and 3x3 to 32, in one launch, against the oracle and the two launches."""
import numpy as np
import pytest

from gpu_common import check_layers, define_retained, with_infinities
from oracle import network as N
from oracle import topology as T
from workload import gen

pytestmark = pytest.mark.gpu
O = T.Op
RELU, HSWISH = 1, 2


def net(k, act1, act2, concat):
    """stem -> 1x1 to k channels -> [1x1 k -> 128, 3x3 -> 32] (twice, the second over the concatenation) -> 1x1 to 256 -> head."""
    ops = [O(T.CONV, 3, 32, 3, 3, 2, 1, RELU, -1, -1), O(T.CONV, 32, k, 1, 1, 1, 0, RELU, -1, 0), O(T.CONV, k, 128, 1, 1, 1, 0, act1, -1, 1), O(T.CONV, 128, 32, 3, 3, 1, 1, act2, -1, 2)]
    last, c = 3, 32
    if concat:
        ops.append(O(T.CONCAT, k, k + 32, 0, 0, 1, 0, 0, 3, 1))
        ops += [O(T.CONV, k + 32, 128, 1, 1, 1, 0, act1, -1, 4), O(T.CONV, 128, 32, 3, 3, 1, 1, act2, -1, 5)]
        last = 6
    ops.append(O(T.CONV, c, 256, 1, 1, 1, 0, RELU, -1, last))
    return ops + [O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, last + 1), O(T.FC, 256, 11, 1, 1, 1, 0, 0, -1, last + 2), O(T.SOFTMAX, 11, 11, 0, 0, 1, 0, 0, -1, last + 3)]


# One to eight stages of 64 channels with and without half a stage at the end, both sizes of a wave's share, the ring of loads shorter and longer than K;
# maps of a pixel, a row and a column, tiles that the map does not divide into, several rounds of tiles
@pytest.mark.parametrize("h,w,k,batch,act1,act2,concat,dtype", [
    (28, 28, 64, 2, RELU, RELU, True, "fp16"), (28, 28, 160, 6, RELU, 0, True, "bf16"), (13, 29, 192, 3, HSWISH, RELU, True, "fp16"), (28, 28, 256, 6, RELU, HSWISH, False, "fp16"),
    (14, 14, 320, 3, RELU, RELU, False, "fp16"), (31, 17, 352, 4, 0, RELU, False, "fp16"), (15, 15, 416, 3, RELU, RELU, False, "bf16"), (28, 28, 480, 6, RELU, RELU, True, "fp16"),
    (56, 56, 32, 3, RELU, RELU, True, "fp16"), (56, 56, 96, 6, RELU, RELU, True, "fp16"), (57, 41, 160, 5, RELU, RELU, True, "bf16"), (40, 40, 256, 6, RELU, 0, False, "fp16"),
    (1, 1, 64, 3, RELU, RELU, True, "fp16"), (1, 19, 128, 1, RELU, RELU, True, "fp16"), (37, 1, 64, 2, HSWISH, RELU, True, "fp16"), (2, 3, 224, 1, RELU, RELU, False, "bf16"), (56, 56, 64, 12, RELU, RELU, False, "fp16")])
def test_densely_connected_layer_in_one_launch(h, w, k, batch, act1, act2, concat, dtype):
    from paper_2006_02464_amd.runner import Worker
    ops = net(k, act1, act2, concat)
    wts, biases = gen.model_tensors(T.weight_shapes(ops), 9, dtype)
    x = gen.images(9, 0, batch, 3, 2 * h, 2 * w, "uniform", dtype)
    ref = N.forward(ops, wts, biases, x, prec="f32")["logits"]
    wk = Worker(workspace_bytes=512 << 20, io_bytes=64 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        got = []
        for on in (1, 0):
            wk.ctx.set_fusion(on)
            mid = wk.ctx.model_define(ops, 3, 2 * h, 2 * w, batch_sizes=(batch,), dtype=dtype)
            joined = {l["op_index"] for i, l in enumerate(wk.ctx.plan(mid, batch)) if l["kind"] == 1 and wk.ctx.plan_launch_joined(mid, batch, i)}
            assert joined - {0} == (({2, 5} if concat else {2}) if on else set())
            wk.load(mid, gen.pack_blob(wts, biases, dtype))
            got.append(wk.infer(mid, x, classes=11)[1])
        # six or eight roundings to the storage type on the way, each at most half a unit in the last place of a value
        tol = 8 * (2.0 ** -11 if dtype == "fp16" else 2.0 ** -8)
        for z in got:
            assert np.abs(z - ref).max() <= tol * np.abs(ref).max()
        assert np.abs(got[0] - got[1]).max() <= tol * np.abs(ref).max()
        wk.ctx.set_fusion(1)   # every stored element
        mid = define_retained(wk.ctx, ops, 2 * h, 2 * w, batch, dtype)
        wk.load(mid, gen.pack_blob(wts, biases, dtype))
        wk.infer(mid, x, classes=11)
        check_layers(wk.ctx, ops, wts, biases, mid, batch, x, dtype, unstored=(2, 5) if concat else (2,))
    finally:
        wk.ctx.set_fusion(1)
        wk.close()


@pytest.mark.parametrize("h,w,k,batch,act,dtype", [(15, 13, 96, 3, 0, "fp16"), (28, 28, 256, 6, HSWISH, "bf16"), (13, 29, 160, 3, RELU, "fp16")])
def test_densely_connected_layer_on_non_finite_values(h, w, k, batch, act, dtype):
    """NaN and infinities in the images, inside and at the edges of the map, and then infinite weights: the same elements are NaN or infinite as in the oracle."""
    from paper_2006_02464_amd.runner import Worker
    ops = [o._replace(relu=0) if o.op == T.CONV and (i < 2 or act == 0) else o for i, o in enumerate(net(k, act, act, True))]   # (ReLU of NaN is 0)
    wts, biases = gen.model_tensors(T.weight_shapes(ops), 9, dtype)
    x = gen.images(9, 0, batch, 3, 2 * h, 2 * w, "uniform", dtype).copy()
    x[0, 0, h, w], x[1, 1, 0, 0], x[1, 2, 2 * h - 1, w], x[2, 0, h // 2, 2 * w - 1] = np.nan, np.inf, -np.inf, np.inf
    wk = Worker(workspace_bytes=512 << 20, io_bytes=64 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        mid = define_retained(wk.ctx, ops, 2 * h, 2 * w, batch, dtype)
        wk.load(mid, gen.pack_blob(wts, biases, dtype))
        wk.infer(mid, x, classes=11)
        # (the first convolution's filter rows are padded with weights of zero, which an infinite pixel beside the filter makes NaN)
        assert check_layers(wk.ctx, ops, wts, biases, mid, batch, x, dtype, (2, 5), given=(0,)) > (0 if act == RELU else 500) - 1
        wts = with_infinities(ops, wts, {3: (7, 5, 0, 0), 5: (100, 40, 0, 0), 6: (9, 3, 2, 2)})
        x = gen.images(4, 0, batch, 3, 2 * h, 2 * w, "uniform", dtype)
        wk.ctx.unload_weights(mid)
        wk.load(mid, gen.pack_blob(wts, biases, dtype))
        wk.infer(mid, x, classes=11)
        assert check_layers(wk.ctx, ops, wts, biases, mid, batch, x, dtype, (2, 5)) > 0
    finally:
        wk.close()
