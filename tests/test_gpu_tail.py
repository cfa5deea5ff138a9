"""The tail of a narrow bottleneck over few pixels, 3x3 64 -> 64, 1x1 to 256 with a residual and the next block's 1x1 back, in one launch, against the oracle and the
launches apart."""
import numpy as np
import pytest

from gpu_common import check_layers, define_retained, with_infinities
from oracle import network as N
from oracle import topology as T
from workload import gen

pytestmark = pytest.mark.gpu
O = T.Op
RELU, HSWISH = 1, 2


def net(act1, act2, act3):
    """stem -> 1x1 to 256 -> two bottlenecks (256 -> 64, 3x3, 64 -> 256 plus the block's input) -> head."""
    ops = [O(T.CONV, 3, 32, 3, 3, 2, 1, RELU, -1, -1), O(T.CONV, 32, 256, 1, 1, 1, 0, RELU, -1, 0)]
    last = 1
    for _ in range(2):
        ops += [O(T.CONV, 256, 64, 1, 1, 1, 0, act3, -1, last), O(T.CONV, 64, 64, 3, 3, 1, 1, act1, -1, last + 1), O(T.CONV, 64, 256, 1, 1, 1, 0, act2, last, last + 2)]
        last += 3
    return ops + [O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, last), O(T.FC, 256, 11, 1, 1, 1, 0, 0, -1, last + 1), O(T.SOFTMAX, 11, 11, 0, 0, 1, 0, 0, -1, last + 2)]


# One and two groups of 16 pixels a workgroup at the edge between them and at the largest that is not the 64-pixel form's, tiles that end within an image or
# a group, maps of a pixel, a row and a column, every activation
@pytest.mark.parametrize("h,w,batch,act1,act2,act3,dtype", [
    (56, 56, 1, RELU, RELU, RELU, "fp16"), (64, 64, 1, RELU, RELU, RELU, "bf16"), (4097, 1, 1, RELU, 0, RELU, "fp16"), (49, 41, 3, RELU, RELU, HSWISH, "bf16"),
    (55, 55, 2, HSWISH, RELU, 0, "fp16"), (1, 1, 1, RELU, RELU, RELU, "fp16"), (1, 19, 3, 0, RELU, RELU, "fp16"), (37, 1, 2, RELU, HSWISH, RELU, "bf16"),
    (3, 5, 7, RELU, RELU, RELU, "fp16"), (7, 9, 1, RELU, RELU, RELU, "bf16"), (13, 17, 16, RELU, RELU, RELU, "fp16"), (33, 31, 5, RELU, RELU, RELU, "fp16"),
    (91, 90, 1, HSWISH, RELU, RELU, "fp16"), (64, 64, 2, RELU, HSWISH, RELU, "bf16")])   # hard swish: up to 8192 pixels, which the 64-pixel form would have
def test_tail_of_a_narrow_bottleneck_in_one_launch(h, w, batch, act1, act2, act3, dtype):
    from paper_2006_02464_amd.runner import Worker
    ops = net(act1, act2, act3)
    wts, biases = gen.model_tensors(T.weight_shapes(ops), 9, dtype)
    x = gen.images(9, 0, batch, 3, 2 * h, 2 * w, "uniform", dtype)
    ref = N.forward(ops, wts, biases, x, prec="f32")["logits"]
    wk = Worker(workspace_bytes=512 << 20, io_bytes=64 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        got = []
        for on in (1, 0):
            wk.ctx.set_fusion(on)
            mid = wk.ctx.model_define(ops, 3, 2 * h, 2 * w, batch_sizes=(batch,), dtype=dtype)
            tail = {l["op_index"]: wk.ctx.plan_launch_tail(mid, batch, i) for i, l in enumerate(wk.ctx.plan(mid, batch)) if l["kind"] == 1}
            assert [tail[k] for k in range(2, 8)] == ([0, 1, 1, 3, 1, 2] if on else [0] * 6)
            wk.load(mid, gen.pack_blob(wts, biases, dtype))
            got.append(wk.infer(mid, x, classes=11)[1])
        # seven roundings to the storage type on the way, each at most half a unit in the last place of a value
        tol = 8 * (2.0 ** -11 if dtype == "fp16" else 2.0 ** -8)
        for z in got:
            assert np.abs(z - ref).max() <= tol * np.abs(ref).max()
        assert np.abs(got[0] - got[1]).max() <= tol * np.abs(ref).max()
        # every stored element; without the third layer the first block's 1x1 and the last one's launches are the same form
        for third in (1, 0):
            wk.ctx.set_fusion_third(third)
            wk.ctx.set_fusion(1)
            mid = define_retained(wk.ctx, ops, 2 * h, 2 * w, batch, dtype)
            assert [t for t in (wk.ctx.plan_launch_tail(mid, batch, i) for i in range(len(wk.ctx.plan(mid, batch)))) if t] == ([1, 1, 3, 1, 2] if third else [1, 2, 1, 2])
            wk.load(mid, gen.pack_blob(wts, biases, dtype))
            wk.infer(mid, x, classes=11)
            check_layers(wk.ctx, ops, wts, biases, mid, batch, x, dtype, unstored=(3, 6))
    finally:
        wk.ctx.set_fusion(1)
        wk.ctx.set_fusion_third(1)
        wk.close()


def net_with_projection(act1, act3):
    """stem -> 1x1 to 64 -> a block whose shortcut is a 1x1 64 -> 256 -> a block with its input as the shortcut -> head."""
    ops = [O(T.CONV, 3, 32, 3, 3, 2, 1, RELU, -1, -1), O(T.CONV, 32, 64, 1, 1, 1, 0, RELU, -1, 0),
           O(T.CONV, 64, 64, 1, 1, 1, 0, RELU, -1, 1), O(T.CONV, 64, 64, 3, 3, 1, 1, act1, -1, 2), O(T.CONV, 64, 256, 1, 1, 1, 0, 0, -1, 1), O(T.CONV, 64, 256, 1, 1, 1, 0, RELU, 4, 3),
           O(T.CONV, 256, 64, 1, 1, 1, 0, act3, -1, 5), O(T.CONV, 64, 64, 3, 3, 1, 1, RELU, -1, 6), O(T.CONV, 64, 256, 1, 1, 1, 0, RELU, 5, 7)]
    return ops + [O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, 8), O(T.FC, 256, 11, 1, 1, 1, 0, 0, -1, 9), O(T.SOFTMAX, 11, 11, 0, 0, 1, 0, 0, -1, 10)]


# One to four tiles of 32 pixels a workgroup (and more, for the other fused form), the last workgroup with all of them, some, and one of a single pixel; maps of a row and a column
@pytest.mark.parametrize("h,w,batch,act1,act3,third,dtype", [
    (79, 77, 1, RELU, RELU, 1, "fp16"), (64, 64, 2, RELU, 0, 1, "bf16"), (8193, 1, 1, RELU, RELU, 1, "fp16"), (1, 6145, 2, 0, RELU, 0, "fp16"), (128, 129, 1, RELU, RELU, 1, "bf16"),
    (56, 56, 16, RELU, RELU, 1, "fp16"), (56, 56, 4, 0, 0, 0, "bf16"), (97, 97, 3, RELU, RELU, 1, "fp16"), (90, 91, 4, RELU, 0, 0, "bf16"), (113, 97, 6, RELU, RELU, 1, "fp16"), (41, 49, 13, RELU, RELU, 1, "bf16")])
def test_tail_of_a_narrow_bottleneck_walks_many_pixels(h, w, batch, act1, act3, third, dtype):
    from paper_2006_02464_amd.runner import Worker
    ops = net_with_projection(act1, act3)
    wts, biases = gen.model_tensors(T.weight_shapes(ops), 9, dtype)
    x = gen.images(9, 0, batch, 3, 2 * h, 2 * w, "uniform", dtype)
    ref = N.forward(ops, wts, biases, x, prec="f32")["logits"]
    wk = Worker(workspace_bytes=1 << 30, io_bytes=128 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=128 << 20)
    try:
        wk.ctx.set_fusion_third(third)
        got = []
        for on in (1, 0):
            wk.ctx.set_fusion(on)
            mid = wk.ctx.model_define(ops, 3, 2 * h, 2 * w, batch_sizes=(batch,), dtype=dtype)
            fused = [l for l in wk.ctx.plan(mid, batch) if l["fused_op"] >= 0 and l["kind"] == 1]
            assert [(l["op_index"], l["proj_op"], l["next_op"]) for l in fused] == ([(5, 4, 6 if third else -1), (8, -1, -1)] if on else [])
            tiles = -(-h * w * batch // (32 * 256))
            walk = [l for l in fused if l["tile_m"] == 32 * tiles and l["block"] == 512]
            assert len(walk) == (on and (tiles <= 4) + (tiles <= 3)) and all(l["proj_op"] == 4 for l in walk[:1])   # with the projection up to four tiles
            assert all(l["grid_x"] <= 256 for l in walk)
            wk.load(mid, gen.pack_blob(wts, biases, dtype))
            got.append(wk.infer(mid, x, classes=11)[1])
        # nine roundings to the storage type on the way, each at most half a unit in the last place of a value
        tol = 8 * (2.0 ** -11 if dtype == "fp16" else 2.0 ** -8)
        for z in got:
            assert np.abs(z - ref).max() <= tol * np.abs(ref).max()
        assert np.abs(got[0] - got[1]).max() <= tol * np.abs(ref).max()
        wk.ctx.set_fusion(1)   # every stored element
        mid = define_retained(wk.ctx, ops, 2 * h, 2 * w, batch, dtype)
        assert len([l for l in wk.ctx.plan(mid, batch) if l["fused_op"] >= 0 and l["tile_m"] == 32 * tiles and l["block"] == 512]) == (tiles <= 4) + (tiles <= 3)
        wk.load(mid, gen.pack_blob(wts, biases, dtype))
        wk.infer(mid, x, classes=11)
        check_layers(wk.ctx, ops, wts, biases, mid, batch, x, dtype, unstored=(3, 4, 7), unrounded=(4,))
    finally:
        wk.ctx.set_fusion(1)
        wk.ctx.set_fusion_third(1)
        wk.close()


def test_layers_stay_apart_where_the_workspace_has_no_room_for_their_joint_launch():
    """The launch keeps the 3x3's input until its last layer is done; a workspace that only has what the launches apart need gets those."""
    import paper_2006_02464_amd as cw
    ops = net(RELU, RELU, RELU)
    tails = lambda c, m: [c.plan_launch_tail(m, 3, i) for i in range(c.plan_num_launches(m, 3))]
    sizes = dict(io_bytes=16 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=16 << 20)
    need = []
    for room in (64 << 20, None, None):
        c = cw.Context(workspace_bytes=room or need[-1] - (len(need) - 1) * 256, **sizes)
        try:
            m = c.model_define(ops, 3, 80, 72, batch_sizes=(3,))
            assert any(tails(c, m)) == (len(need) < 2)
            need.append(c.model_workspace_bytes(m, 3))
        finally:
            c.destroy()
    assert need[0] == need[1] > need[2]


# Few pixels in groups of 16 and 32, and the walk with one tile of 32 pixels and with two
@pytest.mark.parametrize("form,h,w,batch,act,dtype", [("tail", 21, 19, 3, 0, "fp16"), ("tail", 55, 55, 2, 0, "bf16"), ("tail", 21, 19, 3, HSWISH, "fp16"), ("tail", 55, 55, 2, RELU, "fp16"),
                                                      ("walk", 79, 77, 1, 0, "fp16"), ("walk", 64, 71, 3, 0, "bf16"), ("walk", 64, 71, 3, RELU, "fp16")])
def test_tail_of_a_narrow_bottleneck_on_non_finite_values(form, h, w, batch, act, dtype):
    """NaN and infinities in the images, inside and at the edges of the map, and then infinite weights: the same elements are NaN or infinite as in the oracle."""
    from paper_2006_02464_amd.runner import Worker
    ops = net(act, act, act) if form == "tail" else net_with_projection(RELU, RELU)
    ops = [o._replace(relu=0) if o.op == T.CONV and (i < 2 or act == 0) else o for i, o in enumerate(ops)]   # (ReLU of NaN is 0)
    wts, biases = gen.model_tensors(T.weight_shapes(ops), 9, dtype)
    x = gen.images(9, 0, batch, 3, 2 * h, 2 * w, "uniform", dtype).copy()
    x[0, 0, h, w], x[-1, 1, 0, 0], x[-1, 2, 2 * h - 1, w], x[0, 0, h // 2, 2 * w - 1] = np.nan, np.inf, -np.inf, np.inf
    unstored, unrounded = dict(tail=((3, 6), ()), walk=((3, 4, 7), (4,)))[form]
    wk = Worker(workspace_bytes=512 << 20, io_bytes=64 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        mid = define_retained(wk.ctx, ops, 2 * h, 2 * w, batch, dtype)
        wk.load(mid, gen.pack_blob(wts, biases, dtype))
        wk.infer(mid, x, classes=11)
        # (the first convolution's filter rows are padded with weights of zero, which an infinite pixel beside the filter makes NaN)
        assert check_layers(wk.ctx, ops, wts, biases, mid, batch, x, dtype, unstored, unrounded, given=(0,)) > (0 if act == RELU else 1000) - 1
        wts = with_infinities(ops, wts, {3: (7, 5, 0, 0), unstored[-1]: (9, 3, 2, 2), unstored[-1] + 1: (200, 11, 0, 0)})
        x = gen.images(4, 0, batch, 3, 2 * h, 2 * w, "uniform", dtype)
        wk.ctx.unload_weights(mid)
        wk.load(mid, gen.pack_blob(wts, biases, dtype))
        wk.infer(mid, x, classes=11)
        assert check_layers(wk.ctx, ops, wts, biases, mid, batch, x, dtype, unstored, unrounded) > 0
    finally:
        wk.close()
