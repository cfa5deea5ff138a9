"""Input cast, first convolution, max pool and the 1x1 behind it as one launch, against the plan that debug retention makes:
the same launches for everything behind the head, cast, convolution and pool as launches of their own (which other tests hold
against the CPU oracle layer by layer).  Every tensor is rounded at the same places and K runs in the same order: same bits."""
import numpy as np
import pytest
import torch

from oracle import topology as T

pytestmark = pytest.mark.gpu
O = T.Op


def net(head, cin, act, n1):
    """A first convolution in one of the launch's two forms, with a pool behind the 7x7, and a tail that reads all of its results."""
    if head == "3x3":
        ops = [O(T.CONV, cin, 32, 3, 3, 2, 1, act, -1, -1), O(T.CONV, 32, 256, 1, 1, 1, 0, 0, -1, 0)]
    else:
        ops = [O(T.CONV, cin, 64, 7, 7, 2, 3, act, -1, -1), O(T.MAXPOOL, 64, 64, 3, 3, 2, 1, 0, -1, 0)]
        if n1:
            ops += [O(T.CONV, 64, n1, 1, 1, 1, 0, act % 2, -1, 1), O(T.CONV, 64, 64, 3, 3, 1, 1, 1, -1, 1),
                    O(T.CONV, n1, 256, 1, 1, 2, 0, 0, -1, 2), O(T.CONV, 64, 256, 1, 1, 2, 0, 0, 4, 3)]
        else:
            ops += [O(T.CONV, 64, 256, 3, 3, 1, 1, 0, -1, 1)]
    k = len(ops) - 1
    return ops + [O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, k), O(T.FC, 256, 40, 1, 1, 1, 0, 0, -1, k + 1), O(T.SOFTMAX, 40, 40, 0, 0, 1, 0, 0, -1, k + 2)]


def logits(ctx, ops, cin, h, w, batch, dtype, keep, blob, x):
    ctx.set_debug_keep(keep)
    try:
        m = ctx.model_define([tuple(o) for o in ops], cin, h, w, batch_sizes=(batch,), dtype=dtype)
    finally:
        ctx.set_debug_keep(False)
    plan = ctx.plan(m, batch)
    joined = [i for i in range(len(plan)) if ctx.plan_launch_joined(m, batch, i)]
    st = torch.cuda.current_stream()
    ctx.load_weights(m, blob, st)
    out, probs = (torch.zeros(batch, 40).pin_memory() for _ in range(2))
    slot = ctx.input(m, batch, x, st)
    ctx.exec(m, batch, slot, st)
    ctx.output(slot, probs, out, st)
    torch.cuda.synchronize()
    ctx.unload_weights(m)
    return out.numpy().copy(), joined, plan


@pytest.fixture(scope="module")
def ctx():
    from paper_2006_02464_amd.binding import Context
    c = Context(workspace_bytes=512 << 20, io_bytes=64 << 20, weight_pool_bytes=256 << 20, load_staging_bytes=16 << 20)
    yield c
    c.destroy()


# maps of one pixel; just below, at and above a tile; both heights of the pooled tile; C below 4 and 4; every activation
@pytest.mark.parametrize("head,cin,act,n1,h,w,batch,dtype", [
    ("7x7", 3, 1, 0, 1, 1, 1, "fp16"), ("7x7", 3, 1, 0, 27, 33, 3, "fp16"), ("7x7", 4, 0, 0, 29, 31, 2, "bf16"), ("7x7", 1, 2, 0, 64, 65, 1, "fp16"),
    ("7x7", 3, 1, 0, 224, 224, 5, "bf16"), ("7x7", 3, 0, 0, 61, 223, 40, "fp16"),
    ("7x7", 3, 1, 64, 224, 200, 3, "fp16"), ("7x7", 3, 2, 128, 219, 221, 3, "bf16"), ("7x7", 2, 0, 64, 113, 97, 14, "bf16"), ("7x7", 3, 1, 128, 112, 127, 11, "fp16"),
    ("3x3", 3, 1, 0, 1, 1, 2, "fp16"), ("3x3", 3, 2, 0, 33, 63, 3, "bf16"), ("3x3", 4, 0, 0, 130, 31, 2, "fp16"), ("3x3", 1, 1, 0, 16, 34, 1, "bf16"),
])
def test_head_as_one_launch_gives_the_same_bits(ctx, head, cin, act, n1, h, w, batch, dtype):
    ops = net(head, cin, act, n1)
    g = np.random.default_rng(h * 1000 + w)
    half = torch.float16 if dtype == "fp16" else torch.bfloat16
    ws = [torch.from_numpy(g.normal(0, (2.0 / (o.cin * o.kh * o.kw)) ** 0.5, o.cout * o.cin * o.kh * o.kw).astype(np.float32)).to(half) for o in ops if o.op in (T.CONV, T.FC)]
    bs = [torch.from_numpy(g.normal(0, 0.3, o.cout).astype(np.float32)) for o in ops if o.op in (T.CONV, T.FC)]
    wb = torch.cat(ws).view(torch.uint8)
    blob = torch.cat([wb, torch.zeros(-wb.numel() % 4, dtype=torch.uint8), torch.cat(bs).view(torch.uint8)]).pin_memory()
    x = torch.from_numpy(g.normal(0, 1, (batch, cin, h, w)).astype(np.float32)).pin_memory()
    one, joined, plan = logits(ctx, ops, cin, h, w, batch, dtype, False, blob, x)
    apart, none, _ = logits(ctx, ops, cin, h, w, batch, dtype, True, blob, x)
    assert joined == ([0] if head == "3x3" else [0, 2]) and none == []
    assert n1 == 0 or plan[2]["fused_op"] == 2
    assert np.isfinite(one).all() and np.abs(one).max() > 0 and np.array_equal(one, apart)
