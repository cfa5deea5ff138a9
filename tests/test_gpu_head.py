"""Input cast, first convolution, max pool and the 1x1 behind it as one launch, against the plan that debug retention makes:
the same launches for everything behind the head, cast, convolution and pool as launches of their own (which other tests hold
against the CPU oracle layer by layer).  Every tensor is rounded at the same places and K runs in the same order: same bits."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

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


def logits(ctx, ops, cin, h, w, batch, dtype, keep, blob, x, classes=40):
    ctx.set_debug_keep(keep)
    try:
        m = ctx.model_define([tuple(o) for o in ops], cin, h, w, batch_sizes=(batch,), dtype=dtype)
    finally:
        ctx.set_debug_keep(False)
    plan = ctx.plan(m, batch)
    joined = [i for i in range(len(plan)) if ctx.plan_launch_joined(m, batch, i)]
    st = torch.cuda.current_stream()
    ctx.load_weights(m, blob, st)
    out, probs = (torch.zeros(batch, classes).pin_memory() for _ in range(2))
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


def head_reference(head, w, b, x, act, n1, half):
    """Mean over the map of every channel that net_of_identities() shows, in 64 bits but for the roundings of stored tensors."""
    relu = lambda t: torch.where(t > 0, t, torch.zeros_like(t))          # of NaN: 0, as fmaxf has it
    rnd = lambda t: t.float().to(half).double()
    conv = lambda t, i, stride=1: F.conv2d(t, w[i].double(), b[i].double(), stride)
    k, taps = (7, 8) if head == "7x7" else (3, 4)                        # a filter row is padded with weights of zero
    w = [F.pad(w[0], (0, taps - k))] + w[1:]
    p = k // 2
    c = conv(F.pad(x.to(half).double(), (p, p + taps - k, p, p)), 0, 2)
    y = rnd(relu(c) if act else c)
    if head == "7x7":
        y = F.max_pool2d(torch.where(y.isnan(), torch.full_like(y, -np.inf), y), 3, 2, 1)
    if n1:
        y1 = conv(y, 1)
        y1 = rnd(relu(y1) if act else y1)
        t = rnd(relu(conv(y1, 3) + rnd(relu(conv(y, 2)))))
    else:
        t = rnd(relu(conv(y, 1)))
    m = t.mean((2, 3))
    m[~m.isfinite().all(1)] = np.nan                                     # the FC multiplies every mean by every weight, most of them 0
    return m.numpy()


def net_of_identities(head, cin, act, n1):
    """The head and, behind it, 1x1 convolutions that carry every value it stores to a channel of its own, whose mean is a logit."""
    ops = [O(T.CONV, cin, 32, 3, 3, 2, 1, act, -1, -1)] if head == "3x3" else [O(T.CONV, cin, 64, 7, 7, 2, 3, act, -1, -1), O(T.MAXPOOL, 64, 64, 3, 3, 2, 1, 0, -1, 0)]
    y, c = len(ops) - 1, ops[0].cout
    if n1:
        # (with a second reader of y1, or the first 1x1 and the last were one launch instead)
        ops += [O(T.CONV, 64, n1, 1, 1, 1, 0, act, -1, y), O(T.CONV, 64, 256, 1, 1, 1, 0, 1, -1, y), O(T.MAXPOOL, n1, n1, 1, 1, 1, 0, 0, -1, y + 1),
                O(T.CONV, n1, 256, 1, 1, 1, 0, 1, y + 2, y + 1)]
    else:
        ops += [O(T.CONV, c, 256, 1, 1, 1, 0, 1, -1, y)]
    k = len(ops) - 1
    return ops + [O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, k), O(T.FC, 256, 256, 1, 1, 1, 0, 0, -1, k + 1), O(T.SOFTMAX, 256, 256, 0, 0, 1, 0, 0, -1, k + 2)]


# Small whole numbers: every sum is exact in fp32, whatever its order.  One image of each kind: plain; NaN; infinities inside and at
# the edges; what overflows the storage type when it is read and when it is stored; its smallest values; single pixels.
@pytest.mark.parametrize("head,cin,act,n1,h,w,dtype", [
    ("7x7", 3, 1, 64, 97, 97, "fp16"), ("7x7", 3, 0, 128, 97, 101, "bf16"), ("7x7", 2, 0, 64, 100, 98, "fp16"), ("7x7", 4, 0, 0, 61, 53, "fp16"),
    ("7x7", 1, 1, 0, 30, 223, "bf16"), ("7x7", 3, 0, 0, 130, 140, "fp16"), ("3x3", 3, 1, 0, 45, 67, "fp16"), ("3x3", 4, 0, 0, 33, 32, "bf16"),
])
def test_head_stores_what_64_bit_arithmetic_gives(ctx, head, cin, act, n1, h, w, dtype):
    half, batch = torch.float16 if dtype == "fp16" else torch.bfloat16, 12
    ops = net_of_identities(head, cin, act, n1)
    g = np.random.default_rng(h + w)
    ws, bs = [], []
    for i, o in enumerate(o for o in ops if o.op in (T.CONV, T.FC)):
        if i == 0 or (n1 and i == 1):
            ws.append(g.integers(-1, 2, (o.cout, o.cin, o.kh, o.kw)) * (g.random((o.cout, o.cin, o.kh, o.kw)) < 0.3))
            bs.append(g.integers(-3, 4, o.cout))
        else:   # channel c to channel c, the 1x1's to 64 + c
            ws.append(np.eye(o.cout, o.cin, -64 if n1 and i == 3 else 0).reshape(o.cout, o.cin, 1, 1))
            bs.append(np.zeros(o.cout))
    ws, bs = [torch.tensor(v, dtype=torch.float32) for v in ws], [torch.tensor(v, dtype=torch.float32) for v in bs]
    wb = torch.cat([v.flatten() for v in ws]).to(half).view(torch.uint8)
    blob = torch.cat([wb, torch.zeros(-wb.numel() % 4, dtype=torch.uint8), torch.cat(bs).view(torch.uint8)]).pin_memory()
    x = g.integers(-8, 9, (batch, cin, h, w)).astype(np.float32)
    x[1, 0, h // 2, w // 3] = np.nan
    x[2, cin - 1, h // 3, w // 2] = np.inf
    x[3, 0, 0, 0], x[3, 0, h - 1, w - 1] = -np.inf, np.inf
    x[4, 0, 5, 6], x[4, cin - 1, h - 4, 9] = 70000.0, -3.4e38       # above fp16's range; above both
    x[5][g.random(x[5].shape) < 0.05] = 30000.0                     # in the range, sums of them are not
    x[6] *= 2.0 ** -24                                              # fp16's smallest
    x[7], x[8] = 0, 0
    x[7, 0, h - 1, w - 1], x[8, cin - 1, g.integers(h), g.integers(w)] = 5, 7
    x = torch.from_numpy(x)
    one, joined, plan = logits(ctx, ops, cin, h, w, batch, dtype, False, blob, x.pin_memory(), 256)
    assert joined == ([0] if head == "3x3" else [0, 2]) and (n1 == 0 or plan[2]["fused_op"] == 2)
    ref = head_reference(head, ws, bs, x, act, n1, half)
    assert np.isfinite(ref).all(1).sum() >= 9
    # the pool's fp32 sum over non-negative values and, in bf16, the 16 bits that the FC takes of a mean
    assert np.allclose(one, ref, rtol=2e-6 if dtype == "fp16" else 1e-5, atol=1e-7, equal_nan=True), np.nanmax(np.abs(one - ref))
