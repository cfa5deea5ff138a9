"""Global average pool and FC as one launch against the plan that debug retention makes, which has the two as launches of their own
(held against the CPU oracle by other tests).  Sums, products and roundings in the same order: same bits."""
import numpy as np
import pytest
import torch

from oracle import topology as T
from test_gpu_head import ctx, O   # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def logits(ctx, c, h, w, out, batch, dtype, keep, blob, x):
    ops = [O(T.CONV, 3, 32, 3, 3, 2, 1, 1, -1, -1), O(T.CONV, 32, c, 1, 1, 1, 0, 0, -1, 0), O(T.GAVGPOOL, c, c, 0, 0, 1, 0, 0, -1, 1),
           O(T.FC, c, out, 1, 1, 1, 0, 0, -1, 2), O(T.SOFTMAX, out, out, 0, 0, 1, 0, 0, -1, 3)]
    ctx.set_debug_keep(keep)
    try:
        m = ctx.model_define([tuple(o) for o in ops], 3, 2 * h, 2 * w, batch_sizes=(batch,), dtype=dtype)
    finally:
        ctx.set_debug_keep(False)
    plan = ctx.plan(m, batch)
    joined = any(ctx.plan_launch_joined(m, batch, i) for i, l in enumerate(plan) if l["kind"] == 4)
    st = torch.cuda.current_stream()
    ctx.load_weights(m, blob, st)
    z, probs = (torch.zeros(batch, out).pin_memory() for _ in range(2))
    slot = ctx.input(m, batch, x, st)
    ctx.exec(m, batch, slot, st)
    ctx.output(slot, probs, z, st)
    torch.cuda.synchronize()
    ctx.unload_weights(m)
    return z.numpy().copy(), joined


# one to four items of 64 channels a wave with maps up to the pixels that the number allows, and beyond: one pixel more, five
# items, channels that do not divide; several samples; part of a tile of outputs
@pytest.mark.parametrize("c,h,w,out,batch,dtype,one", [
    (512, 1, 1, 40, 1, "fp16", True), (512, 2, 4, 1000, 1, "bf16", True), (512, 3, 3, 17, 1, "fp16", True), (512, 7, 7, 1000, 1, "fp16", True), (512, 8, 8, 10, 1, "bf16", True),
    (512, 2, 4, 33, 2, "fp16", True), (1024, 4, 8, 1000, 1, "fp16", True), (512, 3, 5, 40, 2, "bf16", True), (1536, 4, 4, 16, 1, "fp16", True), (1536, 1, 5, 1, 1, "bf16", True),
    (1024, 3, 3, 40, 2, "bf16", True), (512, 2, 4, 1000, 4, "fp16", True), (512, 3, 5, 40, 3, "fp16", True), (2048, 4, 4, 1000, 1, "fp16", True),
    (512, 5, 13, 40, 1, "fp16", False), (1024, 3, 11, 40, 1, "fp16", False), (2048, 1, 17, 40, 1, "fp16", False), (2560, 1, 1, 40, 1, "fp16", False),
    (768, 2, 2, 40, 1, "fp16", False), (512, 1, 1, 40, 5, "fp16", False),
])
def test_pool_and_fc_in_one_launch(ctx, c, h, w, out, batch, dtype, one):   # noqa: F811
    g = np.random.default_rng(c + h * 100 + w)
    half = torch.float16 if dtype == "fp16" else torch.bfloat16
    shapes = [(32, 27), (c, 32), (out, c)]
    wb = torch.cat([torch.from_numpy(g.normal(0, (2.0 / k) ** 0.5, n * k).astype(np.float32)).to(half) for n, k in shapes]).view(torch.uint8)
    bs = torch.cat([torch.from_numpy(g.normal(0, 0.3, n).astype(np.float32)) for n, _ in shapes])
    blob = torch.cat([wb, torch.zeros(-wb.numel() % 4, dtype=torch.uint8), bs.view(torch.uint8)]).pin_memory()
    x = torch.from_numpy(g.normal(0, 1, (batch, 3, 2 * h, 2 * w)).astype(np.float32)).pin_memory()
    a, apart = logits(ctx, c, h, w, out, batch, dtype, True, blob, x)
    b, joined = logits(ctx, c, h, w, out, batch, dtype, False, blob, x)
    assert not apart and joined == one
    assert np.array_equal(a, b) and np.isfinite(a).all() and np.any(a != 0)


@pytest.mark.parametrize("c,h,w,batch,dtype", [(512, 3, 5, 3, "fp16"), (1024, 2, 4, 2, "bf16"), (2048, 4, 4, 1, "fp16")])
def test_pool_and_fc_in_one_launch_with_non_finite_maps(ctx, c, h, w, batch, dtype):   # noqa: F811
    """Maps with NaN, infinities and large values give the logits of the two launches, NaN where they are NaN."""
    g = np.random.default_rng(c)
    half = torch.float16 if dtype == "fp16" else torch.bfloat16
    shapes = [(32, 27), (c, 32), (40, c)]
    wb = torch.cat([torch.from_numpy(g.normal(0, (128.0 if k == 27 else 2.0 / k) ** 0.5, n * k).astype(np.float32)).to(half) for n, k in shapes]).view(torch.uint8)
    bs = torch.cat([torch.from_numpy(g.normal(0, 0.3, n).astype(np.float32)) for n, _ in shapes])
    blob = torch.cat([wb, torch.zeros(-wb.numel() % 4, dtype=torch.uint8), bs.view(torch.uint8)]).pin_memory()
    plain = torch.from_numpy(g.normal(0, 1, (batch, 3, 2 * h, 2 * w)).astype(np.float32))
    # one pixel whose filter sums overflow when they are stored: infinities and, behind the 1x1, NaN in part of the map; all of a
    # sample like that; averages of a large, finite map
    for value, at in ((6e4 if dtype == "fp16" else 3e38, (batch - 1, 1, h, w)), (6e4 if dtype == "fp16" else 3e37, batch - 1), (30.0, batch - 1)):
        x = plain.clone()
        x[at] = value
        a, apart = logits(ctx, c, h, w, 40, batch, dtype, True, blob, x.pin_memory())
        b, joined = logits(ctx, c, h, w, 40, batch, dtype, False, blob, x.pin_memory())
        assert joined and not apart and np.array_equal(a, b, equal_nan=True) and np.isfinite(a[:batch - 1]).all()
        assert np.isfinite(a[batch - 1]).all() == (value == 30.0)


# one to ten chunks of 32 features a wave, part of a tile of outputs and of samples, a second tile of samples; and 2048 features with few samples, apart as they were
@pytest.mark.parametrize("c,out,batch,dtype,parts", [
    (256, 1000, 5, "fp16", True), (768, 17, 1, "bf16", True), (1024, 1024, 17, "fp16", True), (2048, 1000, 8, "bf16", True), (2560, 40, 16, "fp16", True), (2048, 1000, 7, "fp16", False),
])
def test_fc_in_parts_for_the_softmax(ctx, c, out, batch, dtype, parts):   # noqa: F811
    """The FC's eight parts of K added up by the softmax against the sum inside the FC's launch, in the same order: same bits."""
    g = np.random.default_rng(c + out)
    half = torch.float16 if dtype == "fp16" else torch.bfloat16
    shapes = [(32, 27), (c, 32), (out, c)]
    wb = torch.cat([torch.from_numpy(g.normal(0, (2.0 / k) ** 0.5, n * k).astype(np.float32)).to(half) for n, k in shapes]).view(torch.uint8)
    bs = torch.cat([torch.from_numpy(g.normal(0, 0.3, n).astype(np.float32)) for n, _ in shapes])
    blob = torch.cat([wb, torch.zeros(-wb.numel() % 4, dtype=torch.uint8), bs.view(torch.uint8)]).pin_memory()
    x = torch.from_numpy(g.normal(0, 1, (batch, 3, 18, 18)).astype(np.float32)).pin_memory()
    x[0, 0, 4, 4] = float("inf")
    a, _ = logits(ctx, c, 9, 9, out, batch, dtype, True, blob, x)
    fc = []
    define = ctx.model_define
    ctx.model_define = lambda *args, **kw: fc.append(define(*args, **kw)) or fc[0]
    try:
        b, joined = logits(ctx, c, 9, 9, out, batch, dtype, False, blob, x)
    finally:
        del ctx.model_define
    assert not joined and [l["grid_z"] for l in ctx.plan(fc[0], batch) if l["name"] == "fc"] == [8 if parts else 1]
    assert np.array_equal(a, b, equal_nan=True) and np.isfinite(a[1:]).all() and not np.isfinite(a[0]).all()
