"""Helpers of the GPU parity tests: the same seeded tensors go to the oracle (as
float32 arrays) and to the library (as the canonical blob)."""
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np

from oracle import network as N
from oracle import topology as T
from workload import gen

TOL = 2e-2   # max |z_gpu - z_ref| / max |z_ref| per sample


class Case:
    def __init__(self, ops, in_hw, seed, dtype="fp16", dist="normal", weight_gain=None):
        self.ops = ops
        self.hw = in_hw
        self.seed = seed
        self.dtype = dtype
        self.dist = dist
        self.w, self.b = gen.model_tensors(T.weight_shapes(ops), seed, dtype, weight_gain)
        self.blob = gen.pack_blob(self.w, self.b, dtype)

    def images(self, first, count):
        return gen.images(self.seed, first, count, 3, self.hw, self.hw, self.dist, self.dtype)

    def oracle(self, x, keep="final", threads=None, storage=None):
        return N.forward(self.ops, self.w, self.b, x, prec="f32", threads=threads, keep=keep,
                         storage=storage)


def rel_err_per_sample(z_gpu, z_ref):
    """max_j |z_gpu - z_ref| / max_j |z_ref| for every sample."""
    return np.abs(z_gpu - z_ref).max(axis=1) / np.abs(z_ref).max(axis=1)


def top2_gap(z):
    s = np.sort(z, axis=1)
    return s[:, -1] - s[:, -2]


def check_layers(ctx, ops, w, b, mid, batch, x, dtype, unstored=(), unrounded=(), given=()):
    """Every convolution output that an EXEC over `x` stored, each against the oracle on the tensors that its launch read (debug retention).  The outputs of
    `unstored` stay in a launch: the oracle computes them on the way, rounded to the storage type but for those of `unrounded`, and the library must refuse to
    read them back.  NaN and infinities have to be where the oracle has them."""
    shapes = T.shapes(ops, x.shape[2], x.shape[3])
    of = {i: k for k, i in enumerate(i for i, o in enumerate(ops) if o.op in (T.CONV, T.FC))}
    threads = ThreadPoolExecutor(max_workers=min(16, len(os.sched_getaffinity(0))))
    values = {-1: x}

    def conv(i):
        o, k = ops[i], of[i]
        ph, pw, groups = T.conv_geometry(o)

        def one(s):
            return N.conv2d(s, w[k], b[k], o.stride, o.pad) if groups == 1 and o.kh == o.kw else N.conv2d_grouped(s, w[k], b[k], o.stride, ph, pw, groups)
        src = values[o.input_from]
        y = np.concatenate(list(threads.map(one, [src[n:n + 1] for n in range(batch)])))
        for ko, _, r, q in np.argwhere(~np.isfinite(w[k])) if groups == 1 else ():   # the matrix cores multiply an infinite tap outside the image by zero
            ih, iw = np.arange(y.shape[2]) * o.stride + r - ph, np.arange(y.shape[3]) * o.stride + q - pw
            y[:, ko, (ih < 0) | (ih >= src.shape[2]), :] = np.nan
            y[:, ko, :, (iw < 0) | (iw >= src.shape[3])] = np.nan
        if o.residual_from >= 0:
            y = N.add(y, values[o.residual_from])
        y = N.relu(y) if o.relu == 1 else N.hswish(y) if o.relu == 2 else y
        return y if i in unrounded else gen.quantize(y, dtype)

    ulp = 2.0 ** -10 if dtype == "fp16" else 2.0 ** -7
    seen = 0
    for i, o in enumerate(ops):
        if o.op in (T.GAVGPOOL, T.FC, T.SOFTMAX):
            break
        if i in unstored:
            try:
                ctx.debug_read_op(mid, batch, i, (batch,) + tuple(shapes[i]))
            except Exception:
                values[i] = conv(i)
                continue
            raise AssertionError("op %d can be read back" % i)
        values[i] = got = ctx.debug_read_op(mid, batch, i, (batch,) + tuple(shapes[i]))
        if i in given:
            continue
        if o.op == T.CONCAT:
            np.testing.assert_array_equal(got, N.concat_channels(values[o.input_from], values[o.residual_from]))
        elif o.op == T.MAXPOOL:
            np.testing.assert_array_equal(got, N.maxpool2d(values[o.input_from], o.kh, o.stride, o.pad))
        else:
            want = conv(i)
            special = ~np.isfinite(want)
            assert np.array_equal(got[special], want[special], equal_nan=True) and np.isfinite(got[~special]).all(), "op %d: NaN or infinite elsewhere" % i
            seen += int(special.sum())
            live = np.abs(want[~special])
            if not live.size:
                continue
            # One rounding, which the order of the sums may shift by a unit.  Where an input was rounded on the way, one of its elements on a rounding
            # boundary may be a unit off and moves the sums over it by that times a weight: 0.3 units of the largest value.
            inside = o.input_from in unstored or o.residual_from in unstored
            diff = np.abs(got[~special] - want[~special])
            bad = diff > ulp * live + (0.3 * ulp if inside else 1e-5) * live.max()
            assert not bad.any(), "op %d: %d of %d elements off, worst %.3e of %.3e" % (i, int(bad.sum()), bad.size, diff.max(), live.max())
            assert (diff > (0.3 * ulp if inside else 1e-5) * live.max()).mean() <= (0.05 if inside else 0.02), "op %d: too many elements off by a unit" % i
    threads.shutdown()
    return seen


def define_retained(ctx, ops, h, w, batch, dtype):
    """The model with debug retention and the launches that it has without."""
    plain = ctx.model_define(ops, 3, h, w, batch_sizes=(batch,), dtype=dtype)
    ctx.set_debug_keep(True, joined=True)
    try:
        mid = ctx.model_define(ops, 3, h, w, batch_sizes=(batch,), dtype=dtype)
    finally:
        ctx.set_debug_keep(False)
    convs = lambda m: [l for l in (ctx.plan_launch_issued(m, batch, i) for i in range(len(ctx.plan(m, batch)))) if l["kind"] in (1, 7) and l["op_index"] > 0]
    assert convs(mid) == convs(plain)
    return mid


def with_infinities(ops, w, at):
    """The weights with infinities at `at` (op: index of its weight), positive and negative in turn."""
    of = {i: k for k, i in enumerate(i for i, o in enumerate(ops) if o.op in (T.CONV, T.FC))}
    out = [v.copy() for v in w]
    for n, (i, where) in enumerate(at.items()):
        out[of[i]][where] = np.inf if n % 2 == 0 else -np.inf
    return out
