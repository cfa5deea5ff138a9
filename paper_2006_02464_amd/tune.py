"""The cost model behind the convolution plan (a development tool; its sweep needs an MI355X).

``sweep`` times every convolution of a set of networks, image sizes and batch sizes on every tile shape and
split-K factor, inside whole EXECs (each launch finds the caches as the launches before it leave them), from the start
of a launch's first workgroup to that of the next launch: the stamps of a library built for it (`python -m
paper_2006_02464_amd.build stamps`).  A pair of events around a launch sees nothing below 4.2 us, where more than half of
a batch-1 plan's launches are.  ``fit`` turns those times into csrc/plan_cost.inc: per tile shape a
non-negative linear model of the launch's time in the quantities of :func:`features`, least squares of the relative
error.  The plan compiler evaluates the same model for every convolution it plans and takes the
cheapest tile (plan.cpp: pick_conv_tile), so any image and batch size is planned the same way; nothing is
tuned when EXEC runs.

  python -m paper_2006_02464_amd.tune sweep FILE.jsonl [FAMILY:HxW:BATCH ...]
  python -m paper_2006_02464_amd.tune fit FILE.jsonl [FILE.jsonl ...]
"""
import collections
import json
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
COST = os.path.join(HERE, "csrc", "plan_cost.inc")
# pixels and channels per workgroup and K slice of every tile shape, by its number in the library
TILES = {0: (128, 128, 64), 1: (128, 64, 64), 2: (64, 64, 64), 3: (64, 32, 64), 4: (32, 64, 64), 5: (32, 32, 64), 8: (256, 64, 64),
         9: (128, 128, 64), 10: (128, 64, 128), 11: (64, 64, 128), 12: (64, 32, 128), 13: (32, 64, 128), 14: (32, 32, 128),
         15: (128, 64, 128), 16: (64, 64, 128), 17: (64, 64, 128), 18: (64, 32, 128), 19: (32, 64, 128), 20: (32, 32, 128),
         21: (32, 32, 128), 22: (128, 64, 64), 23: (64, 64, 64), 24: (32, 32, 64), 25: (256, 128, 64), 26: (128, 256, 64),
         27: (256, 256, 64), 28: (256, 128, 64), 29: (32, 32, 256), 30: (32, 32, 256), 31: (64, 32, 256), 32: (64, 32, 256),
         33: (32, 64, 256), 34: (32, 64, 256), 35: (64, 64, 256), 36: (16, 16, 128), 37: (32, 16, 128), 38: (16, 32, 128),
         39: (16, 16, 256), 40: (32, 16, 256)}
SPLIT_TILES = (1, 2, 4, 10, 15, 16, 18, 19, 20, 24, 29, 31, 33, 35, 36, 37, 38, 39, 40)
SPLITS = (1, 2, 4, 8)
LAUNCH_US = 1.2   # from one launch's last store to the next one's first workgroup
PLAIN, STAGED, STEM = 0, 1, 2   # kinds of launch: the main kernel, the register-staged one, the first convolution's form
CONFIGS = (["resnet50:224x224:%d" % b for b in (1, 2, 3, 4, 8, 12, 16)] + ["resnet50:193x161:%d" % b for b in (1, 3, 7)] +
           ["resnet50:97x97:%d" % b for b in (1, 4, 11)] + ["resnet50:160x140:9", "resnet50:64x64:2", "resnet50:210x80:6"] +
           ["resnet18:224x224:%d" % b for b in (1, 3, 8, 16)] + ["resnet18:64x64:%d" % b for b in (1, 4, 16)] + ["resnet18:131x180:5"] +
           ["mobilenet:224x224:%d" % b for b in (1, 4, 16)] + ["mobilenet:150x99:3", "mobilenet:64x100:9"] +
           ["densenet:224x224:%d" % b for b in (1, 6, 16)] + ["densenet:111x150:2", "densenet:80x80:7"] +
           ["inception:224x224:%d" % b for b in (1, 4)] + ["inception:127x127:5", "inception:75x140:2"])


def gemm_form(kh, kw, stride, cin):
    return kh == kw == stride == 1 and cin % 32 == 0


def features(M, N, K, kh, kw, stride, cin, res, cls, tile, split):
    """What the time of a launch is taken to be linear in; the same list as in plan.cpp (conv_cost)."""
    bm, bn, bk = TILES[tile]
    if cls == STAGED:
        bk = 32
    elif cls == STEM:
        bk, K, cin = 64, (kh + 1) // 2 * 64, 4   # a slice is two filter rows of the packed filter
    elif cin % bk and not (gemm_form(kh, kw, stride, cin) and cin > 2 * bk and tile in (10, 11)):
        bk = 64
    slices = -(-K // bk)
    per = -(-slices // split)                        # K slices a workgroup walks
    wgs = -(-M // bm) * -(-N // bn) * split
    more = wgs / 256.0 - 1                           # further workgroups per CU: between the exact and the rounded-up count
    more = max(0.0, more if wgs > 2048 else 0.5 * (max(0.0, more) + -(-wgs // 256) - 1))
    taps = float(kh * kw > 1 or stride > 1)          # general addressing
    out_mb = M * N * 2e-6 * (1 + res)
    in_mb = M * cin * 2e-6 * (stride * stride if kh > 1 else 1) + N * K * 2e-6
    f = [1.0, taps, per, per * taps, per * more, more, out_mb, in_mb]
    return f + ([1.0, split * M * N * 4e-6, float(split)] if split > 1 else [0.0, 0.0, 0.0])


N_FEATURES = 11


def nnls(A, y, sweeps=4000):
    """Least squares with non-negative coefficients, by coordinate descent."""
    G, b, x = A.T @ A, A.T @ y, np.zeros(A.shape[1])
    for _ in range(sweeps):
        for k in range(len(x)):
            if G[k, k] > 0:
                x[k] = max(0.0, x[k] + (b[k] - G[k] @ x) / G[k, k])
    return x


def sweep(path, configs):
    import ctypes

    import torch

    from . import binding, build, measure
    from .binding import Context
    binding.LIB_PATH = build.STAMPED_LIB
    stamps = ctypes.CDLL(binding.lib()._name)
    assert stamps.cw_stamps_reset() == 0

    def times(convs):
        """Microseconds of the launches since the last reset, up to the first workgroup of the next one where that is stamped too."""
        ends = []
        for i, l in enumerate(convs):
            t = np.zeros((min(16384, l["grid_x"] * l["grid_y"] * l["grid_z"]), 2), np.uint64)
            assert stamps.cw_stamps_read(i, len(t), ctypes.c_void_p(t.ctypes.data)) == 0 and t.all()
            ends.append((t[:, 0].min() / 100.0, t[:, 1].max() / 100.0))
        return [ends[i + 1][0] - ends[i][0] if i + 1 < len(convs) and convs[i + 1]["index"] == l["index"] + 1 else ends[i][1] - ends[i][0] + LAUNCH_US
                for i, l in enumerate(convs)]

    lists = {"mobilenet": measure.mobilenet_ops, "densenet": measure.dense_ops, "inception": measure.inception_ops}
    with open(path, "w") as out:
        for cfg in configs:
            family, hw, batch = cfg.split(":")
            h, w = (int(v) for v in hw.split("x"))
            batch = int(batch)
            ctx = Context(workspace_bytes=1 << 30, io_bytes=64 << 20, weight_pool_bytes=256 << 20, load_staging_bytes=128 << 20)
            if family.startswith("resnet"):
                ops = ctx.model_get_ops(ctx.model_define_resnet(int(family[6:]), h, w))
            else:
                ops = lists[family]()
            ctx.set_use_graphs(0)
            blob = None
            x = torch.randn(batch, 3, h, w).half().float().pin_memory()
            stream = torch.cuda.current_stream()
            for tile in TILES:
                for split in SPLITS if tile in SPLIT_TILES else (1,):
                    ctx.set_plan_override(tile, split)
                    mid = ctx.model_define(ops, 3, h, w, batch_sizes=(batch,))
                    if blob is None:   # seeded random weights: with zeros the clocks sit higher, not equally for every tile
                        from .runner import pinned_like
                        blob = pinned_like(measure.resnet_blob(ctx, mid, 0, "fp16"))
                    ctx.load_weights(mid, blob, stream)
                    slot = ctx.input(mid, batch, x, stream)
                    convs = [dict(l, index=i) for i, l in enumerate(ctx.plan(mid, batch)) if l["kind"] == 1 and l["tile_k"] >= 64]   # the main kernel's
                    us = []
                    for _ in range(7):
                        ctx.exec(mid, batch, slot, stream)
                        assert stamps.cw_stamps_reset() == 0
                        ctx.exec(mid, batch, slot, stream)
                        torch.cuda.synchronize()
                        us.append(times(convs))
                    ctx.release(slot)
                    ctx.unload_weights(mid)
                    for l, t in zip(convs, np.median(us, axis=0)):
                        if l["pair_op"] < 0 and l["fused_op"] < 0:
                            o = ops[l["op_index"]]
                            out.write(json.dumps(dict(M=l["gemm_m"], N=l["gemm_n"], K=l["gemm_k"], kh=o[3], kw=o[4], stride=o[5], cin=o[1],
                                                      res=int(o[8] >= 0), stem=int(l["op_index"] == 0), tile=l["conv_tile"],
                                                      split=l["split_k"], us=float(t))) + "\n")
            ctx.destroy()
            print(cfg, flush=True)


def load(paths):
    """{(shape, kind): {(tile, split): us}}, medians over the launches of equal shape."""
    acc = collections.defaultdict(list)
    for path in paths:
        for line in open(path):
            r = json.loads(line)
            cls = (STEM if r["stride"] % 2 == 0 else None) if r["stem"] else (PLAIN if r["cin"] % 64 == 0 or gemm_form(r["kh"], r["kw"], r["stride"], r["cin"]) else STAGED)
            if cls is not None and not (cls == STEM and r["tile"] in (23, 24)):   # a first convolution has no wave groups
                acc[(tuple(r[k] for k in ("M", "N", "K", "kh", "kw", "stride", "cin", "res")), cls), r["tile"], r["split"]].append(r["us"])
    shapes = collections.defaultdict(dict)
    for (shape, tile, split), v in acc.items():
        shapes[shape][tile, split] = float(np.median(v))
    return shapes


def fit(paths):
    shapes = load(paths)
    groups = collections.defaultdict(list)
    for (shape, cls), times in shapes.items():
        for (tile, split), us in times.items():
            groups[cls, tile].append((features(*shape, cls, tile, split), us, split))
    coef = {}
    kept = [l.rstrip() for l in open(COST) if l.startswith("{") and int(l[1]) not in {cls for cls, _ in groups}]   # no such launch in the files
    lines = ["// Generated by tune.py from launch times measured on an MI355X: per kind of launch (COST_*) and tile",
             "// shape the microseconds per unit of each feature (conv_cost in plan.cpp).",
             "// {kind, tile, K may be split, {1, general addressing, K slices, of these with general addressing, slices of",
             "//  further workgroups on a CU, further workgroups, MB out, MB in, split, MB of partial sums, splits}}"]
    for (cls, tile), rows in sorted(groups.items()):
        A, y = np.array([r[0] for r in rows]), np.array([r[1] for r in rows])
        coef[cls, tile] = c = nnls(A / y[:, None], np.ones(len(y)))
        splits = int(any(r[2] > 1 for r in rows))
        lines.append("{%d, %d, %d, {%s}}," % (cls, tile, splits, ", ".join("%.4gf" % v if "." in "%.4g" % v or "e" in "%.4g" % v else "%.4g.f" % v for v in c)))
        print("kind %d tile %2d: %4d launches, rms relative error %.3f" % (cls, tile, len(y), np.sqrt((((A @ c) / y - 1) ** 2).mean())))
    lines += kept
    best = chosen = 0.0
    for (shape, cls), times in shapes.items():
        best += min(times.values())
        chosen += times[min(times, key=lambda ts: float(np.dot(features(*shape, cls, *ts), coef[cls, ts[0]])))]
    print("%d shapes: fastest of each %.1f us, as the model chooses %.1f us" % (len(shapes), best, chosen))
    with open(COST, "w") as f:
        f.write("\n".join(lines) + "\n")


if __name__ == "__main__":
    if len(sys.argv) < 3 or sys.argv[1] not in ("sweep", "fit"):
        sys.exit(__doc__)
    if sys.argv[1] == "sweep":
        sweep(sys.argv[2], sys.argv[3:] or CONFIGS)
    else:
        fit(sys.argv[2:])
