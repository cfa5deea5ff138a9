"""What the worker is measured on: passes through its public entry points, over the range of models, batch sizes,
image sizes, storage types and call forms that its users have it run.

A case names
  model, dtype, batch, h, w   the network (the families of the test-suite and the benchmark), its storage type (ResNet-152
                              runs in bf16, the others in either), and the request's shape;
  call                        how the request arrives:
    "device"  inputs and results in device memory, as a caller has them that produces its images on the GPU:
              Context.exec_static;
    "host"    an INFER action, images and results in pinned host memory: input, exec and output, each on a stream of
              its own as the worker's executors issue them;
    "cold"    an INFER of a model that is not resident: load_weights from pinned host memory, exec_static,
              unload_weights.

Weights are He-normal, with the last convolution of every residual branch scaled down by the number of branches and the
classifier to logits of a few units: activations and logits stay in the range that a trained network with folded
normalisation has.  Images are N(0, 1)."""
import math

import torch

from paper_2006_02464_amd.binding import Context

MIB = 1 << 20
CONV, MAXPOOL, GAVGPOOL, FC, SOFTMAX, CONCAT = 0, 1, 2, 3, 4, 5
CLASSES = 1000
MODELS = ("resnet18", "resnet50", "resnet152", "mobilenet", "densenet", "inception")
SMALLEST, LARGEST, MOST_IMAGES = 64, 224, 16


# ---- the networks, as operator lists for Context.model_define -------------------------------------
class _Net:
    def __init__(self):
        self.ops = []

    def add(self, *row):
        self.ops.append(row)
        return len(self.ops) - 1

    def conv(self, src, cin, cout, k=1, stride=1, act=1, res=-1, kw=None, depthwise=False):
        kw = k if kw is None else kw
        return self.add(CONV, cin, cout, k, kw, stride, k // 2, act, res, src, 0 if kw == k else kw // 2, cin if depthwise else 0)

    def maxpool(self, src, c, k, stride, pad):
        return self.add(MAXPOOL, c, c, k, k, stride, pad, 0, -1, src, 0, 0)

    def concat(self, a, b, ca, cb):
        return self.add(CONCAT, ca, ca + cb, 0, 0, 1, 0, 0, b, a, 0, 0)

    def head(self, src, c):
        g = self.add(GAVGPOOL, c, c, 0, 0, 1, 0, 0, -1, src, 0, 0)
        f = self.add(FC, c, CLASSES, 1, 1, 1, 0, 0, -1, g, 0, 0)
        self.add(SOFTMAX, CLASSES, CLASSES, 0, 0, 1, 0, 0, -1, f, 0, 0)
        return self.ops


def _resnet(depth):
    n, blocks = _Net(), {18: (2, 2, 2, 2), 50: (3, 4, 6, 3), 152: (3, 8, 36, 3)}[depth]
    cur, cin = n.maxpool(n.conv(-1, 3, 64, 7, 2), 64, 3, 2, 1), 64
    for stage, count in enumerate(blocks):
        width = 64 << stage
        cout = width if depth == 18 else 4 * width
        for b in range(count):
            stride, x = (2 if b == 0 and stage else 1), cur
            t = n.conv(x, cin, width, 3, stride) if depth == 18 else n.conv(n.conv(x, cin, width), width, width, 3, stride)
            short = n.conv(x, cin, cout, 1, stride, act=0) if stride != 1 or cin != cout else x
            cur = n.conv(t, width, cout, 3 if depth == 18 else 1, res=short)
            cin = cout
    return n.head(cur, cin)


def _mobilenet():
    n = _Net()
    cur, cin = n.conv(-1, 3, 32, 3, 2), 32
    plan = [(64, 1), (128, 2), (128, 1), (256, 2), (256, 1), (512, 2)] + [(512, 1)] * 5 + [(1024, 2), (1024, 1)]
    for i, (cout, stride) in enumerate(plan):
        act = 2 if i >= 7 else 1          # hard swish in the later blocks
        d = n.conv(cur, cin, cin, 3, stride, act, depthwise=True)
        cur = n.conv(d, cin, cout, act=act, res=cur if stride == 1 and cin == cout else -1)
        cin = cout
    return n.head(cur, cin)


def _densenet():
    n, c = _Net(), 64
    cur = n.maxpool(n.conv(-1, 3, 64, 7, 2), 64, 3, 2, 1)
    for block, layers in enumerate((6, 12)):
        if block:
            c //= 2
            cur = n.maxpool(n.conv(cur, 2 * c, c), c, 2, 2, 0)
        for _ in range(layers):
            t = n.conv(n.conv(cur, c, 128), 128, 32, 3)
            cur = n.concat(cur, t, c, 32)
            c += 32
    return n.head(cur, c)


def _inception():
    n = _Net()
    x = n.conv(n.conv(-1, 3, 32, 3, 2), 32, 256, 3, 2)
    for _ in range(2):
        a, b = n.conv(x, 256, 256), n.conv(x, 256, 256)
        b = n.conv(n.conv(b, 256, 256, 1, kw=7), 256, 256, 7, kw=1)
        x = n.conv(n.concat(a, b, 256, 256), 512, 256, res=x)
    return n.head(x, 256)


def _ops(model):
    return _resnet(int(model[6:])) if model.startswith("resnet") else {"mobilenet": _mobilenet, "densenet": _densenet, "inception": _inception}[model]()


def _shapes(ops, h, w):
    """Height and width of every operator's output."""
    out = []
    for op, _, _, kh, kw, stride, pad, _, _, src, pad_w, _ in ops:
        ih, iw = (h, w) if src < 0 else out[src]
        if op in (CONV, MAXPOOL):
            pw = pad if kh == kw else pad_w
            out.append(((ih + 2 * pad - kh) // stride + 1, (iw + 2 * pw - kw) // stride + 1))
        else:
            out.append((ih, iw) if op == CONCAT else (1, 1))
    return out


# ---- the cases -------------------------------------------------------------------------------------
def listed():
    def case(name, model, dtype, batch, h, w, call):
        return {"name": name, "model": model, "dtype": dtype, "batch": batch, "h": h, "w": w, "call": call}

    return [
        # the smallest request: one thumbnail through the smallest ResNet
        case("resnet18-64-b1-host", "resnet18", "fp16", 1, 64, 64, "host"),
        # the benchmark's network: the latency of one image, the usual small batch, the throughput batch
        case("resnet50-b1-device", "resnet50", "fp16", 1, 224, 224, "device"),
        case("resnet50-b4-host", "resnet50", "fp16", 4, 224, 224, "host"),
        case("resnet50-b16-device", "resnet50", "fp16", 16, 224, 224, "device"),
        # whatever a queue held when its deadline came: an odd batch of odd-sized crops
        case("resnet50-193x161-b3-device", "resnet50", "bf16", 3, 193, 161, "device"),
        # a request for a model that has to be brought in first
        case("resnet50-b1-cold", "resnet50", "fp16", 1, 224, 224, "cold"),
        # the plain 3x3 network at its full image size and a large batch
        case("resnet18-b8-device", "resnet18", "bf16", 8, 224, 224, "device"),
        # the deepest network, the largest request
        case("resnet152-b16-device", "resnet152", "bf16", 16, 224, 224, "device"),
        # the other families: depthwise-separable, densely connected, factorised filters
        case("mobilenet-b1-device", "mobilenet", "fp16", 1, 224, 224, "device"),
        case("mobilenet-b16-host", "mobilenet", "fp16", 16, 224, 224, "host"),
        case("densenet-b6-device", "densenet", "fp16", 6, 224, 224, "device"),
        case("inception-127-b5-host", "inception", "fp16", 5, 127, 127, "host"),
    ]


def draw(rng):
    def side():
        return rng.randint(SMALLEST, LARGEST)

    def spread(most):
        return min(most, int(math.exp(rng.uniform(0.0, math.log(most + 1.0)))))

    model = rng.choice(MODELS)
    dtype = "bf16" if model == "resnet152" else rng.choice(("fp16", "fp16", "bf16"))
    h = side()
    w = h if rng.random() < 0.5 else side()
    call = rng.choice(("device", "device", "device", "host", "host", "cold"))
    # the arena of exec_static holds what a batch of 8 of the widest family needs
    most = 8 if model == "inception" and call != "host" else MOST_IMAGES
    return {"model": model, "dtype": dtype, "batch": spread(most), "h": h, "w": w, "call": call}


# ---- one user's program ----------------------------------------------------------------------------
_streams = []


def _worker_streams():
    """The worker's streams for INPUT, EXEC and OUTPUT: one set per process, as one worker has."""
    if not _streams:
        _streams.extend(torch.cuda.Stream() for _ in range(3))
    return _streams


def _blob(ops, dtype, seed):
    """The canonical weight blob: every W[cout][cin][kh][kw] in the storage type, then (from a multiple of 4 bytes on)
    every bias in fp32."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    half = torch.float16 if dtype == "fp16" else torch.bfloat16
    branches = max(1, sum(o[0] == CONV and o[8] >= 0 for o in ops))
    weights, biases = [], []
    for o in ops:
        if o[0] not in (CONV, FC):
            continue
        cin = o[1] // max(1, o[11])
        std = math.sqrt(2.0 / (cin * o[3] * o[4])) * (0.3 if o[0] == FC else branches ** -0.5 if o[8] >= 0 else 1.0)
        n = o[2] * cin * o[3] * o[4]
        weights.append((torch.randn(n, generator=g, device="cuda") * std).to(half))
        biases.append(torch.randn(o[2], generator=g, device="cuda") * 0.1)
    w = torch.cat(weights).view(torch.uint8)
    pad = torch.zeros(-w.numel() % 4, dtype=torch.uint8, device="cuda")
    return torch.cat([w, pad, torch.cat(biases).view(torch.uint8)])


class _Request:
    """A context with one model, and the buffers of one request."""

    def __init__(self, case, seed):
        self.call, self.batch = case["call"], case["batch"]
        ops = _ops(case["model"])
        nbytes = 4 * 3 * self.batch * case["h"] * case["w"]
        blob = _blob(ops, case["dtype"], seed)
        self.blob = torch.empty(blob.numel(), dtype=torch.uint8, pin_memory=True)
        self.blob.copy_(blob)
        pool = 32 * MIB + blob.numel() * 5 // 4
        self.ctx = Context(workspace_bytes=320 * MIB, io_bytes=4 * MIB + 4 * nbytes, weight_pool_bytes=(pool // (16 * MIB) + 1) * 16 * MIB,
                           load_staging_bytes=blob.numel() + MIB)
        self.model = self.ctx.model_define(ops, 3, case["h"], case["w"], batch_sizes=(self.batch,), dtype=case["dtype"])
        half = torch.float16 if case["dtype"] == "fp16" else torch.bfloat16
        g = torch.Generator(device="cuda").manual_seed(seed + 1)
        x = torch.randn(self.batch, 3, case["h"], case["w"], generator=g, device="cuda").to(half).float()
        if self.call == "host":
            self.x = torch.empty(x.shape, dtype=torch.float32, pin_memory=True)
            self.x.copy_(x)
            where = {"pin_memory": True}
        else:
            self.x = x
            where = {"device": "cuda"}
        self.logits = torch.zeros(self.batch, CLASSES, dtype=torch.float32, **where)
        self.probs = torch.zeros(self.batch, CLASSES, dtype=torch.float32, **where)
        if self.call != "cold":
            self.ctx.load_weights(self.model, self.blob, torch.cuda.current_stream())
        torch.cuda.synchronize()


def prepare(case, seed):
    return _Request(case, seed)


def run(s):
    if s.call == "host":
        inp, exe, out = _worker_streams()
        slot = s.ctx.input(s.model, s.batch, s.x, inp)
        s.ctx.exec(s.model, s.batch, slot, exe)
        s.ctx.output(slot, s.probs, s.logits, out)
    else:
        stream = torch.cuda.current_stream()
        if s.call == "cold":
            s.ctx.load_weights(s.model, s.blob, stream)
        s.ctx.exec_static(s.model, s.batch, s.x, s.logits, s.probs, stream)
        if s.call == "cold":
            s.ctx.unload_weights(s.model)
    return {"logits": s.logits, "probs": s.probs}


# ---- what a pass cannot do without -----------------------------------------------------------------
def work(case):
    """Bytes: the images, the weights and the results once each.  Operations: the multiply-accumulates of every
    convolution and of the fully connected layer."""
    ops, batch = _ops(case["model"]), case["batch"]
    flops = weights = biases = 0
    for o, (h, w) in zip(ops, _shapes(ops, case["h"], case["w"])):
        if o[0] in (CONV, FC):
            n = o[2] * (o[1] // max(1, o[11])) * o[3] * o[4]
            flops += 2 * batch * h * w * n
            weights += 2 * n
            biases += 4 * o[2]
    return {"bytes": 4 * batch * (3 * case["h"] * case["w"] + 2 * CLASSES) + weights + biases, "flops": flops}


def tolerance(case):
    """Every layer rounds its activations to the storage type once, so two correct summation orders drift apart by a few
    units in the last place (2^-11 in fp16, 2^-8 in bf16) over the depth of the network."""
    return {"rel": 2e-3, "max": 2e-2} if case["dtype"] == "fp16" else {"rel": 1.5e-2, "max": 1.5e-1}
