"""INPUT, EXEC and OUTPUT queued far ahead of the GPU: the slots and IO memory of requests that are not over yet are given on."""
import numpy as np
import pytest
import torch

from gpu_common import Case
from oracle import topology as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rooms", [1, 2, 3, 80])   # requests the IO cache holds; with 80 the 64 slots run out first
def test_requests_queued_ahead_of_the_gpu(rooms):
    from paper_2006_02464_amd.runner import Worker
    case = Case(T.resnet(18), 64, seed=2, dist="uniform")
    one = 4 * 3 * 64 * 64 + 2 * 4096
    wk = Worker(workspace_bytes=256 << 20, io_bytes=rooms * one, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        mid = wk.ctx.model_define(case.ops, 3, 64, 64, batch_sizes=(1,))
        wk.load(mid, case.blob)
        x = [torch.from_numpy(np.ascontiguousarray(case.images(i, 1), dtype=np.float32)).pin_memory() for i in range(5)]
        want = [wk.infer(mid, v.numpy())[1] for v in x]
        ins, exe, outs = [torch.cuda.Stream() for _ in range(2)], torch.cuda.Stream(), [torch.cuda.Stream() for _ in range(2)]
        got = [(torch.empty(1, 1000, pin_memory=True), torch.empty(1, 1000, pin_memory=True)) for _ in range(150)]
        for k, (probs, logits) in enumerate(got):
            slot = wk.ctx.input(mid, 1, x[k % 5], ins[k % 2])
            wk.ctx.exec(mid, 1, slot, exe)
            wk.ctx.output(slot, probs, logits, outs[k // 2 % 2])
        torch.cuda.synchronize()
        for k, (_, logits) in enumerate(got):
            assert np.array_equal(logits.numpy(), want[k % 5])
    finally:
        wk.close()


@pytest.mark.parametrize("order", [(0, 1, 2), (1, 0, 2), (2, 2, 0), (0, 0, 1)])   # 0 = the default stream, whose handle is null
def test_io_memory_given_on_in_parts_to_requests_on_several_streams(order):
    """The IO cache holds one request of two images or two of one image.  With OUTPUT held up, a request of one image takes
    half of an unfinished request's memory early, and the next one, on another stream, what is left of it: it must wait too."""
    from paper_2006_02464_amd.runner import Worker
    case = Case(T.resnet(18), 64, seed=4, dist="uniform")
    wk = Worker(workspace_bytes=256 << 20, io_bytes=2 * (4 * 3 * 64 * 64 + 2 * 4096), weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        mid = wk.ctx.model_define(case.ops, 3, 64, 64, batch_sizes=(1, 2))
        wk.load(mid, case.blob)
        x = [torch.from_numpy(np.ascontiguousarray(case.images(2 * i, n), dtype=np.float32)).pin_memory() for i, n in enumerate((2, 1, 1))]
        want = [wk.infer(mid, v.numpy())[:2] for v in x]
        streams = [torch.cuda.default_stream(), torch.cuda.Stream(), torch.cuda.Stream()]
        exe, out = torch.cuda.Stream(), torch.cuda.Stream()
        got = []
        for k in range(9):
            b = x[k % 3].shape[0]
            if k % 3 == 0:
                with torch.cuda.stream(out):
                    torch.cuda._sleep(20_000_000)
            slot = wk.ctx.input(mid, b, x[k % 3], streams[order[(k + k // 3) % 3]])
            wk.ctx.exec(mid, b, slot, exe)
            got.append((torch.empty(b, 1000, pin_memory=True), torch.empty(b, 1000, pin_memory=True)))
            wk.ctx.output(slot, got[-1][0], got[-1][1], out)
        torch.cuda.synchronize()
        for k, (probs, logits) in enumerate(got):
            assert np.array_equal(probs.numpy(), want[k % 3][0]) and np.array_equal(logits.numpy(), want[k % 3][1]), k
    finally:
        wk.close()


def test_memory_of_a_released_input_waits_for_its_copy():
    """A request is released while its INPUT copy is still queued behind other work of its stream; the next one takes the
    same memory through another stream and is executed later than both copies."""
    from paper_2006_02464_amd.runner import Worker
    case = Case(T.resnet(18), 64, seed=5, dist="uniform")
    wk = Worker(workspace_bytes=256 << 20, io_bytes=4 * 3 * 64 * 64 + 2 * 4096, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        mid = wk.ctx.model_define(case.ops, 3, 64, 64, batch_sizes=(1,))
        wk.load(mid, case.blob)
        x = [torch.from_numpy(np.ascontiguousarray(case.images(i, 1), dtype=np.float32)).pin_memory() for i in range(2)]
        want = wk.infer(mid, x[1].numpy())[1]
        late, soon, exe = (torch.cuda.Stream() for _ in range(3))
        for stream, cycles in ((late, 10_000_000), (exe, 40_000_000)):
            with torch.cuda.stream(stream):
                torch.cuda._sleep(cycles)
        wk.ctx.release(wk.ctx.input(mid, 1, x[0], late))
        slot = wk.ctx.input(mid, 1, x[1], soon)
        wk.ctx.exec(mid, 1, slot, exe)
        probs, logits = torch.empty(1, 1000, pin_memory=True), torch.empty(1, 1000, pin_memory=True)
        wk.ctx.output(slot, probs, logits, exe)
        torch.cuda.synchronize()
        assert np.array_equal(logits.numpy(), want)
    finally:
        wk.close()


@pytest.mark.parametrize("us", [0, 1, -1])   # none, one that gives up long before the EXEC ends, the default
@pytest.mark.parametrize("rooms", [1, 6])
def test_streams_that_wait_for_an_exec(us, rooms):
    """OUTPUT and the INPUT that takes an unfinished request's memory wait for the EXEC, whatever their wait launch does."""
    from paper_2006_02464_amd.runner import Worker
    case = Case(T.resnet(18), 64, seed=6, dist="uniform")
    wk = Worker(workspace_bytes=256 << 20, io_bytes=rooms * (4 * 3 * 64 * 64 + 2 * 4096), weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        mid = wk.ctx.model_define(case.ops, 3, 64, 64, batch_sizes=(1,))
        wk.load(mid, case.blob)
        x = [torch.from_numpy(np.ascontiguousarray(case.images(i, 1), dtype=np.float32)).pin_memory() for i in range(5)]
        want = [wk.infer(mid, v.numpy())[:2] for v in x]
        wk.ctx.set_wait_launches(us)
        inp, exe, out = (torch.cuda.Stream() for _ in range(3))
        with torch.cuda.stream(exe):
            torch.cuda._sleep(2_000_000)
        got = [(torch.empty(1, 1000, pin_memory=True), torch.empty(1, 1000, pin_memory=True)) for _ in range(80)]
        for k, (probs, logits) in enumerate(got):
            slot = wk.ctx.input(mid, 1, x[k % 5], inp)
            wk.ctx.exec(mid, 1, slot, exe)
            if k % 7 == 6:
                wk.ctx.release(slot)   # its stream is the library's
            else:
                wk.ctx.output(slot, probs, logits, out)
        torch.cuda.synchronize()
        for k, (probs, logits) in enumerate(got):
            if k % 7 != 6:
                assert np.array_equal(probs.numpy(), want[k % 5][0]) and np.array_equal(logits.numpy(), want[k % 5][1]), k
    finally:
        wk.close()


@pytest.mark.parametrize("batch,classes", [(1, 1), (3, 7), (1, 1000), (5, 1001), (16, 4099)])   # below 16 bytes, odd words, more than a workgroup each
def test_results_in_any_host_memory(batch, classes):
    """Pinned memory is written by the GPU, everything else by copies of the runtime: the same values, and nothing behind them."""
    from paper_2006_02464_amd.runner import Worker
    O = T.Op
    ops = [O(T.CONV, 3, 64, 3, 3, 2, 1, 1, -1, -1), O(T.CONV, 64, 256, 1, 1, 1, 0, 1, -1, 0), O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, 1),
           O(T.FC, 256, classes, 1, 1, 1, 0, 0, -1, 2), O(T.SOFTMAX, classes, classes, 0, 0, 1, 0, 0, -1, 3)]
    case = Case(ops, 16, seed=7, dist="uniform")
    wk = Worker(workspace_bytes=64 << 20, io_bytes=16 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        mid = wk.ctx.model_define(case.ops, 3, 16, 16, batch_sizes=(batch,))
        wk.load(mid, case.blob)
        x = torch.from_numpy(np.ascontiguousarray(case.images(0, batch), dtype=np.float32)).pin_memory()
        n, stream, got = batch * classes, torch.cuda.Stream(), []
        for probs_at, logits_at, pin in ((0, 0, True), (1, 0, True), (0, 2, True), (0, None, True), (0, 0, False)):
            p, z = (torch.full((n + 8,), -5.0, pin_memory=pin) for _ in range(2))
            slot = wk.ctx.input(mid, batch, x, stream)
            wk.ctx.exec(mid, batch, slot, stream)
            wk.ctx.output(slot, p[probs_at:], None if logits_at is None else z[logits_at:], stream)
            stream.synchronize()
            assert (p[:probs_at] == -5).all() and (p[probs_at + n:] == -5).all()
            got.append(p[probs_at:probs_at + n].numpy().copy())
            if logits_at is None:
                assert (z == -5).all()
            else:
                assert (z[:logits_at] == -5).all() and (z[logits_at + n:] == -5).all()
                got.append(np.exp(z[logits_at:logits_at + n].double().numpy().reshape(batch, classes)))
                # fp32 exponentials and sums: a few units in the last place of a probability
                np.testing.assert_allclose(got[-2].reshape(batch, classes), got[-1] / got[-1].sum(1, keepdims=True), rtol=3e-6, atol=1e-30)
            assert np.array_equal(got[0], got[-1 if logits_at is None else -2])
    finally:
        wk.close()


@pytest.mark.parametrize("ahead", [0, 1000, 15 * 1000])   # of the 16 x 1000 probabilities the logits take all, all but a row, a row
def test_results_that_share_pinned_memory(ahead):
    """The logits are written behind the probabilities."""
    from paper_2006_02464_amd.runner import Worker
    case, batch = Case(T.resnet(18), 64, seed=6, dist="uniform"), 16
    wk = Worker(workspace_bytes=256 << 20, io_bytes=16 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        mid = wk.ctx.model_define(case.ops, 3, 64, 64, batch_sizes=(batch,))
        wk.load(mid, case.blob)
        x = torch.from_numpy(np.ascontiguousarray(case.images(0, batch), dtype=np.float32)).pin_memory()
        probs, logits = (v.reshape(-1) for v in wk.infer(mid, x.numpy())[:2])
        stream = torch.cuda.Stream()
        for k in range(20):
            both = torch.full((2 * batch * 1000,), -5.0, pin_memory=True)
            slot = wk.ctx.input(mid, batch, x, stream)
            wk.ctx.exec(mid, batch, slot, stream)
            wk.ctx.output(slot, both, both[ahead:], stream)
            stream.synchronize()
            assert np.array_equal(both[:ahead].numpy(), probs[:ahead]) and np.array_equal(both[ahead:ahead + batch * 1000].numpy(), logits), k
    finally:
        wk.close()


def test_output_by_launch_only_within_one_allocation():
    """Two ends in pinned memory do not make a result of what lies between them."""
    import paper_2006_02464_amd as cw
    c = cw.Context(workspace_bytes=64 << 20, io_bytes=16 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        size = 1 << 20
        pinned = [torch.empty(size, dtype=torch.uint8, pin_memory=True) for _ in range(3)]
        pageable = torch.empty(size + 16, dtype=torch.uint8)
        at = sorted(t.data_ptr() for t in pinned)
        for a in at:
            assert c.output_by_launch(a, size) and c.output_by_launch(a + size - 16, 16) and c.output_by_launch(a + 16, 4)
            assert not c.output_by_launch(a + size - 16, 20 + size) and not c.output_by_launch(a + 4, 16) and not c.output_by_launch(a, 0)
        for a, b in zip(at, at[1:]):
            assert not c.output_by_launch(a, b - a + size) and not c.output_by_launch(a + size - 16, b - a - size + 32)
        assert not c.output_by_launch((pageable.data_ptr() + 15) & ~15, 16)
    finally:
        c.destroy()


def test_results_of_2_gib_are_left_to_the_runtime():
    """The launch's offsets end below 2 GiB; a larger result goes through the copy that takes any size."""
    import paper_2006_02464_amd as cw
    c = cw.Context(workspace_bytes=64 << 20, io_bytes=16 << 20, weight_pool_bytes=64 << 20, load_staging_bytes=64 << 20)
    try:
        pinned = torch.empty(1 << 31, dtype=torch.uint8, pin_memory=True)
        assert c.output_by_launch(pinned.data_ptr(), (1 << 31) - 16) and not c.output_by_launch(pinned.data_ptr(), 1 << 31)
    finally:
        c.destroy()
