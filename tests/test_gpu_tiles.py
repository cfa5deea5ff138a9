"""The tiles with K slices of 256 or in parts (forced on every layer) and the plan's own tile choice at ragged sizes:
every layer teacher-forced against the CPU oracle."""
import pytest

from gpu_common import TOL, Case, rel_err_per_sample
from oracle import topology as T
from test_gpu_parity import check_all_ops, check_head

pytestmark = pytest.mark.gpu
O = T.Op
K256 = {"32x32k256g4": 29, "32x32k256g8": 30, "64x32k256g4": 31, "64x32k256g8": 32, "32x64k256g4": 33, "32x64k256g8": 34, "64x64k256g4": 35}
# one K slice and several, fewer and more than the ring holds; Cout above, below and beside a tile's width; stride 2; residuals; Cin
# = 64 and 96 beside them, where the tile gives way to a narrower slice
OPS = [
    O(T.CONV, 3, 64, 7, 7, 2, 3, 1, -1, -1),
    O(T.CONV, 64, 256, 3, 3, 2, 1, 1, -1, 0),
    O(T.CONV, 256, 256, 1, 1, 1, 0, 1, 1, 1),
    O(T.CONV, 256, 96, 3, 3, 1, 1, 0, -1, 2),
    O(T.CONV, 96, 512, 3, 3, 2, 1, 1, -1, 3),
    O(T.CONV, 512, 512, 3, 3, 1, 1, 1, 4, 4),
    O(T.CONV, 512, 32, 1, 1, 1, 0, 1, -1, 5),
    O(T.CONV, 32, 256, 1, 1, 1, 0, 1, -1, 6),
    O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, 7),
    O(T.FC, 256, 10, 1, 1, 1, 0, 0, -1, 8),
    O(T.SOFTMAX, 10, 10, 0, 0, 1, 0, 0, -1, 9),
]


@pytest.fixture(scope="module")
def worker():
    from paper_2006_02464_amd.runner import Worker
    w = Worker(workspace_bytes=1 << 30, io_bytes=64 << 20, weight_pool_bytes=128 << 20, load_staging_bytes=64 << 20)
    yield w
    w.close()


def run(worker, hw, dtype, batch, tile=-1, split_k=0, ops=OPS):
    case = Case(ops, hw, seed=9, dtype=dtype, dist="uniform")
    worker.ctx.set_plan_override(tile, split_k)
    worker.ctx.set_debug_keep(True)
    try:
        mid = worker.ctx.model_define(case.ops, 3, hw, hw, batch_sizes=(batch,), dtype=dtype)
    finally:
        worker.ctx.set_plan_override(-1, 0)
        worker.ctx.set_debug_keep(False)
    plan = [dict(l, loaders=worker.ctx.plan_launch_loaders(mid, batch, i)) for i, l in enumerate(worker.ctx.plan(mid, batch))]
    worker.load(mid, case.blob)
    x = case.images(0, batch)
    probs, logits, _ = worker.infer(mid, x, classes=10)
    outs, _, gpu = check_all_ops(worker, case, mid, batch, x)
    check_head(case, gpu[-1], logits, probs)
    assert rel_err_per_sample(logits, outs[-2]).max() <= TOL
    worker.ctx.unload_weights(mid)
    return plan


@pytest.mark.parametrize("name", sorted(K256))
@pytest.mark.parametrize("split_k,dtype", [(1, "fp16"), (3, "fp16"), (1, "bf16")])
def test_k256_tiles(worker, name, split_k, dtype):
    plan = run(worker, 45, dtype, 3, K256[name], split_k)
    wide = [l for l in plan if l["kind"] == 1 and l["tile_k"] == 256]
    assert {l["gemm_k"] for l in wide} == {256, 9 * 256, 9 * 512, 512}
    assert any(l["split_k"] > 1 for l in wide) == (split_k > 1)


@pytest.mark.parametrize("tile", [17, 18, 19, 20, 21, 24])
@pytest.mark.parametrize("hw,dtype", [(45, "fp16"), (33, "bf16")])
def test_tiles_whose_wave_groups_finish_together(worker, tile, hw, dtype):
    """64x64, 64x32, 32x64 and 32x32 in four groups, 32x32 in eight (half of them finish nothing), K slices of 64 and 128."""
    run(worker, hw, dtype, 3, tile)


@pytest.mark.parametrize("tile", [36, 37, 38, 39, 40])
@pytest.mark.parametrize("hw,dtype,batch,split_k", [(45, "fp16", 3, 1), (33, "bf16", 3, 1), (9, "fp16", 1, 1), (45, "fp16", 3, 3), (9, "bf16", 1, 2)])
def test_tiles_in_parts(worker, tile, hw, dtype, batch, split_k):
    """32x32 in quarters and halves on workgroups of their own, slices of 128 and 256, whole and split K."""
    small = [l for l in run(worker, hw, dtype, batch, tile, split_k) if l["kind"] == 1 and l["conv_tile"] == tile]
    assert any(l["split_k"] > 1 for l in small) == (split_k > 1)
    assert {l["gemm_k"] for l in small} == {256, 2304, 4608, 512}


@pytest.mark.parametrize("tile", [17, 18, 19, 20, 21, 24, 29, 30, 31, 33, 35, 36, 37, 38, 39, 40])
@pytest.mark.parametrize("split_k,dtype", [(5, "fp16"), (8, "bf16")])
def test_more_splits_than_are_added_up_together(worker, tile, split_k, dtype):
    """The waves of tiles in four and eight groups add partial sums up four splits at a time: one split in the second round, up
    to four, and rounds that hold the wave's own sums."""
    splits = {l["split_k"] for l in run(worker, 45, dtype, 3, tile, split_k) if l["kind"] == 1 and l["conv_tile"] == tile}
    slices = 4608 // {17: 128, 18: 128, 19: 128, 20: 128, 21: 128, 24: 64, 36: 128, 37: 128, 38: 128}.get(tile, 256)
    per = -(-slices // split_k)
    assert max(splits) == -(-slices // per) > 4


@pytest.mark.parametrize("tile", [36, 37, 38])
def test_pair_launches_on_tiles_in_parts(worker, tile):
    """A 3x3 of stride 2 and the projection beside it in one launch, the last tile of pixels part full (3 x 6 x 6 = 108)."""
    ops = OPS[:1] + [O(T.CONV, 64, 128, 3, 3, 2, 1, 1, -1, 0), O(T.CONV, 128, 256, 3, 3, 2, 1, 1, -1, 1), O(T.CONV, 128, 256, 1, 1, 2, 0, 0, -1, 1),
                     O(T.CONV, 256, 256, 3, 3, 1, 1, 1, 3, 2), O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, 4),
                     O(T.FC, 256, 10, 1, 1, 1, 0, 0, -1, 5), O(T.SOFTMAX, 10, 10, 0, 0, 1, 0, 0, -1, 6)]
    worker.ctx.set_plan_table([(108, 256, 1152, 3, 2, tile, 1), (108, 256, 128, 1, 2, tile, 1)])
    try:
        plan = run(worker, 45, "fp16", 3, ops=ops)
    finally:
        worker.ctx.set_plan_table([])
    assert [l["conv_tile"] for l in plan if l["pair_op"] >= 0] == [tile]


@pytest.mark.parametrize("tile,split_k", [("64x64", 1), ("64x64", 3), ("64x64k128", 1), ("32x32k128g4", 2), ("32x32k256g4", 1), ("128x128w8", 1)])
@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_1x1_ending_in_part_of_a_slice(worker, tile, split_k, dtype):
    """Input channels just above whole slices of 64, 128 and 256, as part of one slice, and as a range of a CONCAT."""
    ops = [O(T.CONV, 3, 64, 3, 3, 2, 1, 1, -1, -1)]
    for n in (32, 96, 160, 288, 352, 544, 224):
        ops.append(O(T.CONV, ops[-1].cout, n, 1, 1, 1, 0, 1, -1, len(ops) - 1))
    ops += [O(T.CONV, 224, 64, 1, 1, 1, 0, 1, -1, 7), O(T.CONV, 64, 32, 3, 3, 1, 1, 1, -1, 8), O(T.CONCAT, 64, 96, 0, 0, 1, 0, 0, 9, 8),
            O(T.CONV, 96, 256, 1, 1, 1, 0, 1, -1, 10), O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, 11), O(T.FC, 256, 10, 1, 1, 1, 0, 0, -1, 12),
            O(T.SOFTMAX, 10, 10, 0, 0, 1, 0, 0, -1, 13)]
    run(worker, 26, dtype, 3, K256.get(tile, tile), split_k, ops)


@pytest.mark.parametrize("hw,batch", [(33, 1), (45, 5), (97, 2), (130, 7)])
def test_chosen_tiles_at_ragged_sizes(worker, hw, batch):
    for l in run(worker, hw, "fp16", batch):
        if l["kind"] == 1 and l["op_index"] > 0:
            o = OPS[l["op_index"]]
            assert (o[1] % l["tile_k"] == 0 or (o[3] == 1 and l["tile_k"] == 64)) and l["tile_n"] <= max(32, l["gemm_n"])
            assert l["grid_x"] == -(-l["gemm_m"] // l["tile_m"]) * -(-l["gemm_n"] // l["tile_n"])


# Tiles of one and two wave groups, most of them with waves that only load: one to four channel slices of a filter's tap, 3x3 and 5x5 filters, strides,
# 1x1 whose K is one, two and several slices (fewer than the ring has stages, and more), Cout beside a tile's width, residuals, K whole and split inside and between taps.
LOADER_TILES = {"128x64": 1, "64x64": 2, "64x32": 3, "32x32": 5, "256x64": 8, "128x128w8": 9, "128x64k128": 10, "64x64k128": 11, "128x64k128g2": 15, "64x64k128g2": 16, "128x64g2": 22, "64x64g2": 23}
LARGE_TILES = {"256x128w8": 25, "128x256w8": 26, "256x256w8": 27, "256x128": 28}   # without
LOADER_OPS = [
    O(T.CONV, 3, 64, 7, 7, 2, 3, 1, -1, -1),
    O(T.CONV, 64, 128, 3, 3, 1, 1, 1, -1, 0),
    O(T.CONV, 128, 256, 3, 3, 1, 1, 1, -1, 1),
    O(T.CONV, 256, 256, 5, 5, 1, 2, 1, -1, 2),
    O(T.CONV, 256, 256, 3, 3, 1, 1, 0, 2, 3),
    O(T.CONV, 256, 128, 3, 3, 1, 1, 1, -1, 4),
    O(T.CONV, 128, 512, 3, 3, 2, 1, 1, -1, 5),
    O(T.CONV, 512, 384, 3, 3, 1, 1, 1, -1, 6),
    O(T.CONV, 384, 96, 3, 3, 1, 1, 1, -1, 7),
    O(T.CONV, 96, 256, 1, 1, 1, 0, 1, -1, 8),
    O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, 9),
    O(T.FC, 256, 10, 1, 1, 1, 0, 0, -1, 10),
    O(T.SOFTMAX, 10, 10, 0, 0, 1, 0, 0, -1, 11),
]


@pytest.mark.parametrize("name, hw, batch, split_k, dtype", [(n, *c) for n in sorted(LOADER_TILES) for c in ((45, 2, 1, "fp16"), (27, 1, 1, "bf16"), (27, 1, 3, "bf16"), (4, 1, 1, "fp16"))] +
                         [(n, *c) for n in sorted(LARGE_TILES) for c in ((45, 2, 1, "fp16"), (27, 1, 3, "bf16"))])
def test_tiles_with_loading_waves(worker, name, hw, batch, split_k, dtype):
    tile = {**LOADER_TILES, **LARGE_TILES}[name]
    own = [l for l in run(worker, hw, dtype, batch, tile, split_k, LOADER_OPS) if l["kind"] == 1 and l["conv_tile"] == tile and l["op_index"] > 0]
    wide, basic = "k128" in name, "g2" not in name and name != "256x64" and name not in LARGE_TILES   # slices of 128; a 1x1 over 96 channels has the tile too
    assert sorted(l["gemm_k"] for l in own) == [96] * (basic and not wide) + [576] * (not wide) + [1152, 1152, 2304, 2304, 3456, 4608, 6400]
    assert all(l["split_k"] == (min(split_k, 2) if l["gemm_k"] == 96 else split_k) for l in own)
    assert all((l["loaders"] > 0) == (split_k == 1 and name in LOADER_TILES) for l in own)


# 130 x 130 pixels, 65 x 65 and 33 x 33: 18 to 4232 workgroups, K from half a slice to 36
BOTH_OPS = [
    O(T.CONV, 3, 64, 7, 7, 2, 3, 1, -1, -1),
    O(T.CONV, 64, 32, 3, 3, 1, 1, 1, -1, 0),
    O(T.CONV, 32, 64, 1, 1, 1, 0, 1, 0, 1),
    O(T.CONV, 64, 256, 1, 1, 1, 0, 1, -1, 2),
    O(T.CONV, 256, 128, 1, 1, 1, 0, 1, -1, 3),
    O(T.CONV, 128, 256, 1, 1, 2, 0, 0, -1, 4),
    O(T.CONV, 256, 128, 3, 3, 2, 1, 1, -1, 5),
    O(T.CONV, 128, 256, 1, 1, 1, 0, 1, -1, 6),
    O(T.GAVGPOOL, 256, 256, 0, 0, 1, 0, 0, -1, 7),
    O(T.FC, 256, 10, 1, 1, 1, 0, 0, -1, 8),
    O(T.SOFTMAX, 10, 10, 0, 0, 1, 0, 0, -1, 9),
]


@pytest.mark.parametrize("tile, loaders", [(0, {1, 5, 6}), (1, {1, 2, 4, 5, 6, 7}), (2, {1, 2, 4, 5, 6, 7}), (3, {1, 6, 7}), (4, {6, 7}), (5, {6, 7}), (8, {1, 2, 5, 6}), (9, {1, 4, 5, 6, 7}),
                                           (10, {1, 2, 6}), (11, {1, 2, 4, 5, 6, 7}), (12, {1, 6, 7}), (13, {6, 7}), (14, {6, 7}), (15, {1, 2, 6}), (16, {2, 6}),
                                           (22, {1, 2, 5, 6, 7}), (23, {2, 6, 7})])
def test_layers_with_and_without_loading_waves(worker, tile, loaders):
    """One network whose layers are issued both ways on every tile."""
    plan = run(worker, 259, "bf16" if tile % 2 else "fp16", 1, tile, 1, BOTH_OPS)
    assert {l["op_index"] for l in plan if l["kind"] == 1 and l["loaders"]} == loaders
