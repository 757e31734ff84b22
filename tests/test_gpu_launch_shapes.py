"""GPU: block shapes that follow the size of a launch.  The bf16 3x3 stages and
the two fused pairs take other blocks for one tile than for all of them, and
for one frame than for several, and read packed weights whose packing block is
larger than, as large as or smaller than their own.  The sums run in the same
order whatever the block, so every execution gives the same bits: packed and
KRSC weights, all tiles at once, one and two at a time, each frame of a batch
and that frame alone.  One of them is compared with the oracle."""
import numpy as np
import pytest

from paper_2107_06960_amd import workloads as W

from gpu_util import TOL, normwise_err, require_gpu

pytestmark = pytest.mark.gpu

# (layers, h, w, c_in, tiling, batch)
CASES = {
    "pack 64, small launches": ([W.conv(128)], 40, 36, 64, "2x3", 3),
    "pack 64, pooled": ([W.conv(128), W.maxpool()], 70, 66, 64, "3x2", 2),
    "pack 32, many frames": ([W.conv(96)], 21, 19, 96, "2x2", 24),
    "half a block of channels": ([W.conv(80)], 50, 31, 32, "1x4", 2),
    "fewer channels than a block": ([W.conv(16)], 33, 40, 160, "2x2", 2),
    "deep, ragged": ([W.conv(512)], 19, 23, 256, "2x2", 2),
    "first pair": ([W.conv(32), W.maxpool(), W.conv(64), W.maxpool()], 148, 132, 3, "2x2", 2),
    "first pair, many tiles": ([W.conv(32), W.maxpool(), W.conv(64), W.maxpool()], 300, 260, 3, "4x5", 1),
    "second pair": ([W.conv(128), W.conv(64, 1)], 70, 75, 64, "2x3", 2),
    "second pair, 32 outputs": ([W.conv(128), W.conv(32, 1)], 30, 41, 96, "2x2", 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_blocks_follow_the_launch(orc, name):
    require_gpu()
    import torch
    from paper_2107_06960_amd import mafat as M
    layers, h, w, c, tiling, batch = CASES[name]
    par = W.make_inputs(layers, h, w, c, batch, 23, "bf16")

    def run(x, **kw):
        print(f"[launch shapes] {name}: {kw} batch {x.shape[0]}", flush=True)
        net = M.Network(M.Plan(layers, (h, w, c), tiling, **kw), par, x.shape[0], "bf16")
        net.y.fill_(float("nan"))
        return net.run(torch.from_numpy(x).cuda().bfloat16()).clone()

    base = run(par["x"])
    ref = orc.forward_layers(layers, h, w, c, par["x"], par)
    assert normwise_err(base.float().cpu().numpy(), ref) <= TOL["bf16"]
    for kw in ({"packed_weights": True}, {"tile_batch": 1}, {"packed_weights": True, "tile_batch": 1},
               {"packed_weights": True, "tile_batch": 2}, {"packed_weights": True, "row_reuse": True}):
        assert torch.equal(run(par["x"], **kw), base), kw
    for f in (0, batch - 1):
        one = np.ascontiguousarray(par["x"][f:f + 1])
        assert torch.equal(run(one, packed_weights=True)[0], base[f]), f


def test_tile_batch_changed_on_a_used_plan():
    # the plan keeps what it worked out for a run; a new tile batch works it out again
    require_gpu()
    import torch
    from paper_2107_06960_amd import mafat as M
    layers = W.YOLOV2_16[:8]
    par = W.make_inputs(layers, 160, 160, 3, 1, 3, "bf16")
    plan = M.Plan(layers, (160, 160, 3), "4x4", packed_weights=True)
    x = torch.from_numpy(par["x"]).cuda().bfloat16()
    base = M.Network(plan, par, 1, "bf16").run(x).clone()
    for tb in (1, 3, 0):
        print(f"[launch shapes] tile batch {tb}", flush=True)
        M.mafat_plan_set_tile_batch(plan.handle, tb)
        net = M.Network(plan, par, 1, "bf16")
        net.y.fill_(float("nan"))
        assert torch.equal(net.run(x), base), tb
