"""GPU: the first pair's kernel (first layer, pool and the 3x3 layer after it in
one workgroup) hands its pooled values from wave to wave through LDS, behind a
barrier that has to wait for the writes.  Many runs of many workgroups, every
block shape, several workgroups per compute unit: every run gives the bits of
the two stages run apart."""
import pytest

from paper_2107_06960_amd import workloads as W

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,tiling,batch", [(144, 144, "1x1", 1), (144, 144, "1x1", 4), (304, 304, "2x2", 2),
                                              (608, 608, "5x5", 1)])
def test_first_pair_repeats(h, w, tiling, batch):
    require_gpu()
    import torch
    from paper_2107_06960_amd import mafat as M
    print(f"[first pair] {h}x{w} {tiling} batch {batch}", flush=True)
    layers = W.YOLOV2_16[:4]
    par = W.make_inputs(layers, h, w, 3, batch, 29, "bf16")
    plan = M.Plan(layers, (h, w, 3), tiling, packed_weights=True)
    assert plan.stage_fused(0, 0, batch)
    net = M.Network(plan, par, batch, "bf16")
    x = torch.from_numpy(par["x"]).cuda().bfloat16()
    for s in range(2):
        net.run_stage(0, s, x, net.y)
    apart = net.y.clone()
    outs = [net.run(x).clone() for _ in range(40)]
    assert all(torch.equal(o, apart) for o in outs)
