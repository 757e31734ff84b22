"""GPU parity of the float32 1x1 layers (and 3x3 ones without whole 32-channel
chunks) on both sides of the rule that sends small launches to the any-filter
kernel, and of bf16 1x1 layers on both sides of their block rule.

Tolerance: max|gpu - oracle| / max|oracle| <= 1e-4 (f32) and 2e-2 (bf16); tile
batches give the bits of all tiles at once."""
import pytest

from paper_2107_06960_amd import workloads as W

from gpu_util import TOL, normwise_err, require_gpu

pytestmark = pytest.mark.gpu

# (dtype, c_in, c_out, f, h, w, pool, tiling, batch)
CASES = [("f32", 512, 256, 1, 26, 26, False, "3x3", 1), ("f32", 512, 256, 1, 26, 26, False, "3x3", 2),
         ("f32", 16, 32, 3, 32, 32, False, "2x2", 1), ("f32", 16, 32, 3, 100, 90, True, "2x2", 1),
         ("f32", 80, 96, 3, 30, 29, True, "2x2", 1), ("f32", 64, 16, 1, 9, 7, False, "1x1", 3),
         ("bf16", 256, 128, 1, 76, 75, False, "2x2", 1), ("bf16", 256, 128, 1, 76, 75, False, "2x2", 5),
         ("bf16", 480, 256, 1, 37, 38, False, "1x1", 6), ("bf16", 96, 48, 1, 41, 38, True, "2x1", 2),
         ("bf16", 32, 32, 1, 9, 7, False, "1x1", 1)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v) for v in c))
def test_both_sides_of_the_rules(orc, case):
    require_gpu()
    import torch
    from paper_2107_06960_amd import mafat as M
    dtype, cin, cout, f, h, w, pool, tiling, batch = case
    print(f"[small f32] {case}", flush=True)
    layers = [W.conv(cout, f)] + ([W.maxpool()] if pool else [])
    par = W.make_inputs(layers, h, w, cin, batch, 31, dtype)
    ref = orc.forward_layers(layers, h, w, cin, par["x"], par)
    base = None
    for kw in ({}, {"tile_batch": 1}, {"row_reuse": True}):
        plan = M.Plan(layers, (h, w, cin), tiling, **kw)
        assert plan.stage_kernel(0, 0, batch, dtype) == ("mfma_f32" if dtype == "f32" else "ring")
        net = M.Network(plan, par, batch, dtype)
        net.y.fill_(float("nan"))
        out = net.run(net.input_tensor(par["x"])).clone()
        assert normwise_err(out.float().cpu().numpy(), ref) <= TOL[dtype], kw
        base = out if base is None else base
        if "tile_batch" in kw:
            assert torch.equal(out, base)
