"""GPU parity of the any-filter matrix-core convolution (conv_any.hip) at the
edges of its dispatch: whole and ragged input channels, output channels that
fill no block or no 16-byte store, one and several K groups, strides, windows
that hang over the image on every side, the fused pool, batches and tiles.  It
takes ragged channels only where their patch and weights fill more LDS than the
thin-input kernel has; the ragged cases that fit it run there.  test_dispatch.py
checks what the cases reach.

Tolerance: as for every kernel, max|gpu - oracle| / max|oracle| <= 1e-4 (f32)
and 2e-2 (bf16): one layer's fp32 sum of K <= 7200 terms is off by at most
K 2^-24 = 4.3e-4 of the sum of magnitudes in the worst case and by about
sqrt(K) 2^-24 = 5e-6 for independent roundings; a bf16 output by 2^-9."""
import numpy as np
import pytest

from paper_2107_06960_amd import workloads as W

from gpu_util import TOL, normwise_err, require_gpu, run_gpu, stage_config

pytestmark = pytest.mark.gpu

# (c_in, c_out, f, s, p, h, w, pool, tiling, batch)
CASES = [
    (3, 32, 7, 2, 3, 61, 47, False, "2x2", 2),      # an image layer (thin)
    (3, 20, 3, 1, 1, 30, 33, True, "3x1", 1),       # pooled, c_out past no block (thin)
    (8, 24, 3, 2, 1, 29, 35, False, "2x3", 2),      # one bf16 piece per tap, two fp32 ones
    (4, 33, 5, 1, 2, 17, 19, False, "1x1", 1),      # fp32 whole, bf16 thin; stores value by value
    (16, 17, 5, 1, 4, 21, 18, True, "2x2", 1),      # padding past the window's centre
    (64, 64, 5, 1, 2, 28, 25, False, "2x2", 1),     # long K, few pixels: K groups
    (1, 1, 11, 4, 10, 40, 37, False, "1x1", 2),     # the largest filter, stride and padding (thin)
    (40, 72, 3, 1, 0, 23, 21, False, "2x2", 1),     # no padding
    (256, 40, 1, 2, 0, 31, 27, False, "1x2", 1),    # strided 1x1
    (128, 256, 3, 2, 1, 76, 76, False, "2x2", 4),
    (40, 96, 3, 1, 1, 85, 82, False, "2x1", 2),     # "same" 3x3 with a partial channel chunk
    (288, 16, 5, 3, 2, 9, 9, False, "1x1", 1),      # K = 7200 on 9 outputs
    (32, 64, 3, 2, 1, 112, 100, False, "2x1", 4),   # one K group, small and
    (32, 64, 3, 2, 1, 112, 100, False, "2x1", 16),  # large blocks
    (7, 70, 11, 4, 10, 60, 50, False, "1x1", 1),    # ragged channels from here on: the largest filter
    (130, 40, 3, 2, 1, 41, 39, False, "2x2", 1),
    (90, 16, 3, 1, 1, 40, 40, True, "2x1", 2),      # pooled
    (33, 40, 7, 1, 3, 25, 23, True, "2x2", 1),
    (90, 16, 3, 1, 1, 40, 40, False, "2x1", 16),
    (91, 33, 5, 1, 0, 24, 26, True, "1x2", 1),      # odd channels, stores value by value
    (13, 200, 11, 2, 5, 60, 54, False, "1x2", 2),   # wide blocks
    (130, 96, 3, 1, 1, 60, 50, True, "2x2", 2),
    (130, 130, 3, 1, 1, 100, 96, False, "2x2", 4),  # the widest
    (132, 128, 3, 1, 1, 100, 96, True, "2x2", 8),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v) for v in c[:8]))
def test_any_filter(orc, case, dtype):
    require_gpu()
    from paper_2107_06960_amd import mafat as M
    cin, cout, f, s, p, h, w, pool, tiling, batch = case
    print(f"[any filter] {case} {dtype}", flush=True)
    layers = [W.conv(cout, f, s=s, p=p)] + ([W.maxpool()] if pool else [])
    par = W.make_inputs(layers, h, w, cin, batch, 7, dtype)
    par["x"] = (par["x"] - 0.5).astype(np.float32) if dtype == "f32" else W.bf16_round(par["x"] - 0.5)
    ref = orc.forward_layers(layers, h, w, cin, par["x"], par)
    assert M.Plan(layers, (h, w, cin), tiling).stage_kernel(0, 0, batch, dtype) == "generic"
    for kw in ({}, {"part": True}, {"reuse": True}):
        out = run_gpu(layers, h, w, cin, par, tiling, batch, dtype, want_cuts=False, **kw)
        err = normwise_err(out, ref)
        assert err <= TOL[dtype], (kw, err)


# (c_in, c_out, f, s, p, h, w, pool, batch): one frame of them takes more K groups than a batch
BATCHED = [(32, 64, 3, 2, 1, 112, 100, False, 4), (32, 64, 3, 2, 1, 112, 100, False, 16), (128, 256, 3, 2, 1, 76, 76, False, 8),
           (64, 64, 5, 1, 2, 28, 26, True, 24), (90, 16, 3, 1, 1, 40, 40, True, 16), (130, 96, 3, 1, 1, 40, 38, False, 16),
           (132, 128, 3, 1, 1, 100, 96, True, 4)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", BATCHED, ids=lambda c: "-".join(str(v) for v in c))
def test_any_filter_frame_in_a_batch(case, dtype):
    # the block and the K groups follow the batch, a frame's bits do not
    require_gpu()
    import torch
    from paper_2107_06960_amd import mafat as M
    cin, cout, f, s, p, h, w, pool, batch = case
    layers = [W.conv(cout, f, s=s, p=p)] + ([W.maxpool()] if pool else [])
    par = W.make_inputs(layers, h, w, cin, batch, 13, dtype)
    plan = M.Plan(layers, (h, w, cin), "2x1")
    print(f"[any filter] {case} {dtype}: one frame {stage_config(plan, 1, dtype)}, all {stage_config(plan, batch, dtype)}",
          flush=True)

    def run(x):
        net = M.Network(plan, par, len(x), dtype)
        return net.run(net.input_tensor(x)).clone()

    base = run(par["x"])
    for k in (0, batch // 2, batch - 1):
        equal = torch.equal(run(np.ascontiguousarray(par["x"][k:k + 1]))[0], base[k])
        assert equal, k
