"""GPU parity of the thin-input convolution (conv_thin.hip): input channels that
fill no 16-byte piece, at the edges of its blocks and of its pieces (filter
rows of less than a piece, exactly one, one value more), odd channel counts and
strides (pixels at any alignment), both block sizes, the fused pool, ragged
output channels, and values a window must not see: the pixels around a tile's
edge windows are infinite where the layer does not read them.

Tolerance: max|gpu - oracle| / max|oracle| <= 1e-4 (f32) and 2e-2 (bf16), as
for every kernel."""
import numpy as np
import pytest

from paper_2107_06960_amd import workloads as W

from gpu_util import TOL, normwise_err, require_gpu, run_gpu

pytestmark = pytest.mark.gpu

# (c_in, c_out, f, s, p, h, w, pool, tiling, batch)
CASES = [
    (3, 32, 3, 1, 1, 70, 66, True, "2x2", 1),      # the float32 first layer
    (3, 64, 3, 1, 1, 131, 97, False, "3x2", 2),
    (3, 16, 3, 1, 1, 64, 64, True, "2x2", 1),
    (3, 32, 7, 2, 3, 224, 200, False, "2x3", 4),   # 16x16 blocks
    (3, 8, 3, 1, 1, 20, 21, False, "1x1", 1),
    (2, 24, 4, 3, 2, 33, 30, False, "2x1", 2),     # a filter row of one bf16 piece
    (1, 40, 9, 1, 4, 19, 37, False, "1x2", 1),     # one value more than a piece
    (5, 33, 5, 2, 0, 40, 41, False, "2x2", 1),     # odd channels, stores value by value
    (7, 70, 11, 4, 10, 60, 50, False, "1x1", 1),   # the largest filter: 8x8 blocks of 32 channels
    (13, 20, 3, 1, 2, 26, 22, True, "2x2", 2),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v) for v in c[:8]))
def test_thin(orc, case, dtype):
    require_gpu()
    cin, cout, f, s, p, h, w, pool, tiling, batch = case
    print(f"[thin] {case} {dtype}", flush=True)
    layers = [W.conv(cout, f, s=s, p=p)] + ([W.maxpool()] if pool else [])
    par = W.make_inputs(layers, h, w, cin, batch, 17, dtype)
    x = par["x"] - np.float32(0.5)
    par["x"] = x if dtype == "f32" else W.bf16_round(x)
    ref = orc.forward_layers(layers, h, w, cin, par["x"], par)
    for kw in ({}, {"part": True}, {"reuse": True}):
        out = run_gpu(layers, h, w, cin, par, tiling, batch, dtype, want_cuts=False, **kw)
        assert normwise_err(out, ref) <= TOL[dtype], kw


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_thin_sees_its_window_only(dtype):
    # an infinite pixel reaches the outputs whose windows hold it and no other
    require_gpu()
    h, w, cin, cout = 21, 35, 3, 24
    for f, s, p in ((3, 1, 1), (7, 2, 3), (5, 1, 0)):
        print(f"[thin window] f={f} s={s} p={p} {dtype}", flush=True)
        layers = [W.conv(cout, f, s=s, p=p)]
        par = W.make_inputs(layers, h, w, cin, 1, 3, dtype)
        par["x"][0, 10, 17, 2] = np.inf
        out = run_gpu(layers, h, w, cin, par, "1x1", 1, dtype, want_cuts=False)[0]
        ho, wo = out.shape[:2]
        hit = np.zeros((ho, wo), bool)
        for y in range(ho):
            for x in range(wo):
                hit[y, x] = 0 <= 10 - (y * s - p) < f and 0 <= 17 - (x * s - p) < f
        assert np.array_equal(np.isfinite(out).all(axis=2), ~hit)
        assert not np.isfinite(out[hit]).any()
