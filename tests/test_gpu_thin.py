"""GPU parity of the thin-input convolution (conv_thin.hip): input channels that
fill no 16-byte piece, at the edges of its blocks and of its pieces (filter
rows of less than a piece, exactly one, one value more), odd channel counts and
strides (pixels at any alignment), every block it has and why it takes it (the
launch, the channels, the LDS), the fused pool, ragged output channels, and
values a window must not see: the pixels around a tile's edge windows are
infinite where the layer does not read them.  Layers of few products, which stay
on the vector ALUs; in float32 those give the same bits, so the choice may follow
the launch.  test_dispatch.py checks what the cases reach.

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
    (3, 32, 7, 2, 3, 224, 200, False, "2x3", 4),
    (3, 8, 3, 1, 1, 20, 21, False, "1x1", 1),
    (2, 24, 4, 3, 2, 33, 30, False, "2x1", 2),     # a filter row of one bf16 piece
    (1, 40, 9, 1, 4, 19, 37, False, "1x2", 1),     # one value more than a piece
    (5, 33, 5, 2, 0, 40, 41, False, "2x2", 1),     # odd channels, stores value by value
    (7, 70, 11, 4, 10, 60, 50, False, "1x1", 1),   # the largest filter: past the LDS, the any-filter kernel
    (13, 20, 3, 1, 2, 26, 22, True, "2x2", 2),
    (3, 32, 7, 2, 3, 448, 400, False, "2x3", 4),   # 16x16 blocks of 32 channels
    (3, 32, 3, 1, 1, 300, 310, True, "2x2", 2),
    (5, 64, 3, 1, 1, 196, 190, False, "2x2", 4),   # 16x16 blocks of 64 channels
    (3, 48, 5, 1, 2, 260, 270, True, "2x2", 2),
    (5, 96, 7, 2, 0, 300, 290, False, "1x1", 4),   # float32: 8x8 blocks of 32 channels by the LDS, past 32 outputs
    (5, 70, 9, 1, 4, 33, 30, True, "2x2", 1),
    (10, 48, 9, 1, 4, 30, 28, False, "2x1", 1),    # bf16: the same
    (10, 48, 9, 1, 4, 30, 28, True, "2x1", 1),
    (4, 40, 3, 1, 1, 30, 34, True, "2x2", 1),      # bf16: 8x8 blocks of 64 channels, pooled
    (3, 40, 3, 1, 1, 30, 34, True, "2x2", 1),
]

# Few products: the vector ALUs
FEW = [
    (1, 1, 3, 1, 1, 150, 140, False, "2x2", 1),
    (1, 1, 3, 1, 1, 740, 720, True, "2x2", 1),     # float32 by the size of the launch
    (2, 4, 1, 1, 0, 133, 129, False, "3x2", 1),
    (2, 4, 1, 1, 0, 131, 130, True, "2x2", 2),
    (1, 8, 1, 2, 0, 257, 261, False, "2x1", 1),    # strided
    (3, 1, 2, 1, 0, 140, 131, False, "1x2", 2),    # no "same" filter
    (1, 2, 2, 2, 1, 261, 259, True, "2x1", 1),
    (8, 2, 1, 1, 0, 133, 130, False, "2x2", 2),    # whole pieces
    (4, 8, 1, 1, 0, 262, 257, False, "2x2", 1),
    (8, 2, 1, 1, 0, 270, 262, True, "3x2", 1),
    (3, 8, 3, 1, 1, 200, 190, False, "2x2", 1),    # the image kernel
    (3, 8, 3, 1, 1, 200, 190, True, "3x2", 1),
    (3, 16, 3, 1, 1, 33, 35, False, "2x1", 1),
    (3, 16, 3, 1, 1, 200, 190, True, "3x2", 1),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES + FEW, ids=lambda c: "-".join(str(v) for v in c[:8]))
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


@pytest.mark.parametrize("case", [(3, 16, 3, 1, 1, 200, 190, True), (3, 8, 3, 1, 1, 200, 190, True), (1, 1, 3, 1, 1, 740, 720, True),
                                  (2, 8, 1, 1, 0, 740, 720, True), (5, 4, 1, 1, 0, 731, 745, False)],
                         ids=lambda c: "-".join(str(v) for v in c))
def test_float32_bits_on_either_unit(case):
    # all tiles at once run on the vector ALUs, one at a time on the matrix cores (or the other way round for some tiles)
    require_gpu()
    import torch
    from paper_2107_06960_amd import mafat as M
    cin, cout, f, s, p, h, w, pool = case
    print(f"[thin bits] {case}", flush=True)
    layers = [W.conv(cout, f, s=s, p=p)] + ([W.maxpool()] if pool else [])
    par = W.make_inputs(layers, h, w, cin, 1, 9, "f32")
    par["x"] = par["x"] - np.float32(0.5)
    out = []
    for tb in (0, 1):
        net = M.Network(M.Plan(layers, (h, w, cin), "3x3", tile_batch=tb), par, 1, "f32")
        out.append(net.run(net.input_tensor(par["x"])).clone())
    equal = torch.equal(*out)
    assert equal
