"""GPU: the float32 3x3 convolution on split operands (conv_split.hip).

Finite data against the oracle: blocks that are cut off on every side, output
channels that fill no block, one and several chunks, the fused pool, batches
and every execution of a plan.  The tolerance is that of plain float32: sums of
K products of which each is off by at most 2^-24 (what the dropped part products
hold, of either sign) and rounded at most K times, so
max|gpu - oracle| <= 4 sqrt(K) 2^-24 max|sum| for independent roundings.

Single products and sums of equal ones against float64: the error of a product
shows there, where a dense sum's roundings hide it.

Data the split cannot carry (infinities, NaN, sums past the largest float)
against the same sums in float64 on the CPU: the kernel computes such outputs
again in plain float32.  Operands down to subnormals are no such data: the
parts are of 2^24 times the value."""
import numpy as np
import pytest

from paper_2107_06960_amd import workloads as W

from gpu_util import normwise_err, require_gpu, run_gpu

pytestmark = pytest.mark.gpu

# (c_in, c_out, h, w, pool, tiling, batch)
CASES = [(32, 64, 8, 16, False, "1x1", 1), (32, 16, 17, 9, False, "1x1", 2), (64, 80, 33, 35, True, "2x2", 1),
         (96, 32, 20, 21, True, "1x3", 2), (256, 128, 26, 26, False, "3x3", 1), (32, 48, 130, 150, True, "2x3", 2),
         (512, 32, 6, 5, False, "1x1", 1), (128, 256, 76, 70, False, "1x1", 2)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v) for v in c))
def test_split_conv(orc, case):
    require_gpu()
    from paper_2107_06960_amd import mafat as M
    cin, cout, h, w, pool, tiling, batch = case
    print(f"[split] {case}", flush=True)
    layers = [W.conv(cout)] + ([W.maxpool()] if pool else [])
    par = W.make_inputs(layers, h, w, cin, batch, 11, "f32")
    par["x"] = (par["x"] * 2 - 1).astype(np.float32)
    ref = orc.forward_layers(layers, h, w, cin, par["x"], par)
    assert M.Plan(layers, (h, w, cin), tiling).stage_kernel(0, 0, batch, "f32") == "mfma_f32"
    for kw in ({}, {"part": True}, {"reuse": True}):
        out = run_gpu(layers, h, w, cin, par, tiling, batch, "f32", want_cuts=False, **kw)
        assert normwise_err(out, ref) <= 4 * np.sqrt(9 * cin) * 2.0 ** -24, kw


def _center_sums(x, w, terms):
    """conv outputs (linear, unit scale, no bias) of x (pixels) times w (channels), the same pair in the first `terms`
    channels of the centre tap and zeros elsewhere, as (pixels, channels)."""
    import torch
    from paper_2107_06960_amd import mafat as M
    n, cout, cin = len(x), len(w), 32
    par = {"w": [np.zeros((cout, 3, 3, cin), np.float32)], "scale": [np.ones(cout, np.float32)],
           "bias": [np.zeros(cout, np.float32)]}
    par["w"][0][:, 1, 1, :terms] = w[:, None]
    xt = np.zeros((1, n // 32, 32, cin), np.float32)
    xt[..., :terms] = x.reshape(1, n // 32, 32, 1)
    net = M.Network(M.Plan([W.conv(cout, act=W.LINEAR)], (n // 32, 32, cin), "1x1"), par, 1, "f32")
    return net.run(torch.from_numpy(xt).cuda()).double().cpu().numpy().reshape(n, cout)


def test_split_single_products():
    # A sum of one term is off by its final rounding (at most 2^-24, rms 0.74 / sqrt(3) 2^-24 = 2.5e-8 over
    # mantissas spread evenly in their logarithm), the rounding of the five small terms (at most 2^-30) and the dropped ones (at
    # most 2^-24, rms 5.5e-9): 2^-23 and 2^-25 in all.
    require_gpu()
    rng = np.random.default_rng(19)
    x, w = rng.standard_normal(4096).astype(np.float32), rng.standard_normal(64).astype(np.float32)
    print("[split] single products", flush=True)
    ref = x.astype(np.float64)[:, None] * w.astype(np.float64)[None]
    err = _center_sums(x, w, 1) / ref - 1.0
    assert np.max(np.abs(err)) <= 2.0 ** -23
    assert np.sqrt(np.mean(err ** 2)) <= 2.0 ** -25


# the largest dropped terms of parts cut off, and of parts rounded to nearest (the second part just below a tie)
@pytest.mark.parametrize("units", [2 ** 16 - 1, 32703, -32703, 2 ** 15, 3 * 2 ** 14 + 1])
def test_split_equal_products(units):
    # 32 equal products: dropped terms that do not average out (2^-24), one rounding of the sum of the first parts' products, one
    # of the small ones' (2^-32), one of the end: 3 * 2^-24.
    require_gpu()
    v = np.float32(1.0 + units * 2.0 ** -23)
    print(f"[split] 32 times ({float(v)!r})^2", flush=True)
    out = _center_sums(np.full(32, v, np.float32), np.full(32, v, np.float32), 32)
    assert np.max(np.abs(out / (32 * float(v) ** 2) - 1.0)) <= 3 * 2.0 ** -24


# binary exponents of the inputs (of every other pixel's; the rest are near 1) and of the weights: parts as they are would fall
# below the smallest bf16, beside sums of any size in the same wave
@pytest.mark.parametrize("xe,we", [(-118, 0), (-118, 60), (-125, 30), (-140, 100), (60, -118), (90, -140)])
def test_split_small_operands(xe, we):
    # as for single products: 2^-23
    require_gpu()
    rng = np.random.default_rng(29)
    print(f"[split] inputs 2^{xe}, weights 2^{we}", flush=True)
    x = np.where(np.arange(4096) % 2 == 0, 2.0 ** xe, 1.0) * rng.uniform(1, 2, 4096) * rng.choice([-1, 1], 4096)
    x, w = x.astype(np.float32), (2.0 ** we * rng.uniform(1, 2, 64)).astype(np.float32)
    ref = x.astype(np.float64)[:, None] * w.astype(np.float64)[None]
    ok = np.abs(ref) >= 2.0 ** -126  # normal results
    assert ok[::2].mean() == 1.0 or we == 0
    err = _center_sums(x, w, 1)[ok] / ref[ok] - 1.0
    assert np.max(np.abs(err)) <= 2.0 ** -23


def _conv64(x, par, pool):
    """conv + scale, bias, leaky (+ pool) with the arithmetic of IEEE in float64 (CPU)."""
    import torch
    w = torch.from_numpy(par["w"][0]).double().permute(0, 3, 1, 2)
    v = torch.nn.functional.conv2d(torch.from_numpy(x).double().permute(0, 3, 1, 2), w, padding=1)
    v = v * torch.from_numpy(par["scale"][0]).double()[None, :, None, None]
    v = v + torch.from_numpy(par["bias"][0]).double()[None, :, None, None]
    v = torch.maximum(v, 0.1 * v)
    if pool:
        v = torch.nn.functional.max_pool2d(v, 2)
    return v.permute(0, 2, 3, 1).numpy()


@pytest.mark.parametrize("pool", [False, True])
@pytest.mark.parametrize("kind", ["inf", "nan", "huge", "tiny", "one tiny block", "zero"])
def test_split_special(kind, pool):
    require_gpu()
    print(f"[split special] {kind} pool={pool}", flush=True)
    h, w, cin, cout = 24, 40, 64, 48
    layers = [W.conv(cout)] + ([W.maxpool()] if pool else [])
    par = W.make_inputs(layers, h, w, cin, 1, 5, "f32")
    par["w"][0] = W.bf16_round(par["w"][0])  # whole in the first part: its others are zero
    par["bias"][0][:] = 0.0
    x = par["x"]
    if kind == "inf":
        x[0, 5, 7, 3] = np.inf
    elif kind == "nan":
        x[0, 20, 30, 1] = np.float32(np.nan)
    elif kind == "huge":
        x[0, 3:6] = 3e38  # sums overflow
    elif kind == "tiny":
        x *= np.float32(2.0 ** -118)
    elif kind == "one tiny block":
        x[0, :12, :20] *= np.float32(2.0 ** -118)
    else:
        x[:] = 0.0
    out = run_gpu(layers, h, w, cin, par, "1x1", 1, "f32", want_cuts=False)
    ref = _conv64(x, par, pool)
    with np.errstate(over="ignore"):
        ref = ref.astype(np.float32).astype(np.float64)  # past the largest float: infinite
    if kind in ("inf", "huge", "nan"):
        if kind == "nan":  # a pool window drops a NaN beside a number: only where the whole window is NaN
            far = np.ones(ref.shape, bool)
            s = 2 if pool else 1
            far[0, 19 // s:22 // s + 1, 29 // s:32 // s + 1] = False
            if not pool:
                assert np.array_equal(np.isnan(out), np.isnan(ref))
        elif kind == "huge":  # the rows that read no huge value; what an overflowing sum leaves is not fixed
            far = np.zeros(ref.shape, bool)
            far[0, 8 // (2 if pool else 1):] = True
        else:
            far = np.isfinite(ref)
            assert np.array_equal(out[~far & ~np.isnan(ref)], ref[~far & ~np.isnan(ref)])
        assert np.isfinite(out[far]).all() and far.mean() > 0.5
        assert np.max(np.abs(out[far] - ref[far]) / np.max(np.abs(ref[far]))) <= 4 * np.sqrt(9 * cin) * 2.0 ** -24
    else:
        # every output to the precision of float32 against the block's own scale
        for part in (np.s_[0, : 8 // (2 if pool else 1), : 16 // (2 if pool else 1)], np.s_[0]):
            m = np.max(np.abs(ref[part]))
            assert np.max(np.abs(out[part] - ref[part])) <= 4 * np.sqrt(9 * cin) * 2.0 ** -24 * m + 2.0 ** -148


def test_split_special_time():
    # A NaN in every window has every output computed again in plain float32: on the fp32 MFMA that takes some times as long
    # as the layer, not the hundreds of times of one thread per output.
    require_gpu()
    import torch
    from paper_2107_06960_amd import mafat as M
    h, w, cin, cout = 26, 26, 512, 512
    par = W.make_inputs([W.conv(cout)], h, w, cin, 1, 5, "f32")
    net = M.Network(M.Plan([W.conv(cout)], (h, w, cin), "1x1"), par, 1, "f32")

    def us(x):
        t = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            net.run(x)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b) * 1e3)
        return sorted(t)[len(t) // 2]

    x = net.input_tensor(par["x"])
    plain = us(x)
    x[..., 7] = float("nan")
    special = us(x)
    print(f"[split] 3x3 512->512 on 26x26: {plain:.1f} us, with a NaN in every window {special:.1f} us", flush=True)
    assert torch.isnan(net.y).all()
    assert special <= 8 * plain


# Small launches take smaller blocks than those of all tiles or frames: other outputs share a wave.
@pytest.mark.parametrize("pool", [False, True])
@pytest.mark.parametrize("kind", ["inf", "nan", "huge"])
def test_split_special_bits(kind, pool):
    # which outputs the split could not carry, and what they get, does not follow the blocks: the same bits all tiles at once,
    # one and two at a time, and for a frame alone
    require_gpu()
    import torch
    from paper_2107_06960_amd import mafat as M
    h, w, cin, cout, batch = 60, 52, 64, 128, 3
    layers = [W.conv(cout)] + ([W.maxpool()] if pool else [])
    par = W.make_inputs(layers, h, w, cin, batch, 5, "f32")
    x = par["x"]
    v = {"inf": np.inf, "nan": np.nan, "huge": 3e38}[kind]
    for f in range(batch):
        x[f, 13, 9 + f, 3] = v
        x[f, 40 + f, 30, 60] = v

    def run(x, tile_batch):
        print(f"[split bits] {kind} pool={pool} batch {len(x)} tile batch {tile_batch}", flush=True)
        net = M.Network(M.Plan(layers, (h, w, cin), "3x3", tile_batch=tile_batch), par, len(x), "f32")
        return net.run(net.input_tensor(x)).clone()

    def same(a, b):
        num = ~torch.isnan(a)
        return torch.equal(num, ~torch.isnan(b)) and torch.equal(a[num], b[num])

    base = run(x, 0)
    assert torch.isfinite(base).float().mean() > 0.9
    for tb in (1, 2):
        equal = same(run(x, tb), base)
        assert equal, tb
    for f in range(batch):
        equal = same(run(np.ascontiguousarray(x[f:f + 1]), 0)[0], base[f])
        assert equal, f
