"""GPU: max-pool stages on their own.  A pool only selects, so every output
equals the maximum taken with torch on the CPU, bit for bit: windows known at
compile time and not, channels that fill 16-byte pieces and not, windows that
hang over every side, values that are all negative, infinite or the lowest
finite one, batches, tiles and every execution of a plan."""
import numpy as np
import pytest

from paper_2107_06960_amd import workloads as W

from gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def _ref(x, f, s, p):
    import torch
    b, h, w, c = x.shape
    ho, wo = (h + 2 * p - f) // s + 1, (w + 2 * p - f) // s + 1
    pad = torch.full((b, h + 2 * p, w + 2 * p, c), float("-inf"))
    pad[:, p:p + h, p:p + w] = x
    out = None
    for ky in range(f):
        for kx in range(f):
            t = pad[:, ky:ky + s * (ho - 1) + 1:s, kx:kx + s * (wo - 1) + 1:s]
            out = t.clone() if out is None else torch.maximum(out, t)
    return out


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("f,s,p", [(2, 2, 0), (3, 2, 1), (3, 1, 1), (3, 2, 2), (2, 1, 1), (5, 3, 4), (1, 2, 0)])
def test_pool_selects(f, s, p, dtype):
    require_gpu()
    import torch
    from paper_2107_06960_amd import mafat as M
    for c, h, w, tiling, batch in ((8, 23, 31, "2x3", 2), (64, 17, 40, "3x1", 3), (3, 19, 15, "1x1", 2),
                                   (20, 9, 13, "2x2", 1), (2048, 7, 6, "1x2", 1), (256, 64, 60, "2x2", 4)):
        print(f"[pool] {f}/{s}/{p} c={c} {h}x{w} {tiling} b{batch} {dtype}", flush=True)
        tdt = torch.float32 if dtype == "f32" else torch.bfloat16
        x = torch.from_numpy(np.random.default_rng(c).standard_normal((batch, h, w, c)).astype(np.float32) - 3.0).to(tdt)
        x[0, : h // 2, : w // 2] = torch.finfo(tdt).min
        x[0, 0, 0], x[0, h - 1, w - 1], x[0, h // 2, w // 2] = float("-inf"), float("-inf"), float("inf")
        ref = _ref(x.float(), f, s, p)
        for kw in ({}, {"stage_partition": True}, {"row_reuse": True}, {"tile_batch": 1}):
            plan = M.Plan([W.maxpool(f, s, p)], (h, w, c), tiling, **kw)
            net = M.Network(plan, {"w": [None], "scale": [None], "bias": [None]}, batch, dtype)
            net.y.fill_(float("nan"))
            got = net.run(x.cuda()).float().cpu()
            assert torch.equal(got, ref), (c, kw)
