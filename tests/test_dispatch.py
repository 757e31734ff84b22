"""Which kernel and block the tables of the GPU tests reach (host code, no GPU):
a rule that moves must not leave a form of a kernel without its test."""
from paper_2107_06960_amd import mafat as M
from paper_2107_06960_amd import workloads as W

import test_gpu_any_filter
import test_gpu_thin
from gpu_util import stage_config


def _plan(case, tiling):
    cin, cout, f, s, p, h, w, pool = case[:8]
    return M.Plan([W.conv(cout, f, s=s, p=p)] + ([W.maxpool()] if pool else []), (h, w, cin), tiling)


def test_frames_and_batches_take_other_k_groups():
    seen = set()
    for case in test_gpu_any_filter.BATCHED:
        plan = _plan(case, "2x1")
        for dtype in ("f32", "bf16"):
            one, many = stage_config(plan, 1, dtype), stage_config(plan, case[-1], dtype)
            if one["kernel"] == many["kernel"] == "any" and one["kg"] != many["kg"]:
                seen.add((one["gather"], case[7], one["kg"], many["kg"]))
    assert {(g, p) for g, p, _, _ in seen} == {(0, False), (0, True), (1, False), (1, True)}, seen
    assert {(a, b) for _, _, a, b in seen} >= {(4, 1), (4, 2), (2, 1)}, seen


def _reached():
    """(kernel, block, ...) of every single-layer case and data type."""
    out = set()
    for case in test_gpu_any_filter.CASES + test_gpu_thin.CASES + test_gpu_thin.FEW:
        pool, tiling, batch = case[7:]
        for dtype in ("f32", "bf16"):
            c = stage_config(_plan(case, tiling), batch, dtype)
            f, s, p = case[2:5]
            same = f if f in (1, 3) and s == 1 and p == f // 2 else 0
            form = {"thin": (c["br"], c["bn"]), "any": (c["gather"],), "direct": (same,)}.get(c["kernel"], ())
            out.add((c["kernel"], dtype, pool, *form))
            if c["kernel"] == "any":
                out.add(("any block", c["gather"], c["bm"], c["bn"], c["kg"]))
            if c["kernel"] == "thin" and c["bn"] == 32 and case[1] > 32:
                out.add(("thin, 32 of more channels", dtype, pool))
    return out


def test_cases_reach_every_form():
    got = _reached()
    want = {("thin", d, p, b, n) for d in ("f32", "bf16") for p in (False, True) for b in (8, 16) for n in (32, 64)}
    want |= {("thin, 32 of more channels", d, p) for d in ("f32", "bf16") for p in (False, True)}
    want |= {("any", d, p, g) for d in ("f32", "bf16") for p in (False, True) for g in (0, 1)}
    want |= {("any block", g, *b) for g in (0, 1) for b in ((32, 32, 1), (32, 32, 2), (32, 32, 4), (64, 32, 1), (64, 64, 1))}
    want |= {("any block", 1, 32, 64, 2), ("any block", 1, 128, 64, 2)}
    want |= {("rgb", d, p) for d in ("f32", "bf16") for p in (False, True)}
    want |= {("direct", d, p, f) for d in ("f32", "bf16") for p in (False, True) for f in (0, 1, 3)
             if (d, p, f) != ("bf16", True, 3)}  # 2^31-byte frames only
    assert not want - got, sorted(want - got)
