"""Which kernel and block the tables of the GPU tests reach (host code, no GPU):
a rule that moves must not leave a form of a kernel without its test."""
from paper_2107_06960_amd import mafat as M
from paper_2107_06960_amd import workloads as W

import test_gpu_any_filter
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
