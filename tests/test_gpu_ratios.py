"""rsdgc_dynamic_ratios call after call with one workspace: what a call leaves behind for the next, on the one-pass form, on the general
path after it and back, and with a compress call, new ratios or another workspace in between.  Against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2312_17530_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_layers", [3, 300])
def test_ratios_call_after_call(n_layers):
    import torch
    shapes = [(1024, 700), (600, 613), (1, 4099)] + [(1, 1 + l % 90) for l in range(n_layers - 3)]
    rng = np.random.default_rng(n_layers)
    plan = binding.rsdgc_plan(shapes, 3, 0.5, [0.02] * n_layers)
    ws, other = (torch.zeros(plan.workspace_bytes, dtype=torch.uint8, device="cuda") for _ in range(2))

    def arena(weights):
        host = np.zeros(plan.total_elems, np.float32)
        for l, w in enumerate(weights):
            o = plan.layer_offset(l)
            host[o:o + w.size] = w.reshape(-1)
        return torch.from_numpy(host).cuda()

    def weights(kind):
        if kind == "equal":                       # (no bracket: the general path)
            return [np.full(sh, 0.25, np.float32) for sh in shapes]
        scale = 10.0 ** rng.uniform(-4, 1) if kind == "normal" else 1e-41      # (subnormal)
        return [(rng.standard_normal(sh) * scale * rng.uniform(0.5, 2.0)).astype(np.float32) for sh in shapes]

    for step, kind in enumerate(["normal", "normal", "equal", "normal", "tiny", "normal", "compress", "normal", "set_ratios", "normal", "other", "normal"]):
        where = other if kind == "other" else ws
        w = weights(kind if kind in ("equal", "tiny") else "normal")
        a = arena(w)
        if kind == "compress":
            out = (torch.zeros(plan.out_capacity, dtype=torch.int32, device="cuda"), torch.zeros(plan.out_capacity, device="cuda"),
                   torch.zeros(n_layers, dtype=torch.int32, device="cuda"))
            binding.rsdgc_compress(plan, a, torch.zeros_like(a), torch.zeros_like(a), *out, ws)
        elif kind == "set_ratios":
            binding.rsdgc_plan_set_ratios(plan, [0.03] * n_layers)
        for rho in (0.02, 0.3):
            assert binding.rsdgc_dynamic_ratios(plan, a, rho, where) == oracle.dynamic_ratios(w, rho), (step, kind, rho)
            # A histogram that a call had left behind would mislead the next one's sample, whose weights are on another scale.  (In the
            # middle of a million weights, and among subnormal ones, the sample's bracket holds too many of them.)
            if rho == 0.02:
                assert binding.rsdgc_ratio_passes(plan) == (5 if kind in ("equal", "tiny") else 1), (step, kind, rho)
