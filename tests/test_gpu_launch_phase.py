"""pe_plan_launch_phase on plans of the fast rectangular iteration: the phases are
the ordinary iteration's, so running all of them in order gives its result, and
the plan's own launches are as before.  FP32 bar of the path, 1e-5 (2e-4 for the
fast iteration)."""
import numpy as np
import pytest

import synth
from oracle import fastapply as FA
from tests.gpu_util import device_input, oracle_same_iteration, oracle_schedule, relf, to_np

pytestmark = pytest.mark.gpu

NS = (1.875, -1.25, 0.375)


@pytest.mark.parametrize("growing", [False, True])
@pytest.mark.parametrize("shape", [(300, 1100), (1100, 300), (9, 200), (700, 2000)])
def test_phases_of_a_fast_plan(shape, growing):
    """The FP32 planes, fewer than 16 rows, and (growing) FP32 MFMA."""
    import torch
    import paper_2505_16932_amd as pe
    G, vals = device_input(synth.rng(9800 + shape[0]).standard_normal(shape), torch.float32)
    abc = np.array([(6.0 if min(shape) > 16 else 1.5, 0.0, 0.0)] + [NS] * 4) if growing else oracle_schedule(5)
    plan = pe.Plan([G], T=5, abc=abc, compute="f32", out_dtype=torch.float32, fast_restart=3, fast_eps=0.0)
    fast = FA.fast_polar_express(vals, abc, restart=3, eps=0.0)
    for _ in range(2):
        plan.launch()
        torch.cuda.synchronize()
        assert relf(to_np(plan.outs[0]), fast) <= 2e-4
        plan.launch_phase(0, 0)
        for t in range(5):
            for phase in (1, 2, 3):
                plan.launch_phase(t, phase)
        torch.cuda.synchronize()
        assert relf(to_np(plan.outs[0]), oracle_same_iteration(vals, abc)) <= 1e-5
    plan.close()
