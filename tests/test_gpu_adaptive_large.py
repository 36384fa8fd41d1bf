"""An adaptive tree of more cells than the reflection-orbit M2L's 32-bit byte offsets reach
(1398100 at p = 8) runs the dense operators.  The velocity at every 5000th
particle against the direct sum, at the paper's accuracy for p = 10 (5e-4) scaled to
p = 8 by the method's convergence of about 0.55 a degree: 2e-3, and ten times that for
the worst one."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import direct as D
from tests._gates import close

pytestmark = pytest.mark.gpu
L = 2 * math.pi


def test_more_cells_than_32_bit_offsets_reach():
    import torch

    import paper_1110_2921_amd as vm
    ctx = vm.FMM()
    x, a = W.random_particles(1100000, 17)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v.T)).cuda()
    print("[adaptive] 1.1e6 particles, ncrit 1, p 8", flush=True)
    u, _, _ = ctx.eval_adaptive(dev(x), dev(a), L / 1024, 8, 1, 8)
    assert len(ctx.debug_adaptive("cells")) > 1398100
    pick = slice(0, None, 5000)
    ud, _ = D.direct(x[pick], x, a, L / 1024, L, K=0)
    close(u.cpu().numpy().T[pick], ud, (2e-3, 2e-2), "u")
