"""Adaptive evaluations whose translations run all levels in one launch: degrees
with the reflection-orbit M2L (6, 8, 10) and one with the dense form, trees from a
root with leaf children to several levels with leaves on each (octant groups of
one cell and of a part of a tile), free and periodic, against
the oracle's evaluation of the same tree at the FP64 gates."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import adaptive as A
from tests._gates import FP64, close

pytestmark = pytest.mark.gpu
L = 2 * math.pi


@pytest.fixture(scope="module")
def ctx():
    import paper_1110_2921_amd as vm
    return vm.FMM()


@pytest.mark.parametrize("n,ncrit,ml,periodic,p", [
    (40, 39, 1, 0, 6), (40, 39, 1, 1, 10), (150, 6, 4, 0, 8), (120, 6, 3, 1, 10), (300, 5, 5, 0, 6),
    (250, 5, 4, 1, 4)])
def test_levels_in_one_launch(ctx, n, ncrit, ml, periodic, p):
    import torch
    x, a = W.clustered_particles(n, 900 + n)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v.T)).cuda()
    print(f"[adaptive] one launch n={n} ncrit={ncrit} ml={ml} K={periodic} p={p}", flush=True)
    u, _, J = ctx.eval_adaptive(dev(x), dev(a), L / 64, p, ncrit, ml, periodic=periodic, want_grad=True)
    uo, Jo = A.fmm(x, a, L / 64, p, ncrit, ml, periodic=periodic)
    close(u.cpu().numpy().T, uo, FP64, "u")
    close(J.cpu().numpy().T.reshape(-1, 9), Jo.reshape(-1, 9), FP64, "J")
