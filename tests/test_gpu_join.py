"""Evaluations beyond p = 10, whose M2L from level 4 on waits for the near field on the
side stream: values against the oracle at sampled particles (FP64 and mixed
gates), on the tree's first level that waits, on one below it and on one above, and
replays of a captured graph (two waits for one event) against eager calls."""
import math

import numpy as np
import pytest

import workloads as W
from oracle import fmm as OF
from tests._gates import FP64, MIXED_J, MIXED_U, close

pytestmark = pytest.mark.gpu
L = 2 * math.pi


@pytest.fixture(scope="module")
def ctx():
    import paper_1110_2921_amd as vm
    return vm.FMM()


def _dev(v):
    import torch
    return torch.from_numpy(np.ascontiguousarray(v.T)).cuda()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("p,level,periodic", [(11, 4, 0), (12, 4, 1), (12, 3, 0), (12, 5, 0)])
def test_values(ctx, p, level, periodic, precision):
    x, a = W.random_particles(4000, 60 + p)
    sigma = L / 2 ** level / 4
    gu, gj = (FP64, FP64) if precision == "fp64" else (MIXED_U, MIXED_J)
    print(f"[join] p={p} level={level} K={periodic} {precision}", flush=True)
    u, _, J = ctx.eval(_dev(x), _dev(a), sigma, p, level, periodic=periodic, precision=precision, want_grad=True)
    pick = np.arange(0, 4000, 200)
    uo, Jo = OF.fmm_at(x, a, sigma, p, level, pick, periodic=periodic)
    close(u.cpu().numpy().T[pick], uo, gu, "u")
    close(J.cpu().numpy().T[pick].reshape(-1, 9), Jo.reshape(-1, 9), gj, "J")


def test_captured(ctx):
    import torch
    x0, a0 = W.random_particles(20000, 3)
    x, a = _dev(x0), _dev(a0)
    out = (torch.empty_like(x), torch.empty_like(x), None)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ctx.eval(x, a, L / 64, 12, 4, periodic=1, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ctx.eval(x, a, L / 64, 12, 4, periodic=1, out=out)
    torch.cuda.synchronize()
    for rep in range(3):
        print(f"[join] replay {rep}", flush=True)
        a.copy_(_dev(a0 * (1.0 + 0.1 * rep)))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        ue, de, _ = ctx.eval(x, a, L / 64, 12, 4, periodic=1)
        assert torch.equal(out[0], ue) and torch.equal(out[1], de), rep
