"""Strengths and positions that are not numbers through the near field's tables (whose
rows come from the exponent bits of r^2), in a near field alone (free space, level 1,
every leaf a neighbour).  A NaN strength or position makes every velocity NaN, as
in the defining sum; an infinite strength every component that it enters non-finite,
and the others agree with that sum (FP64 1e-12: sums of 300 terms; mixed at its gates)."""
import numpy as np
import pytest

import workloads as W
from oracle import direct as D
from tests._gates import MIXED_U, rel

pytestmark = pytest.mark.gpu
L = 2 * np.pi


@pytest.fixture(scope="module")
def ctx():
    import paper_1110_2921_amd as vm
    return vm.FMM()


def _eval(ctx, x, a, precision):
    import torch
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v.T)).cuda()
    u, _, J = ctx.eval(dev(x), dev(a), 0.3, 3, 1, periodic=0, precision=precision, want_grad=True)
    return u.cpu().numpy().T, J.cpu().numpy().T


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("what", ["strength", "position", "negative position"])
def test_nan(ctx, what, precision):
    x, a = W.random_particles(300, 31)
    print(f"[near] nan {what} {precision}", flush=True)
    if what == "strength":
        a[7] = np.nan
    else:
        x[7] = np.copysign(np.nan, -1.0 if what.startswith("neg") else 1.0)
    u, J = _eval(ctx, x, a, precision)
    assert np.isnan(u).all() and np.isnan(J).all()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_infinite_strength(ctx, precision):
    x, a = W.random_particles(300, 32)
    a[7, 0] = np.inf
    print(f"[near] infinite strength {precision}", flush=True)
    u, _ = _eval(ctx, x, a, precision)
    rest = np.arange(300) != 7
    # alpha x r of alpha along x has no x component
    assert not np.isfinite(u[rest, 1:]).any()
    a[7, 0] = 0.0
    ud, _ = D.direct(x, x, a, 0.3, L, K=0)
    e = rel(u[rest, :1], ud[rest, :1])
    print(f"[near] x component {e:.2e}", flush=True)
    assert e < (1e-12 if precision == "fp64" else MIXED_U[0])
