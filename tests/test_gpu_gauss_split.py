"""Gaussian sums where their deals of work and their exponential change.

Exponential: one source at its leaf's centre and targets on exactly representable
offsets, so that each sum is one pair's, against 40-digit arithmetic from r = 0 to
beyond the underflow of the smallest value.  q = log2(e) r^2 / (2 sigma^2) is
formed with 4 roundings (FP64 eps = 1.1e-16: relative 4 eps q in the result), the
power with 4 and the norm with 4: (4 q + 8) eps; FP32: eps = 6e-8, plus 2 ulp of
the exponential's argument reduction: (4 q + 8) eps down to the smallest normal.

Deals: level 4 splits a leaf over 8 waves, level 5 takes a wave per leaf; leaf
populations around every lane-group size, against the oracle at the gates of the
general case (1e-13 and 2e-6 of the sum of magnitudes)."""
import mpmath as mp
import numpy as np
import pytest

import workloads as W
from oracle import rbf as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_1110_2921_amd as vm
    return vm.FMM()


def _dev(v):
    import torch
    return torch.from_numpy(np.ascontiguousarray(np.asarray(v, np.float64).T)).cuda()


@pytest.mark.parametrize("precision,eps,tiny", [("fp64", 2.0 ** -53, 2.0 ** -1022), ("mixed", 2.0 ** -24, 2.0 ** -126)])
def test_exponential(ctx, precision, eps, tiny):
    mp.mp.dps = 40
    sigma, box = 2.0 ** -5, 8.0
    r = np.unique(np.rint(np.concatenate([[0.0], np.geomspace(0.0002, 1.4, 900)]) * 2 ** 16)) / 2 ** 16
    x = np.full((len(r) + 1, 3), 5.0)
    x[1:, 0] += r
    g = np.zeros_like(x)
    g[0] = [1.0, -2.0, 0.5]
    out = ctx.gauss_sum(_dev(x), _dev(g), sigma, 2, periodic=0, box_len=box,
                        precision=precision).cpu().numpy().T[1:]
    norm = 1 / mp.sqrt(2 * mp.pi * mp.mpf(sigma) ** 2) ** 3
    for ri, o in zip(r, out):
        e = mp.mpf(float(ri)) ** 2 / (2 * mp.mpf(sigma) ** 2)
        want = norm * mp.exp(-e)
        tol = (4 * float(e / mp.log(2)) + 8) * eps * float(want) + 2 * float(norm) * tiny
        for k in range(3):
            assert abs(float(mp.mpf(o[k]) - want * g[0][k])) <= tol * abs(g[0][k]), (ri, k)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("level", [4, 5])
def test_deals_of_work(ctx, level, precision):
    counts = np.zeros(8 ** level, int)
    edges = [1, 7, 8, 9, 13, 24, 33, 34, 48, 49, 63, 64, 65, 96, 100, 130]
    counts[::8 ** level // 64] = edges * 4
    counts[1::8 ** level // 64] = 3
    x, g = W.particles_with_leaf_counts(counts, level, 7)
    sigma = 2 * np.pi / 2 ** level / 3
    want = R.gauss_sum(x, g, sigma, level, periodic=1)
    scale = R.gauss_sum(x, np.abs(g), sigma, level, periodic=1)
    got = ctx.gauss_sum(_dev(x), _dev(g), sigma, level, periodic=1, precision=precision).cpu().numpy().T
    tol = 1e-13 if precision == "fp64" else 2e-6
    assert np.all(np.abs(got - want) <= tol * scale + 1e-300)
