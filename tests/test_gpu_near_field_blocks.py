"""Near fields that deal a leaf's target blocks and its sources over workgroups at
once (several blocks of 64 targets a leaf on average, several shares), with uneven and
empty leaves, and distinct targets, against the oracle's evaluation of the same tree
(FP64 and mixed gates).  At level 2 a launch takes ceil(targets per leaf / 64)
blocks and as many shares, up to 8, as fill 512 workgroups (mixed 768): 2 x 4 and
2 x 6 for 5000 particles, 3 x 2 and 3 x 4 for 9000; at level 1 2 x 8 for 1000."""
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


def _counts(level, n, seed):
    """Uneven leaf counts of about n in all: empty leaves, ends of pieces, several blocks."""
    rng = np.random.default_rng(seed)
    c = rng.choice([0, 1, 33, 64, 65, 100, 129, 260], size=8 ** level).astype(float)
    return np.rint(c * n / c.sum()).astype(int)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,level,periodic", [(5000, 2, 0), (5000, 2, 1), (9000, 2, 0), (9000, 2, 1), (1000, 1, 1)])
def test_blocks_and_shares(ctx, n, level, periodic, precision):
    x, a = W.particles_with_leaf_counts(_counts(level, n, n), level, n + 1)
    sigma = L / 2 ** level / 8
    gu, gj = (FP64, FP64) if precision == "fp64" else (MIXED_U, MIXED_J)
    print(f"[near] blocks and shares n={len(x)} level={level} K={periodic} {precision}", flush=True)
    u, da, J = ctx.eval(_dev(x), _dev(a), sigma, 4, level, periodic=periodic, precision=precision, want_grad=True)
    uo, Jo = OF.fmm(x, a, sigma, 4, level, periodic=periodic)
    close(u.cpu().numpy().T, uo, gu, "u")
    close(J.cpu().numpy().T.reshape(-1, 9), Jo.reshape(-1, 9), gj, "J")
    close(da.cpu().numpy().T, np.einsum("na,nab->nb", a, Jo), gj, "dalpha")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,m", [(300, 6000), (3000, 6000), (9000, 70)])
def test_targets_apart_from_sources(ctx, n, m, precision):
    x, a = W.random_particles(n, 23)
    y = W.particles_with_leaf_counts(_counts(2, m, 5), 2, 6)[0]
    sigma = L / 32
    gu, gj = (FP64, FP64) if precision == "fp64" else (MIXED_U, MIXED_J)
    print(f"[near] points n={n} m={len(y)} {precision}", flush=True)
    u, J = ctx.eval_at(_dev(x), _dev(a), _dev(y), sigma, 4, 2, periodic=1, precision=precision, want_grad=True)
    uo, Jo = OF.fmm_points(x, a, sigma, 4, 2, y, periodic=1)
    close(u.cpu().numpy().T, uo, gu, "u")
    close(J.cpu().numpy().T.reshape(-1, 9), Jo.reshape(-1, 9), gj, "J")
