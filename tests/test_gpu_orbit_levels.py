"""The reflection-orbit M2L at every level and degree it is built for (p = 6, 8,
10): the coarse levels (1 to 3) in one launch whose waves read the operators
from L2, the finer ones through LDS, level 4 split over orbit ranges.

FP64 against the oracle FMM of the same definition at sampled particles
(1e-10: round-off), mixed against FP64 (1e-5 / 1e-4); the adjoint's gather by
<ubar, u(alpha)> = <alpha_bar(ubar), alpha> (1e-12 of the sum of magnitudes, the
round-off of 1e4 terms), and the adaptive tree's form by its equality with the
uniform one on a uniform tree."""
import numpy as np
import pytest

import workloads as W
from oracle import fmm as OF
from tests._gates import FP64, MIXED_J, MIXED_U, close

pytestmark = pytest.mark.gpu
L = 2 * np.pi


@pytest.fixture(scope="module")
def ctx():
    import paper_1110_2921_amd as vm
    return vm.FMM()


def _dev(v):
    import torch
    return torch.from_numpy(np.ascontiguousarray(v.T)).cuda()


# level 1 (one target per octant), 2 and 3 (part-filled and whole column tiles),
# level 4 (orbit ranges), free space (sources beyond the domain) and periodic
# (wrapped: at level 1 and 2 an offset's source can be its own image)
@pytest.mark.parametrize("p,level,K", [(6, 1, 2), (8, 1, 1), (10, 1, 3), (6, 2, 0), (8, 2, 3), (10, 2, 1), (6, 3, 1),
                                       (8, 3, 0), (10, 3, 0), (6, 4, 3), (8, 4, 0)])
def test_every_level_matches_the_oracle(ctx, p, level, K):
    n = 24 * 8 ** min(level, 3)
    x, a = W.random_particles(n, 100 * p + 10 * level + K)
    sigma = L / n ** (1 / 3)
    print(f"[orbit-levels] p={p} level={level} K={K} n={n}", flush=True)
    out = {}
    for prec in ("fp64", "mixed"):
        u, _, J = ctx.eval(_dev(x), _dev(a), sigma, p, level, periodic=K, precision=prec, want_grad=True)
        out[prec] = (u.cpu().numpy().T, J.cpu().numpy().T.reshape(-1, 3, 3))
    close(out["mixed"][0], out["fp64"][0], MIXED_U, "u mixed vs fp64")
    close(out["mixed"][1], out["fp64"][1], MIXED_J, "J mixed vs fp64")
    t = np.sort(np.random.default_rng(p + level + K).choice(n, 16, replace=False))
    uo, Jo = OF.fmm_at(x, a, sigma, p, level, t, periodic=K)
    close(out["fp64"][0][t], uo, FP64, "u vs oracle (sampled)")
    close(out["fp64"][1][t], Jo, FP64, "J vs oracle (sampled)")


@pytest.mark.parametrize("p,level,K", [(6, 3, 1), (8, 2, 3), (8, 4, 0)])
def test_adjoint_gather_is_the_transpose(ctx, p, level, K):
    n = 4096
    x, a = W.random_particles(n, 7 * p + level)
    ub, _ = W.random_particles(n, 1000 + p)
    sigma = L / 16
    u, _, _ = ctx.eval(_dev(x), _dev(a), sigma, p, level, periodic=K)
    _, ab = ctx.adjoint(_dev(x), _dev(a), _dev(ub), sigma, p, level, periodic=K, want_x=False)
    u, ab = u.cpu().numpy().T, ab.cpu().numpy().T
    lhs, rhs = float(np.sum(ub * u)), float(np.sum(ab * a))
    assert abs(lhs - rhs) < 1e-12 * float(np.sum(np.abs(ub * u)))


@pytest.mark.parametrize("p", [6, 8])
def test_adaptive_equals_uniform_on_a_uniform_tree(ctx, p):
    x, a = W.particles_with_leaf_counts([5] * 512, 3, 60 + p)
    ua, _, Ja = ctx.eval_adaptive(_dev(x), _dev(a), L / 32, p, 4, 3, periodic=1, want_grad=True)
    uu, _, Ju = ctx.eval(_dev(x), _dev(a), L / 32, p, 3, periodic=1, want_grad=True)
    close(ua.cpu().numpy().T, uu.cpu().numpy().T, (1e-12, 1e-11), "u adaptive vs uniform")
    close(Ja.cpu().numpy().T, Ju.cpu().numpy().T, (1e-12, 1e-11), "J adaptive vs uniform")
