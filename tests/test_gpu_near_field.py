"""The near field's pair function and its deals of work.

Pair function: one source at the box centre and targets on exactly
representable offsets, so that each velocity and gradient is one pair's; against
40-digit arithmetic over rho from 1e-2 to 90 (the table's first row, every
octave, beyond its end at rho = 45) and, with cores too small for the table's
units, through the polynomial form.
FP64 tolerance: table 2.1e-16 (q) and 7.0e-16 (q'/r), the rounding of t = r^2/sigma^2
(3 operations, entering 1.5 and 2.5 times) and 5 further roundings: 2e-15 and
3e-15.  FP32: 1.0e-7 and 1.6e-7 with the same roundings at 6e-8: 8e-7 and 1.2e-6.

Work: leaf populations around every lane-group and block size, trees that split
a leaf over waves, workgroups and shares of the sources, and one that does not,
against the direct sum of the oracle (FP64 1e-12: sums of up to 1e4 terms;
mixed at its gates)."""
import mpmath as mp
import numpy as np
import pytest

import workloads as W
from oracle import direct as D
from tests._gates import MIXED_J, MIXED_U, close

pytestmark = pytest.mark.gpu
L = 2 * np.pi


@pytest.fixture(scope="module")
def ctx():
    import paper_1110_2921_amd as vm
    return vm.FMM()


def _dev(v):
    import torch
    return torch.from_numpy(np.ascontiguousarray(np.asarray(v, np.float64).T)).cuda()


def _pair(rho, sigma):
    """q and q'/r of one pair, 40 digits."""
    r, s = mp.mpf(float(rho)), mp.mpf(sigma)
    k = mp.sqrt(2 / mp.pi)
    if r < mp.mpf("0.5"):
        c = [(-mp.mpf(1) / 2) ** n / (mp.factorial(n) * (2 * n + 3)) for n in range(40)]
        q = k * mp.fsum(c[n] * r ** (2 * n) for n in range(40))
        d = k * mp.fsum(2 * n * c[n] * r ** (2 * n - 2) for n in range(1, 40))
    else:
        e = mp.exp(-r * r / 2)
        q = (mp.erf(r / mp.sqrt(2)) - k * r * e) / r ** 3
        d = (k * e - 3 * q) / r ** 2
    return q / s ** 3, d / s ** 5


@pytest.mark.parametrize("precision,sigma,bits,tol_u,tol_j", [
    ("fp64", 2.0 ** -6, 30, 2e-15, 3e-15), ("mixed", 2.0 ** -6, 16, 8e-7, 1.2e-6),
    ("fp64", 2.0 ** -110, 30, 2e-15, 6e-15), ("mixed", 2.0 ** -25, 16, 1.5e-6, 4e-6)])
def test_pair_function(ctx, precision, sigma, bits, tol_u, tol_j):
    mp.mp.dps = 40
    box = 8.0
    # offsets along x, multiples of 2^-bits: exact in the records (FP32: up to 2 with
    # 16 fractional bits); rho from 0.01 to 90 at sigma = 2^-6
    r = np.unique(np.rint(np.geomspace(0.0002, 1.4, 700) * 2 ** bits)) / 2 ** bits
    r = r[r > 0]
    x = np.full((len(r) + 1, 3), 4.0)
    x[1:, 0] += r
    a = np.zeros_like(x)
    a[0] = [0.0, 0.0, 1.0]
    print(f"[near] {precision} sigma={sigma:g} {len(r)} pairs", flush=True)
    u, _, J = ctx.eval(_dev(x), _dev(a), sigma, 2, 0, periodic=0, box_len=box, precision=precision, want_grad=True)
    u, J = u.cpu().numpy().T[1:], J.cpu().numpy().T[1:].reshape(-1, 3, 3)
    f = 1 / (4 * mp.pi)
    eu = ej = 0.0
    for i, ri in enumerate(r):
        q, d = _pair(mp.mpf(float(ri)) / mp.mpf(sigma), sigma)
        R = mp.mpf(float(ri))
        # alpha x r = (0, r, 0): u_y = q r, J[x][y] = q'/r r^2 + q, J[y][x] = -q
        eu = max(eu, abs(float(mp.mpf(u[i, 1]) / (f * q * R) - 1)))
        ej = max(ej, abs(float(mp.mpf(J[i, 1, 0]) / (-f * q) - 1)))
        scale = max(q, abs(d) * R * R)
        ej = max(ej, abs(float((mp.mpf(J[i, 0, 1]) - f * (d * R * R + q)) / (f * scale))))
    print(f"[near] u {eu:.2e} (gate {tol_u:.1e}), J {ej:.2e} (gate {tol_j:.1e})", flush=True)
    assert eu < tol_u and ej < tol_j


COUNTS = [1, 8, 9, 12, 13, 16, 17, 24, 25, 32, 33, 34, 40, 41, 48, 49, 63, 64, 65, 80, 100, 130, 0, 200]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("level", [0, 1])
def test_target_pieces_against_the_direct_sum(ctx, level, precision):
    """Free space below level 2 is the direct sum: every leaf a neighbour."""
    if level == 0:
        sets = [W.random_particles(n, 300 + n) for n in COUNTS if n > 0]
    else:
        sets = [W.particles_with_leaf_counts(COUNTS[i:i + 8], 1, 50 + i) for i in range(0, 24, 8)]
        sets.append(W.random_particles(5000, 3))   # target blocks over workgroups
    for x, a in sets:
        sigma = 0.3
        print(f"[near] pieces level={level} {precision} n={len(x)}", flush=True)
        u, da, J = ctx.eval(_dev(x), _dev(a), sigma, 3, level, periodic=0, precision=precision, want_grad=True)
        ud, Jd = D.direct(x, x, a, sigma, L, K=0)
        gu, gj = ((1e-12, 1e-11), (1e-12, 1e-11)) if precision == "fp64" else (MIXED_U, MIXED_J)
        if len(x) > 1:
            close(u.cpu().numpy().T, ud, gu, "u")
        close(J.cpu().numpy().T.reshape(-1, 9), Jd.reshape(-1, 9), gj, "J")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_deals_of_work_agree(ctx, precision):
    """The same particles at points and at themselves, few targets in many leaves and
    many in few: the near field's shares, target blocks and waves give the sums
    of the general deal to round-off (levels 2, 3 and 5; 5 is a wave per leaf)."""
    x, a = W.random_particles(3000, 5)
    for level in (2, 3, 5):
        sigma = L / 2 ** level / 4
        u, _, J = ctx.eval(_dev(x), _dev(a), sigma, 4, level, periodic=1, precision=precision, want_grad=True)
        for m in (7, 900, 3000):
            up, Jp = ctx.eval_at(_dev(x), _dev(a), _dev(x[:m]), sigma, 4, level, periodic=1, precision=precision,
                                 want_grad=True)
            gu, gj = ((1e-13, 1e-12), (1e-13, 1e-12)) if precision == "fp64" else (MIXED_U, MIXED_J)
            close(up.cpu().numpy().T, u.cpu().numpy().T[:m], gu, f"u level {level} m {m}")
            close(Jp.cpu().numpy().T, J.cpu().numpy().T[:m], gj, f"J level {level} m {m}")
