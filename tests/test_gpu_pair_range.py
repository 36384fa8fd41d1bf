"""The mixed near field's pair table over units: boxes, cores and strengths whose
terms in physical units (q alpha about alpha / r^3) are well inside FP32, but whose
terms in units of the core are not unless the table's scale follows the core.

One source at the box centre and targets at exactly representable offsets, so that each
velocity and gradient is one pair's, against the oracle's FP64 sum.  Tolerances: the
FP32 table's 1.0e-7 (q) and 1.6e-7 (q'/r), the rounding of t = r^2 / sigma^2 (3
operations at 6e-8, entering 1.5 and 2.5 times) and 5 further roundings: 8e-7 and 1.2e-6."""
import numpy as np
import pytest

from oracle import direct as D

pytestmark = pytest.mark.gpu
TOL_U, TOL_J = 8e-7, 1.2e-6


@pytest.fixture(scope="module")
def ctx():
    import paper_1110_2921_amd as vm
    return vm.FMM()


# box, core / box, strength: ordinary cores in small units, with small strengths; in
# large ones; cores far below the leaf, up to the table's last (2^-20 of the leaf)
@pytest.mark.parametrize("box,ratio,strength", [
    (2.0 ** -12, 2.0 ** -3, 1e-30), (2.0 ** -12, 2.0 ** -3, 1e-5), (2.0 ** -24, 2.0 ** -3, 1e-20),
    (2.0 ** 30, 2.0 ** -3, 1e20), (0.25, 2.0 ** -12, 1e-25), (8.0, 2.0 ** -16, 1e-18), (1.0, 2.0 ** -19.9, 1e-12),
    (2.0 ** 20, 2.0 ** -19.9, 1.0)])
def test_pairs_in_any_units(ctx, box, ratio, strength):
    import torch
    r = np.unique(np.rint(np.geomspace(64, 22000, 300))) * 2.0 ** -16 * box
    x = np.full((len(r) + 1, 3), 0.5 * box)
    x[1:, 0] += r
    a = np.zeros_like(x)
    a[0, 2] = strength
    sigma = ratio * box
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v.T)).cuda()
    print(f"[near] box {box:g} sigma {sigma:g} strength {strength:g}", flush=True)
    u, _, J = ctx.eval(dev(x), dev(a), sigma, 3, 0, periodic=0, box_len=box, precision="mixed", want_grad=True)
    u, J = u.cpu().numpy().T[1:], J.cpu().numpy().T[1:].reshape(-1, 3, 3)
    ud, Jd = D.direct(x[1:], x, a, sigma, box, K=0)
    Jd = np.asarray(Jd).reshape(-1, 3, 3)
    # alpha x r along y; J[x][y] = q'/r r^2 + q, J[y][x] = -q: relative to the larger term
    q = -Jd[:, 1, 0]
    scale = np.maximum(np.abs(q), np.abs(Jd[:, 0, 1] - q))
    eu = np.abs(u[:, 1] / ud[:, 1] - 1).max()
    ej = max(np.abs(J[:, 1, 0] / Jd[:, 1, 0] - 1).max(), (np.abs(J[:, 0, 1] - Jd[:, 0, 1]) / scale).max())
    print(f"[near] u {eu:.2e} (gate {TOL_U:.1e}), J {ej:.2e} (gate {TOL_J:.1e})", flush=True)
    assert eu < TOL_U and ej < TOL_J
