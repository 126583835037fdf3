"""Boxes of exactly three (or four) cutoffs with lattice particles on the cell faces:
with three cells every pair at the cutoff is half a box from the middle of the cell that sees
it, and with finer cells its particles are a rounding away from being one cell too far
apart.  The library's definition decides which of them are inside (r^2 <= r_c^2 of the
record differences), and decides the same for both particles: forces and the
energy equal the sums over those pairs, formed here in double precision.  The lattices
have pairs at the cutoff along the axes only, so that r^2 is one rounded square
and the decision can be repeated exactly."""
import numpy as np
import pytest
import torch
from scipy.special import erfc

import paper_2010_01559_amd.rbe as R
from gpu_util import host, rel_l2

pytestmark = pytest.mark.gpu


def _inside(x, L, r_cut, prec):
    """(i, j) matrix of the library's decision, and the displacements."""
    # x / L - floor(x / L) is one fused multiply-add
    t = x.astype(np.longdouble) * np.longdouble(1.0 / L)
    s = (t - np.floor(x * (1.0 / L))).astype(np.float64)
    s[s >= 1.0] = 0.0
    if prec == R.RBE_FP64:
        d = s[:, None, :] - s[:, :, None]
        d = (d - np.round(d)) * L
        return (d * d).sum(0) <= r_cut * r_cut, d
    u = np.floor(s * 2.0 ** 32).astype(np.uint32)
    w = (u[:, None, :] - u[:, :, None]).view(np.int32).astype(np.float32) * np.float32(L * 2.0 ** -32)
    return (w * w).sum(0) <= np.float32(r_cut * r_cut), w.astype(np.float64)


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("cuts, m", [(3, 3), (3, 6), (3, 12), (4, 16)])
@pytest.mark.parametrize("L", [3.0, 6.0, 7.7, 10.0, 12.0])
@pytest.mark.parametrize("shift", [0.0, 1e-7, -1e-7, 0.3])
def test_pairs_at_the_cutoff(shift, L, cuts, m, prec):
    ax = (np.arange(m) / m + shift) * L
    pos = np.stack(np.meshgrid(ax, ax, ax, indexing="ij")).reshape(3, -1)
    n = m ** 3
    q = np.random.default_rng(m).normal(size=n)
    q -= q.mean()
    r_cut, alpha = L / cuts, 9.0 / L ** 2
    assert int(np.floor(L / r_cut)) == cuts
    ctx = R.rbe_create(R.Params(n=n, p=4, box=L, alpha=alpha, r_cut=r_cut, precision=prec, skin=0.0))
    dt = torch.float64 if prec == R.RBE_FP64 else torch.float32
    P = torch.as_tensor(pos, dtype=dt, device="cuda").contiguous()
    Q = torch.as_tensor(q, dtype=dt, device="cuda").contiguous()
    F = torch.zeros_like(P)
    R.rbe_real_forces(ctx, P, Q, F)
    x, qq = host(P), host(Q)
    inside, d = _inside(x, L, r_cut, prec)
    np.fill_diagonal(inside, False)
    assert np.array_equal(inside, inside.T)
    r = np.sqrt((d * d).sum(0))
    r[~inside] = 1.0
    b = np.sqrt(alpha)
    cq = qq[:, None] * qq[None, :] * inside
    g = (erfc(b * r) / r + 2 * b / np.sqrt(np.pi) * np.exp(-alpha * r * r)) / r ** 2
    f = host(F)
    # one lost pair changes the forces by 1e-2 of their norm; the sums' own tolerances
    # are those of the real-space tests
    tol = 1e-12 if prec == R.RBE_FP64 else 1e-5
    assert rel_l2(f, -(cq * g * d).sum(-1)) <= tol
    assert np.abs(f.sum(1)).max() <= tol * np.abs(f).sum()
    R.rbe_sample_k(ctx, 0)
    st, (e,) = R.rbe_energy(ctx, P, Q, allow_status=(R.RBE_OK, R.RBE_ERR_NOT_NEUTRAL))
    ref = 0.5 * (cq * erfc(b * r) / r)
    assert abs(e["e_real"] - ref.sum()) <= tol * np.abs(ref).sum()
