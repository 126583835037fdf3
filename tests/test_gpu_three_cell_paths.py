"""Boxes of exactly three search radii, with three cells along them (up to 120 particles in
each) and with eight: lattices whose pairs at the radius sit half a box from the middle of a
cell.  Forces at both shapes, the adjoint (its sum over the particles is zero, unless a
pair acts on one side only) and steps whose list radius is a third of the box."""
import numpy as np
import pytest
import torch
from scipy.special import erfc

import paper_2010_01559_amd.rbe as R
from gpu_util import host, rel_l2
from test_gpu_three_cells import _inside

pytestmark = pytest.mark.gpu

TOL = {R.RBE_FP64: 1e-12, R.RBE_FP32: 1e-5}


def _lattice(m, L, copies, shift=0.0):
    """`copies` cubic lattices of m^3 sites; a copy is at no pair at the cutoff from the others."""
    out = []
    for c in range(copies):
        off = np.array([0.31, 0.17, 0.05]) * c
        ax = [(np.arange(m) + off[d]) * L / m + shift * L for d in range(3)]
        out.append(np.stack(np.meshgrid(*ax, indexing="ij")).reshape(3, -1))
    return np.concatenate(out, 1)


def _context(n, L, prec, r_cut, skin=0.0, dt=0.0):
    return R.rbe_create(R.Params(n=n, p=4, box=L, alpha=9.0 / L ** 2, r_cut=r_cut, precision=prec, skin=skin, dt=dt,
                                 seed=5))


def _tensors(pos, prec):
    dt = torch.float64 if prec == R.RBE_FP64 else torch.float32
    q = np.random.default_rng(pos.shape[1]).normal(size=pos.shape[1])
    q -= q.mean()
    P = torch.as_tensor(pos, dtype=dt, device="cuda").contiguous()
    return P, torch.as_tensor(q, dtype=dt, device="cuda").contiguous(), torch.zeros_like(P)


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("copies", [1, 2])   # 64 and 128 particles a radius cubed: three and eight cells
@pytest.mark.parametrize("L", [6.0, 7.7])
def test_forces_on_both_sides_of_the_line(L, copies, prec):
    pos = _lattice(12, L, copies)
    P, Q, F = _tensors(pos, prec)
    r_cut = L / 3
    R.rbe_real_forces(_context(pos.shape[1], L, prec, r_cut), P, Q, F)
    x, q = host(P), host(Q)
    inside, d = _inside(x, L, r_cut, prec)
    np.fill_diagonal(inside, False)
    r = np.sqrt((d * d).sum(0))
    if copies == 2:
        n1 = pos.shape[1] // 2
        assert np.abs(r[:n1, n1:] / r_cut - 1.0).min() > 1e-5
    r[~inside] = 1.0
    b = 3.0 / L
    g = (q[:, None] * q[None, :] * inside) * (erfc(b * r) / r + 2 * b / np.sqrt(np.pi) * np.exp(-b * b * r * r)) / r ** 2
    f = host(F)
    assert rel_l2(f, -np.stack([(g * d[k]).sum(-1) for k in range(3)])) <= TOL[prec]
    assert np.abs(f.sum(1)).max() <= TOL[prec] * np.abs(f).sum()


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("m, copies", [(6, 1), (12, 1), (12, 2)])
@pytest.mark.parametrize("L, shift", [(3.0, 0.0), (6.0, 1e-7), (10.0, -1e-7), (12.0, 0.3)])
def test_adjoint_acts_on_both_sides(L, shift, m, copies, prec):
    pos = _lattice(m, L, copies, shift)
    P, Q, gp = _tensors(pos, prec)
    G = torch.as_tensor(np.random.default_rng(1).normal(size=pos.shape), dtype=P.dtype, device="cuda").contiguous()
    R.rbe_forces_vjp(_context(pos.shape[1], L, prec, L / 3), P, Q, G, gp, torch.zeros_like(Q), R.RBE_PART_REAL)
    g = host(gp)
    assert np.abs(g).max() > 0
    assert np.abs(g.sum(1)).max() <= TOL[prec] * np.abs(g).sum()


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("m, copies", [(3, 1), (6, 1), (12, 1), (12, 2)])
@pytest.mark.parametrize("L", [6.0, 7.7])
def test_steps_with_a_list_radius_of_a_third(L, m, copies, prec):
    pos = _lattice(m, L, copies)
    P, Q, F = _tensors(pos, prec)
    skin = 0.1 * L / 3
    r_cut = L / 3 - skin
    ctx = _context(pos.shape[1], L, prec, r_cut, skin)
    V = torch.zeros_like(P)
    R.rbe_step(ctx, P, V, Q, F, 0, 1)
    R.rbe_check(ctx)
    assert R.rbe_list_builds(ctx) == 1
    other, W = _context(pos.shape[1], L, prec, r_cut), torch.zeros_like(F)
    R.rbe_sample_k(other, 0)
    R.rbe_kspace_forces(other, P, Q, W)
    R.rbe_real_forces(other, P, Q, W, accumulate=True)
    assert rel_l2(host(F), host(W)) <= TOL[prec]
    R.rbe_step(ctx, P, V, Q, F, 0, 2)      # from the list
    R.rbe_sample_k(other, 1)
    R.rbe_kspace_forces(other, P, Q, W)
    R.rbe_real_forces(other, P, Q, W, accumulate=True)
    assert rel_l2(host(F), host(W)) <= TOL[prec]
