"""Dense mode lists (rbe_set_k with the modes of a ball, or most of one) on the
matrix cores: structure factors, forces, energies and the adjoint against the FP64
oracle's sums by mode.  Lists: whole balls of radii on both sides of a 16- and a
32-row tile of cosines and sines, half balls (no mode with its negative), balls
with holes, shuffled, with weights that differ between m and -m, boxes of one long
column; a list with a repeated mode and a sparse one keep the sums by mode.
Particle counts at the edges of a tile, a chunk and a group.  Tolerances are those
of the Fourier tests (1e-12 in double, 1e-5 in single precision)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2010_01559_amd.rbe as R
from paper_2010_01559_amd import workloads as W
from gpu_util import device_state, host, make_ctx, rel_l2, rounded

pytestmark = pytest.mark.gpu

TOL = {R.RBE_FP64: 1e-12, R.RBE_FP32: 1e-5}


def _ball(r2):
    k = int(np.sqrt(r2))
    ax = np.arange(-k, k + 1)
    m = np.stack(np.meshgrid(ax, ax, ax, indexing="ij")).reshape(3, -1)
    s = (m * m).sum(0)
    return m[:, (s > 0) & (s <= r2)].astype(np.int32)


def _list(kind, r2, rng):
    m = _ball(r2)
    if kind == "half":
        m = m[:, (m[0] > 0) | ((m[0] == 0) & ((m[1] > 0) | ((m[1] == 0) & (m[2] > 0))))]
    elif kind == "holes":
        m = m[:, rng.random(m.shape[1]) < 0.8]
        m = m[:, rng.permutation(m.shape[1])]
    elif kind == "repeated":
        m = np.concatenate([m, m[:, 5:6]], 1)
    elif kind == "sparse":
        m = m[:, rng.random(m.shape[1]) < 0.2]
    elif kind == "column":
        z = np.concatenate([np.arange(-80, 0), np.arange(1, 81)])
        m = np.concatenate([np.stack([np.full(160, a), np.full(160, b), z]) for a in (-1, 0, 1) for b in (-1, 0, 1)], 1)
    return np.ascontiguousarray(m.astype(np.int32))


def _check(n, kind, r2, prec):
    rng = np.random.default_rng(n + r2)
    L = 14.0
    s = W.System("cols", n, L, 0.6, 3.0, 10, rng.random((3, n)) * L * 3 - L, rng.normal(size=n), np.zeros((3, n)), 7)
    m = _list(kind, r2, rng)
    w = rng.random(m.shape[1]) * np.exp(-(m * m).sum(0) / (1.0 + 0.3 * (m * m).sum(0).max()))
    ctx = make_ctx(s, prec)
    P, Q, V, F = device_state(ctx, s)
    pos, q = rounded(s, prec)
    R.rbe_reserve_modes(ctx, m.shape[1])
    R.rbe_set_k(ctx, m, w)
    R.rbe_kspace_forces(ctx, P, Q, F)
    Fo = O.kspace_force(pos, q, L, m, w)
    tol = TOL[prec]
    if n == 1:
        # a lone particle's force vanishes: against the size of the terms that cancel
        terms = q[0] ** 2 * (w * 2.0 / np.sqrt((m * m).sum(0))).sum() / L ** 2
        assert np.abs(host(F)).max() <= tol * terms
        return
    assert rel_l2(host(F), Fo) <= tol
    assert rel_l2(R.rbe_get_rho(ctx), np.stack(O.rho(pos, q, L, m), -1)) <= tol
    R.rbe_kspace_forces(ctx, P, Q, F, accumulate=True)
    assert rel_l2(host(F), 2 * Fo) <= tol
    st, (e,) = R.rbe_energy(ctx, P, Q, V, allow_status=(R.RBE_OK, R.RBE_ERR_NOT_NEUTRAL))
    assert e["e_kspace"] == pytest.approx(O.kspace_energy(pos, q, L, m, w), rel=1e-11 if prec == R.RBE_FP64 else 1e-5)
    gF = np.random.default_rng(1).normal(size=(3, n))
    G = torch.as_tensor(gF, dtype=P.dtype, device="cuda").contiguous()
    gp, gq = torch.empty_like(P), torch.empty_like(Q)
    R.rbe_forces_vjp(ctx, P, Q, G, gp, gq, R.RBE_PART_KSPACE)
    gqo, gpo = O.forces_vjp(pos, q, L, s.alpha, s.r_cut, m, w, host(G), parts=R.RBE_PART_KSPACE)
    assert rel_l2(host(gp), gpo) <= (1e-10 if prec == R.RBE_FP64 else 1e-5)
    assert rel_l2(host(gq), gqo) <= (1e-10 if prec == R.RBE_FP64 else 1e-5)
    # a fresh sample afterwards leaves the columns
    modes = torch.zeros((3, s.p), dtype=torch.int32, device="cuda")
    R.rbe_sample_k(ctx, 4, modes)
    R.rbe_kspace_forces(ctx, P, Q, F)
    assert rel_l2(host(F), O.kspace_force(pos, q, L, host(modes).astype(np.int32),
                                          O.rbe_weights(s.alpha, L, s.p))) <= tol


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("kind", ["ball", "half", "holes", "repeated", "sparse", "column"])
def test_lists(kind, prec):
    _check(200, kind, 70, prec)


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("r2", [30, 56, 64, 15 * 15, 16 * 16 + 3, 33 * 33])
def test_radii(r2, prec):
    _check(97, "ball", r2, prec)


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("n", [1, 15, 16, 33, 64, 65, 128, 1025, 16384, 16450])
def test_particle_counts(n, prec):
    _check(n, "ball", 40, prec)
