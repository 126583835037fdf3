"""All-pairs real space (fewer than three cells along the box): one particle
per wave, its partners queued and evaluated 64 at a time.  Particle counts at
the edges of a wave, of a round of candidates and of a block; uniform systems,
where a share of the partners is inside the cutoff, and clusters, where all of
them are (the queue fills completely every round).  Forces, energies, the
adjoint and a short run against the FP64 oracle; tolerances are those of the
real-space force tests (1e-12 in double, 1e-5 in single precision)."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2010_01559_amd.rbe as R
from paper_2010_01559_amd import workloads as W
from gpu_util import check_trajectory, device_state, host, make_ctx, rel_l2, rounded

pytestmark = pytest.mark.gpu

TOL = {R.RBE_FP64: 1e-12, R.RBE_FP32: 1e-5}


def _system(n, cluster, lj=(0.0, 1.0, 2.5)):
    """n charges in a box of side 8 (r_c = 3.9, one cell), uniform or inside a
    ball of diameter 3.5 about a corner (so that it spans the periodic faces)."""
    rng = np.random.default_rng(1000 + n)
    L = 8.0
    if cluster:
        pos = rng.uniform(-1.0, 1.0, (3, n)) * 1.01 % L
    else:
        pos = rng.uniform(0.0, L, (3, n))
    q = W.gaussian_charges(n, rng, 0.5) if n > 1 else np.zeros(1)
    return W.System("allpairs", n, L, 0.6, 3.9, 20, pos, q, rng.normal(size=(3, n)), 11 + n, lj=lj)


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("cluster", [False, True])
@pytest.mark.parametrize("n", [1, 2, 5, 63, 64, 65, 128, 129, 193, 257])
def test_forces_energy_adjoint(n, cluster, prec):
    s = _system(n, cluster)
    ctx = make_ctx(s, prec)
    P, Q, V, F = device_state(ctx, s)
    pos, q = rounded(s, prec)
    R.rbe_real_forces(ctx, P, Q, F)
    Fo, er, _ = O.real_force(pos, q, s.L, s.alpha, s.r_cut, s.coulomb, s.lj)
    if n == 1:
        assert not host(F).any()
        return
    assert rel_l2(host(F), Fo) <= TOL[prec]
    m = torch.zeros((3, s.p), dtype=torch.int32, device="cuda")
    R.rbe_sample_k(ctx, 3, m)
    modes = host(m).astype(np.int32)
    w = O.rbe_weights(s.alpha, s.L, s.p)
    R.rbe_kspace_forces(ctx, P, Q, F, accumulate=True)
    assert rel_l2(host(F), Fo + O.kspace_force(pos, q, s.L, modes, w)) <= TOL[prec]
    st, (e,) = R.rbe_energy(ctx, P, Q, V, allow_status=(R.RBE_OK, R.RBE_ERR_NOT_NEUTRAL))
    assert abs(e["e_real"] - er.sum()) <= (1e-12 if prec == R.RBE_FP64 else 1e-6) * np.abs(er).sum()
    gF = np.random.default_rng(n).normal(size=(3, n))
    G = torch.as_tensor(gF, dtype=P.dtype, device="cuda").contiguous()
    gp, gq = torch.empty_like(P), torch.empty_like(Q)
    R.rbe_forces_vjp(ctx, P, Q, G, gp, gq)
    gqo, gpo = O.forces_vjp(pos, q, s.L, s.alpha, s.r_cut, modes, w, host(G), s.coulomb, s.lj)
    assert rel_l2(host(gp), gpo) <= (1e-10 if prec == R.RBE_FP64 else 1e-5)
    assert rel_l2(host(gq), gqo) <= (1e-10 if prec == R.RBE_FP64 else 1e-5)


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("skin", [0.0, 0.3])
@pytest.mark.parametrize("n", [2, 66, 300])
def test_steps(n, skin, prec):
    """Langevin steps of a one-cell system, with and without a skin."""
    s = W.electrolyte_system(f"ap{n}", n, n / 512.0, 0.6, 3.9, 10, 40 + n, lj=(1.0, 0.4, 1.0), L=8.0)
    ctx = make_ctx(s, prec, skin=skin)
    P, Q, V, F = device_state(ctx, s)
    R.rbe_sample_k(ctx, 0)
    R.rbe_kspace_forces(ctx, P, Q, F)
    R.rbe_real_forces(ctx, P, Q, F, accumulate=True)
    p0 = host(P)
    po, q = rounded(s, prec)
    vo = host(V)
    sysd = O.make_sys(s.n, s.p, s.L, s.alpha, s.r_cut, s.coulomb, s.lj, s.kT, s.gamma, s.dt, s.mass, s.seed)
    po, vo = po.copy(), vo.copy()
    Fo = O.total_force(sysd, po, q, 0)
    R.rbe_step(ctx, P, V, Q, F, 1, 6)
    for k in range(1, 7):
        O.baoab_step(sysd, po, vo, q, Fo, k)
    check_trajectory(prec, P, V, F, po, vo, p0, s.L, lambda x: O.total_force(sysd, x, q, 6))
    if skin > 0.0:
        assert R.rbe_list_builds(ctx) == -1   # a one-cell system keeps no list
