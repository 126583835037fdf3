"""Default structure-factor shape of a context whose list is longer or shorter than the
one it was created for: it follows the list, back and forth, unless rbe_set_tiles
chose it; forces and steps with the fixed sampler stay those of the oracle."""
import numpy as np
import pytest

import oracle as O
import paper_2010_01559_amd.rbe as R
from paper_2010_01559_amd import workloads as W
from gpu_util import device_state, host, make_ctx, rel_l2, rounded

pytestmark = pytest.mark.gpu

TOL = {R.RBE_FP64: 1e-12, R.RBE_FP32: 1e-5}


def _shape(ctx):
    t = R.rbe_get_tiles(ctx)
    return t["rho_chunk"], t["rho_block"]


def _modes(nm, rng):
    m = rng.integers(-40, 41, size=(3, nm)).astype(np.int32)     # sparse: summed by mode
    m[0] += (m == 0).all(0)
    return m


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("n, p, first, nm, then", [
    (300, 10, (128, 256), 513, (64, 1024)),      # one cell: also the chunk
    (300, 10, (128, 256), 401, (64, 1024)),
    (300, 10, (128, 256), 400, (64, 512)),
    (30000, 100, (120, 512), 300, (120, 1024)),
    (5000, 10, (64, 256), 63, (64, 256)),
    (5000, 10, (64, 256), 64, (64, 512)),
    (5000, 10, (64, 256), 700, (64, 1024)),
    (5000, 700, (64, 1024), 20, (64, 256)),
])
def test_shape_follows_the_list(n, p, first, nm, then, prec):
    rng = np.random.default_rng(n + nm)
    L = 7.0 if n == 300 else 30.0
    s = W.System("long", n, L, 1.0, 3.0, p, rng.random((3, n)) * L, rng.normal(size=n), np.zeros((3, n)), 7)
    if n == 300 and prec == R.RBE_FP64:
        s.p = p = 4
    ctx = make_ctx(s, prec)
    assert _shape(ctx) == first
    P, Q, V, F = device_state(ctx, s)
    pos, q = rounded(s, prec)
    m, w = _modes(nm, rng), rng.random(nm) * 1e-3
    R.rbe_reserve_modes(ctx, max(nm, p))
    R.rbe_set_k(ctx, m, w)
    assert _shape(ctx) == then
    R.rbe_kspace_forces(ctx, P, Q, F)
    assert rel_l2(host(F), O.kspace_force(pos, q, L, m, w)) <= TOL[prec]
    R.rbe_sample_k(ctx, 3)
    assert _shape(ctx) == first
    R.rbe_kspace_forces(ctx, P, Q, F)
    md, _ = O.sample_modes(s.alpha, L, p, s.seed, 3)
    assert rel_l2(host(F), O.rbe_kspace_force(pos, q, L, s.alpha, md)) <= TOL[prec]
    R.rbe_set_tiles(ctx, rho_block=512)
    R.rbe_set_k(ctx, m, w)
    assert _shape(ctx) == (first[0], 512)
    R.rbe_kspace_forces(ctx, P, Q, F)
    assert rel_l2(host(F), O.kspace_force(pos, q, L, m, w)) <= TOL[prec]


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("n, L", [(300, 7.0), (2000, 27.0)])
def test_fixed_sampler_steps(n, L, prec):
    """One step with a long list: the force it leaves is the oracle's at its positions."""
    rng = np.random.default_rng(n)
    g = int(np.ceil(n ** (1 / 3)))
    ax = (np.arange(g) + 0.5) * L / g
    pos = np.stack(np.meshgrid(ax, ax, ax, indexing="ij")).reshape(3, -1)[:, :n] + rng.random((3, n)) * 0.1
    q = np.where(np.arange(n) % 2 == 0, 1.0, -1.0)
    s = W.System("fixed", n, L, 1.0, 3.0, 10, pos, q, rng.normal(size=(3, n)), 7, lj=(0.0, 1.0, 2.5))
    ctx = make_ctx(s, prec, sampler=R.RBE_SAMPLER_FIXED, dt=1e-3)
    m, w = _modes(700, rng), rng.random(700) * 1e-2
    R.rbe_reserve_modes(ctx, 700)
    R.rbe_set_k(ctx, m, w)
    P, Q, V, F = device_state(ctx, s)
    R.rbe_kspace_forces(ctx, P, Q, F)
    R.rbe_real_forces(ctx, P, Q, F, accumulate=True)
    R.rbe_step(ctx, P, V, Q, F, 1, 3)
    x, qq = host(P), host(Q)
    Fo = O.kspace_force(x, qq, L, m, w) + O.real_force(x, qq, L, s.alpha, s.r_cut, lj=(0.0, 1.0, 2.5))[0]
    assert rel_l2(host(F), Fo) <= (1e-11 if prec == R.RBE_FP64 else 1e-5)
