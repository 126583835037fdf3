"""Shifted LJ of eq. (4.1) with per-particle diameters around the reach of a pair,
r_off + R_c: mixed diameters below and above sigma (r_off of either sign) and a cutoff
shorter than sigma (some pairs have no reach at all), on the cell list, the neighbour
list and all pairs, against the FP64 oracle.

Tolerances: those of the real-space force (1e-12 in double, 1e-5 in single precision;
1e-11 for the force a step leaves).
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2010_01559_amd.rbe as R
from paper_2010_01559_amd import workloads as W
from gpu_util import device_state, host, make_ctx, rel_l2, rounded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("r_lj", [0.5, 2.5])
@pytest.mark.parametrize("box,n", [(16.0, 400), (8.5, 60)])
def test_reach_of_mixed_diameters(box, n, r_lj, prec):
    rng = np.random.default_rng(17)
    diam = rng.choice([0.3, 1.0, 2.0], n)
    s = W.System("diam", n, box, 0.6, 3.5, 20, W.positions(n, box, rng, 1.6), W.gaussian_charges(n, rng),
                 rng.normal(size=(3, n)), 3, lj=(1.0, 1.0, r_lj), dt=1e-5, extra={"diameter": diam})
    ctx = make_ctx(s, prec)
    P, Q, V, F = device_state(ctx, s)
    pos, q = rounded(s, prec)
    fp64 = prec == R.RBE_FP64
    R.rbe_real_forces(ctx, P, Q, F)
    fo, _, el = O.real_force(pos, q, s.L, s.alpha, s.r_cut, s.coulomb, s.lj, diam=diam)
    assert el.sum() != 0.0 or r_lj == 0.5   # no pair is within 1.5, the longest reach then
    assert rel_l2(host(F), fo) <= (1e-12 if fp64 else 1e-5)
    R.rbe_sample_k(ctx, 0)
    R.rbe_kspace_forces(ctx, P, Q, F, accumulate=True)
    R.rbe_step(ctx, P, V, Q, F, 1, 3)   # the first step builds the list, the others use it
    x, qs = host(P), host(Q)
    modes, _ = O.sample_modes(s.alpha, s.L, s.p, s.seed, 3)
    fo = O.real_force(x, qs, s.L, s.alpha, s.r_cut, s.coulomb, s.lj, diam=diam)[0]
    fo = fo + O.rbe_kspace_force(x, qs, s.L, s.alpha, modes)
    assert rel_l2(host(F), fo) <= (1e-11 if fp64 else 1e-5)
