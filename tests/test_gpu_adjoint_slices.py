"""Adjoint of the Fourier part where the partial sums of all modes do not fit at once:
large single systems at the smallest chunk, which take the modes in slices, down to
one mode at a time."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2010_01559_amd.rbe as R
from paper_2010_01559_amd import workloads as W
from gpu_util import device_state, host, make_ctx, rel_l2, rounded

pytestmark = pytest.mark.gpu

TOL = {R.RBE_FP64: 1e-10, R.RBE_FP32: 1e-5}


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("n, p, chunk", [(65536, 1, 64), (65601, 1, 120), (65536, 3, 64), (70000, 2, 0)])
def test_slices(n, p, chunk, prec):
    rng = np.random.default_rng(n + p)
    L = 30.0
    s = W.System("slices", n, L, 0.6, 3.0, p, rng.random((3, n)) * L, rng.normal(size=n), np.zeros((3, n)), 5)
    ctx = make_ctx(s, prec)
    if chunk:
        R.rbe_set_tiles(ctx, rho_chunk=chunk)
    P, Q, V, F = device_state(ctx, s)
    pos, q = rounded(s, prec)
    m = rng.integers(-6, 7, size=(3, p)).astype(np.int32)
    m[0] += (m == 0).all(0)
    R.rbe_set_k(ctx, m)
    G = torch.as_tensor(rng.normal(size=(3, n)), dtype=P.dtype, device="cuda").contiguous()
    gp, gq = torch.empty_like(P), torch.empty_like(Q)
    R.rbe_forces_vjp(ctx, P, Q, G, gp, gq, R.RBE_PART_KSPACE)
    gqo, gpo = O.forces_vjp(pos, q, L, s.alpha, s.r_cut, m, O.rbe_weights(s.alpha, L, p), host(G),
                            parts=R.RBE_PART_KSPACE)
    assert rel_l2(host(gp), gpo) <= TOL[prec]
    assert rel_l2(host(gq), gqo) <= TOL[prec]
