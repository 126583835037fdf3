"""rbe_kspace_forces_noalloc equals a context bit for bit also where the context was
created for another number of modes than the list that rbe_set_k made active, on both
sides of the size (2^23 particle-mode terms) from which single precision takes the
structure factor in polar form."""
import numpy as np
import pytest
import torch

import paper_2010_01559_amd.rbe as R

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("n, p_created, p_used", [(131072, 1, 64), (131072, 100, 63), (65536, 128, 10), (65537, 10, 128)])
def test_same_bits_as_a_context(n, p_created, p_used, prec):
    L = 40.0
    kw = dict(n=n, box=L, alpha=0.6, r_cut=3.0, precision=prec)
    ctx = R.rbe_create(R.Params(p=p_created, **kw))
    chunk = min(512, max(64, -(-(-(-n // 256)) // 8) * 8))
    R.rbe_set_tiles(ctx, rho_chunk=chunk, rho_block=1024, force_split=4)
    rng = np.random.default_rng(n + p_used)
    m = rng.integers(-7, 8, size=(3, p_used)).astype(np.int32)
    m[0] += (m == 0).all(0)
    if p_used > p_created:
        R.rbe_reserve_modes(ctx, p_used)
    R.rbe_set_k(ctx, m)
    dt = torch.float64 if prec == R.RBE_FP64 else torch.float32
    P = torch.as_tensor(rng.random((3, n)) * L, dtype=dt, device="cuda").contiguous()
    Q = torch.as_tensor(rng.normal(size=n), dtype=dt, device="cuda").contiguous()
    F, G = torch.zeros_like(P), torch.zeros_like(P)
    R.rbe_kspace_forces(ctx, P, Q, F)
    M = torch.as_tensor(m, device="cuda").contiguous()
    R.rbe_kspace_forces_noalloc(R.Params(p=p_used, **kw), M, P, Q, G)
    torch.cuda.synchronize()
    assert F.abs().max() > 0
    assert torch.equal(F, G)
