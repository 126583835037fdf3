"""Chunk sizes accepted after rbe_reserve_modes: down to a block of particles per compute
unit (64 at least, 512 at most), whatever larger default the context was created with,
and the same forces from them."""
import numpy as np
import pytest
import torch

import paper_2010_01559_amd.rbe as R
from gpu_util import host, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("n, p", [(300, 10), (5000, 60), (150000, 200), (600000, 200), (600000, 20)])
def test_chunks_after_reserving(n, p, prec):
    L = 6.0 if n == 300 else 60.0
    ctx = R.rbe_create(R.Params(n=n, p=p, box=L, alpha=1.0, r_cut=2.9, precision=prec))
    rng = np.random.default_rng(n + p)
    nm = 700
    m = rng.integers(-60, 61, size=(3, nm)).astype(np.int32)    # sparse: summed by mode
    m[0] += (m == 0).all(0)
    R.rbe_reserve_modes(ctx, nm)
    R.rbe_set_k(ctx, m, rng.random(nm) * 1e-3)
    dt = torch.float64 if prec == R.RBE_FP64 else torch.float32
    P = torch.as_tensor(rng.random((3, n)) * L, dtype=dt, device="cuda").contiguous()
    Q = torch.as_tensor(rng.normal(size=n), dtype=dt, device="cuda").contiguous()
    F, G = torch.zeros_like(P), torch.zeros_like(P)
    R.rbe_kspace_forces(ctx, P, Q, F)
    R.rbe_set_tiles(ctx, rho_chunk=min(512, max(64, -(-(-(-n // 256)) // 8) * 8)), rho_block=1024)
    R.rbe_kspace_forces(ctx, P, Q, G)
    assert rel_l2(host(F), host(G)) <= (1e-12 if prec == R.RBE_FP64 else 1e-5)
