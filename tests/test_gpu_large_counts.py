"""Pair counts beyond 2^32 in one bin of one class: 2e5 particles of one system in
a batch of 256, whose jobs four blocks share (5e9 pairs each, all in the first
bin).  The particles fill a cube of a quarter of the box, so every pair is
inside r_max = L/2 and the counts are those of the charges alone."""
import pytest
import torch

import paper_2010_01559_amd.rbe as R
from paper_2010_01559_amd import observables as X

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n, minus", [(200000, 0), (200000, 2)])
def test_counts_beyond_32_bits(n, minus):
    L = 10.0
    prm = [R.Params(n=k, p=1, box=L, alpha=1.0, r_cut=3.0, skin=0.0) for k in [n] + [1] * 255]
    ctx = R.rbe_batch_create(prm)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    P = torch.rand((3, n + 255), generator=gen, device="cuda") * (0.25 * L)
    Q = torch.ones(n + 255, device="cuda")
    Q[:minus] = -1.0
    got = X.pair_counts(ctx, P, Q, 0.5 * L, 1).cpu()
    plus = n - minus
    assert got[0, :, 0].tolist() == [plus * (plus - 1) // 2, plus * minus, minus * (minus - 1) // 2]
    assert (got[1:] == 0).all()
