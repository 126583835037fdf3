"""Pair counts at the edges of their jobs (particle counts around the tile and
the chunk sizes), with every pair exactly on a bin edge, with bins finer than
32-bit box fractions resolve, and with coordinates far outside the box or not
finite: every count equals the oracle's enumeration of the definition."""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2010_01559_amd.rbe as R
from paper_2010_01559_amd import observables as X
from paper_2010_01559_amd import workloads as W
from gpu_util import make_ctx

pytestmark = pytest.mark.gpu

PREC = [R.RBE_FP64, R.RBE_FP32]


def _counts(prec, pos, q, L, r_max, nbins):
    n = q.shape[0]
    s = W.System("h", n, L, 1.0, 0.4 * L if 0.4 * L < 3 else 3.0, 10, pos, q, np.zeros((3, n)), 1)
    ctx = make_ctx(s, prec)
    dt = torch.float64 if prec == R.RBE_FP64 else torch.float32
    P = torch.as_tensor(np.ascontiguousarray(pos), dtype=dt, device="cuda").contiguous()
    Q = torch.as_tensor(q, dtype=dt, device="cuda").contiguous()
    got = X.pair_counts(ctx, P, Q, r_max, nbins).cpu().numpy()[0]
    return got, P.double().cpu().numpy(), Q.double().cpu().numpy()


@pytest.mark.parametrize("prec", PREC)
@pytest.mark.parametrize("n", [1, 2, 16, 17, 255, 256, 257, 2047, 2048, 2113, 8191, 8192, 8449])
def test_sizes(n, prec):
    rng = np.random.default_rng(n)
    L = 11.0
    pos, q = rng.random((3, n)) * L, rng.normal(size=n)
    got, p, qq = _counts(prec, pos, q, L, 0.5 * L, 90)
    assert np.array_equal(got, O.pair_histogram(p, qq, L, 0.5 * L, 90))


@pytest.mark.parametrize("prec", PREC)
@pytest.mark.parametrize("nbins", [16, 4096])
def test_every_pair_on_an_edge(nbins, prec):
    ax = np.arange(10, dtype=float)
    pos = np.stack(np.meshgrid(ax, ax, ax, indexing="ij")).reshape(3, -1)
    q = np.where(pos.sum(0) % 2 == 0, 1.0, -1.0)
    got, p, qq = _counts(prec, pos, q, 10.0, 4.0, nbins)
    assert np.array_equal(got, O.pair_histogram(p, qq, 10.0, 4.0, nbins))


@pytest.mark.parametrize("prec", PREC)
def test_bins_finer_than_the_fractions(prec):
    rng = np.random.default_rng(4)
    L = 1000.0
    pos = 500.0 + rng.normal(size=(3, 600)) * 1e-6
    got, p, qq = _counts(prec, pos, rng.normal(size=600), L, 4e-6, 500)
    assert np.array_equal(got, O.pair_histogram(p, qq, L, 4e-6, 500))


@pytest.mark.parametrize("prec", PREC)
def test_far_and_nonfinite_positions(prec):
    rng = np.random.default_rng(5)
    n, L = 700, 9.0
    pos, q = rng.random((3, n)) * L, rng.normal(size=n)
    pos[:, ::5] += np.round(rng.normal(size=(3, n))[:, ::5] * 1e3) * L
    pos[:, 1::50] += np.round(rng.normal(size=(3, n))[:, 1::50] * 1e9) * L
    got, p, qq = _counts(prec, pos, q, L, 4.4, 64)
    ref = O.pair_histogram(p, qq, L, 4.4, 64)
    assert np.array_equal(got, ref)
    # a particle without a position adds no pair
    pos2 = np.concatenate([pos, np.array([[np.nan], [1.0], [2.0]]), np.array([[1.0], [np.inf], [2.0]])], 1)
    got2, _, _ = _counts(prec, pos2, np.concatenate([q, [1.0, -1.0]]), L, 4.4, 64)
    assert np.array_equal(got2, ref)
