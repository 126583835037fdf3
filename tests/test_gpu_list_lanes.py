"""Lanes per particle of the list pass: as the caller sets them (rbe_set_tiles), 4
among them; only a context on which nothing was set chooses by size and list length.
All leave the same state in single precision."""
import ctypes as C

import numpy as np
import pytest

import paper_2010_01559_amd.rbe as R
from paper_2010_01559_amd import workloads as W
from gpu_util import device_state, host, make_ctx

pytestmark = pytest.mark.gpu


def _lanes(ctx):
    v = np.zeros(6, np.int32)
    f = R.lib().rbe_plan_of_context
    f.argtypes = [C.c_void_p, C.c_void_p]
    f.restype = None
    f(ctx.handle, v.ctypes.data)
    return int(v[0])


def _steps(ctx, s, n):
    P, Q, V, F = device_state(ctx, s)
    R.rbe_sample_k(ctx, 0)
    R.rbe_kspace_forces(ctx, P, Q, F)
    R.rbe_real_forces(ctx, P, Q, F, accumulate=True)
    R.rbe_step(ctx, P, V, Q, F, 0, n)
    return host(P), host(V), host(F)


@pytest.mark.parametrize("n, r_cut, default", [(300, 4.0, 32), (4096, 4.0, 16), (8192, 3.5, 8), (16384, 3.5, 4)])
def test_lanes(n, r_cut, default):
    s = W.electrolyte_system("lanes", n, 0.1, 0.5, r_cut, 30, 9)
    out = []
    for split in (0, 1, 2, 4, 8):
        ctx = make_ctx(s, R.RBE_FP32, dt=0.002)
        # (the same Fourier shape for all; setting it does not touch the lanes)
        R.rbe_set_tiles(ctx, rho_block=512, real_split=split)
        assert _lanes(ctx) == (split or default)
        assert R.rbe_get_tiles(ctx)["real_split"] == (split or 4)
        out.append(_steps(ctx, s, 10))
    for o in out[1:]:
        for a, b in zip(out[0], o):
            assert np.array_equal(a, b)


def test_tuning_keeps_the_choice():
    """rbe_autotune sets the Fourier shapes; neither the default lanes nor those that
    were set change with it."""
    s = W.electrolyte_system("lanes", 4096, 0.1, 0.5, 4.0, 30, 9)
    for split, lanes in ((0, 16), (4, 4)):
        ctx = make_ctx(s, R.RBE_FP32)
        if split:
            R.rbe_set_tiles(ctx, real_split=split)
        P, Q, V, F = device_state(ctx, s)
        R.rbe_sample_k(ctx, 0)
        R.rbe_autotune(ctx, P, Q, 1)
        assert _lanes(ctx) == lanes


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("sizes", [[2568], [5130], [5136], [10271], [10272], [20543], [20544], [33] * 40,
                                   [1, 1, 2500, 4999], [64, 8192, 300]])
def test_list_tiles_have_room(sizes, prec):
    """The tiles of every shape of the list pass fit their buffer: sizes around the last
    that takes 32, 16 and 8 lanes by default, batches with many remainders, and one-cell
    systems among list systems."""
    prm = []
    for k, n in enumerate(sizes):
        L = (n / 0.1) ** (1 / 3.0) if n > 100 else 30.0
        prm.append(R.Params(n=n, p=4, box=L, alpha=1.0, r_cut=min(5.0, 0.4 * L), skin=0.3, seed=k, precision=prec))
    ctx = R.rbe_batch_create(prm)
    f = R.lib().rbe_plan_of_context
    f.argtypes = [C.c_void_p, C.c_void_p]
    v = np.zeros(6, np.int32)
    for split in (0, 1, 2, 4, 8):
        R.rbe_set_tiles(ctx, real_split=split)
        f(ctx.handle, v.ctypes.data)
        assert 0 < v[1] <= v[2]
        if len(sizes) == 1:
            assert v[1] == -(-sizes[0] // (256 // v[0]))
