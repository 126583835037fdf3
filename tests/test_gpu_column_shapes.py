"""Which lists take the columns, in which shape, and their results: balls, balls with
holes and boxes do; half balls (no slot of the zero mode, so just under half of
the slots), repeated and sparse lists do not; lists with components beyond 28
stage 32 particles per structure-factor block, and those with long columns 32 per
force block.  Structure factors and forces against the FP64 oracle's sums by mode
(1e-12 in double, 1e-5 in single precision)."""
import ctypes as C

import numpy as np
import pytest

import oracle as O
import paper_2010_01559_amd.rbe as R
from paper_2010_01559_amd import workloads as W
from gpu_util import device_state, host, make_ctx, rel_l2, rounded

pytestmark = pytest.mark.gpu

TOL = {R.RBE_FP64: 1e-12, R.RBE_FP32: 1e-5}


def _box(x, y, z):
    m = np.stack(np.meshgrid(np.arange(-x, x + 1), np.arange(-y, y + 1), np.arange(-z, z + 1), indexing="ij"))
    m = m.reshape(3, -1)
    return m[:, (m != 0).any(0)]


def _list(kind, rng):
    m = _box(6, 6, 6)
    m = m[:, (m * m).sum(0) <= 40]
    if kind == "half":
        m = _box(8, 8, 8)
        m = m[:, (m * m).sum(0) <= 70]
        m = m[:, (m[0] > 0) | ((m[0] == 0) & ((m[1] > 0) | ((m[1] == 0) & (m[2] > 0))))]
    elif kind == "holes":
        m = m[:, rng.random(m.shape[1]) < 0.8]
    elif kind == "repeated":
        m = np.concatenate([m, m[:, 5:6]], 1)
    elif kind == "sparse":
        m = _box(9, 9, 9)
        m = m[:, rng.random(m.shape[1]) < 0.2]
    elif kind == "wide":        # 32 particles per structure-factor block
        m = _box(30, 1, 5)
    elif kind == "large":
        m = _box(7, 7, 7)
        m = m[:, (m * m).sum(0) <= 60]
    elif kind == "long":        # and per force block
        m = _box(2, 2, 70)
    elif kind == "edge28":
        m = _box(28, 1, 5)
    return np.ascontiguousarray(m.astype(np.int32))


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("kind, n, columns, rho_nb, force_nb", [
    ("ball", 3100, True, 64, 32), ("half", 3100, False, 0, 0), ("holes", 3100, True, 64, 32),
    ("repeated", 3100, False, 0, 0), ("sparse", 3100, False, 0, 0),
    ("large", 16384, True, 64, 32), ("large", 16385, True, 64, 64),
    ("edge28", 3100, True, 64, 32), ("wide", 1025, True, 32, 32), ("wide", 3100, True, 32, 32),
    ("wide", 3135, True, 32, 32), ("wide", 16400, True, 32, 64), ("long", 16400, True, 64, 32),
])
def test_shapes(kind, n, columns, rho_nb, force_nb, prec):
    rng = np.random.default_rng(n)
    L = 14.0
    s = W.System("cols", n, L, 0.6, 3.0, 10, rng.random((3, n)) * L, rng.normal(size=n), np.zeros((3, n)), 7)
    m = _list(kind, rng)
    assert m.shape[1] > 512
    w = rng.random(m.shape[1]) / (1.0 + (m * m).sum(0))
    ctx = make_ctx(s, prec)
    R.rbe_reserve_modes(ctx, m.shape[1])
    R.rbe_set_k(ctx, m, w)
    v = np.zeros(6, np.int32)
    f = R.lib().rbe_plan_of_context
    f.argtypes = [C.c_void_p, C.c_void_p]
    f(ctx.handle, v.ctypes.data)
    assert (v[3] > 0, v[4], v[5]) == (columns, rho_nb, force_nb)
    P, Q, V, F = device_state(ctx, s)
    pos, q = rounded(s, prec)
    R.rbe_kspace_forces(ctx, P, Q, F)
    assert rel_l2(host(F), O.kspace_force(pos, q, L, m, w)) <= TOL[prec]
    assert rel_l2(R.rbe_get_rho(ctx), np.stack(O.rho(pos, q, L, m), -1)) <= TOL[prec]


@pytest.mark.parametrize("prec", [R.RBE_FP64, R.RBE_FP32])
@pytest.mark.parametrize("n", [1, 65, 97, 1000])
def test_few_groups(n, prec):
    """Contexts whose partials hold fewer groups than the columns would take."""
    rng = np.random.default_rng(n)
    L = 14.0
    s = W.System("cols", n, L, 0.6, 3.0, 10, rng.random((3, n)) * L, rng.normal(size=n), np.zeros((3, n)), 7)
    m = _list("ball", rng)
    w = rng.random(m.shape[1]) / (1.0 + (m * m).sum(0))
    ctx = make_ctx(s, prec)
    R.rbe_set_tiles(ctx, rho_chunk=1024)
    R.rbe_reserve_modes(ctx, m.shape[1])
    R.rbe_set_k(ctx, m, w)
    P, Q, V, F = device_state(ctx, s)
    pos, q = rounded(s, prec)
    R.rbe_kspace_forces(ctx, P, Q, F)
    assert rel_l2(R.rbe_get_rho(ctx), np.stack(O.rho(pos, q, L, m), -1)) <= TOL[prec]
    if n > 1:
        assert rel_l2(host(F), O.kspace_force(pos, q, L, m, w)) <= TOL[prec]
