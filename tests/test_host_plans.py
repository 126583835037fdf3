"""Bounds of the library's launch shapes and workspaces, as host arithmetic over the
whole range of sizes a context accepts (no device)."""
import ctypes as C

import numpy as np
import pytest

import paper_2010_01559_amd.rbe as R


def _sizes(limit):
    out, n = set(), 1
    while n <= limit:
        out |= {n - 1, n, n + 1, n + n // 3}
        n *= 2
    return sorted(k for k in out | {limit} if 1 <= k <= limit)


@pytest.mark.parametrize("nsys", [1, 2, 3, 16, 63, 64, 65, 256, 1000])
def test_pair_count_counters_do_not_wrap(nsys):
    """Between two flushes a block adds at most flush * tile * jw to one 32-bit
    counter; and a block of the largest systems does flush that often."""
    f = R.lib().rbe_plan_pair_hist
    f.argtypes = [C.c_int64, C.c_int32] + [C.c_void_p] * 4
    f.restype = None
    v = (C.c_int32 * 4)()
    for n in _sizes(2 ** 31 - 1):
        f(n, nsys, *(C.addressof(v) + 4 * k for k in range(4)))
        tile, jw, blocks, flush = v
        assert jw in (16, 64, 256) and blocks >= 1 and flush >= 1
        assert flush * tile * jw < 2 ** 32
        assert (flush + 1) * tile * jw >= 2 ** 32 - 1   # and no more often than it has to


@pytest.mark.parametrize("p", [1, 2, 3, 17, 100, 512])
@pytest.mark.parametrize("chunk", [64, 72, 120, 128, 256, 1024])
def test_adjoint_partials_fit(chunk, p):
    """Every slice of the modes has room for its four sums per tile and mode, for
    every mode count up to the capacity and any chunk a caller may set."""
    f = R.lib().rbe_plan_adjoint
    f.argtypes = [C.c_int32] * 4 + [C.c_void_p] * 2
    f.restype = None
    room, slices = C.c_int64(), C.c_int32()
    for n in _sizes(2 ** 27) + [65535, 65536, 70001]:
        tiles = -(-n // chunk)
        for modes in {1, (p + 1) // 2, p}:
            f(n, p, chunk, modes, C.addressof(room), C.addressof(slices))
            k = slices.value
            assert 1 <= k <= modes
            widest = max(modes * (i + 1) // k - modes * i // k for i in range(k))
            assert 4 * tiles * widest <= room.value
            assert room.value >= 2 * -(-n // 64) * p   # the structure factor's own


def _columns(m, n, room=1 << 40, prec=R.RBE_FP64):
    f = R.lib().rbe_plan_columns
    f.argtypes = [C.c_void_p, C.c_int32, C.c_int64, C.c_int32, C.c_int64, C.c_void_p]
    f.restype = None
    m = np.ascontiguousarray(m, np.int32)
    out = np.zeros(5, np.int32)
    f(m.ctypes.data, m.shape[1], n, prec, room, out.ctypes.data)
    return dict(zip(("ncols", "slots", "rho_nb", "force_nb", "groups"), out.tolist()))


def _ball(r2):
    k = int(np.sqrt(r2))
    ax = np.arange(-k, k + 1)
    m = np.stack(np.meshgrid(ax, ax, ax, indexing="ij")).reshape(3, -1)
    s = (m * m).sum(0)
    return m[:, (s > 0) & (s <= r2)].astype(np.int32)


@pytest.mark.parametrize("component", [0, 1, 2])
@pytest.mark.parametrize("value", [129, -129, 2 ** 31 - 1, -2 ** 31 + 1, -2 ** 31])
def test_lists_with_a_far_mode_keep_the_sums_by_mode(value, component):
    m = _ball(40)
    assert m.shape[1] > 512 and _columns(m, 5000)["ncols"] > 0
    m[component, 100] = value
    assert _columns(m, 5000)["ncols"] == 0


@pytest.mark.parametrize("r2, n", [(r2, n) for r2 in (30, 40, 150, 33 * 33) for n in (64, 97, 1000, 1025, 30000, 10 ** 6)
                                   if n >= 512 or r2 <= 150])
def test_column_groups_fit_the_partials(r2, n):
    """A dense list keeps its columns whatever room the sums by mode left for the
    partials (two doubles per mode at least): fewer groups share it."""
    m = _ball(r2)
    free = _columns(m, n)
    assert free["ncols"] > 0
    for room in (2 * m.shape[1], 2 * m.shape[1] * 2, 2 * m.shape[1] * 100, 1 << 40):
        c = _columns(m, n, room)
        assert c["ncols"] == free["ncols"] and c["rho_nb"] == free["rho_nb"]
        assert 1 <= c["groups"] <= free["groups"] and 2 * c["slots"] * c["groups"] <= room


@pytest.mark.parametrize("prec, n, r2, columns", [
    (R.RBE_FP32, 64, 80, True), (R.RBE_FP32, 64, 150, False), (R.RBE_FP32, 3499, 150, False),
    (R.RBE_FP32, 3500, 150, True), (R.RBE_FP32, 6000, 28, True), (R.RBE_FP32, 6001, 28, False),
    (R.RBE_FP32, 30000, 40, False), (R.RBE_FP32, 30000, 60, True), (R.RBE_FP32, 10 ** 6, 25, False),
    (R.RBE_FP64, 64, 25, True), (R.RBE_FP64, 511, 250, True), (R.RBE_FP64, 511, 400, False),
    (R.RBE_FP64, 512, 400, True), (R.RBE_FP64, 10 ** 6, 25, True),
])
def test_columns_only_where_they_are_faster(prec, n, r2, columns):
    """Both sides of each measured line: few particles with long lists, and in single
    precision many particles with short ones, keep the sums by mode."""
    assert (_columns(_ball(r2), n, prec=prec)["ncols"] > 0) == columns
