"""Real space of double precision beside particles without a position (NaN, infinite):
they have no pairs, so the other particles' forces, adjoint, energy and virial are those of
the system without them, on the cell pass and on all pairs."""
import numpy as np
import pytest
import torch

import paper_2010_01559_amd.rbe as R
from gpu_util import host, rel_l2

pytestmark = pytest.mark.gpu


def _run(pos, q, G, L, **kw):
    n = q.shape[0]
    ctx = R.rbe_create(R.Params(n=n, p=4, box=L, alpha=0.5, r_cut=3.0, lj_eps=1.0, lj_sigma=0.5, lj_rcut=1.2,
                                precision=R.RBE_FP64, **kw))
    P, Q, g = (torch.as_tensor(np.ascontiguousarray(a), device="cuda") for a in (pos, q, G))
    F, gp, gq = torch.zeros_like(P), torch.zeros_like(P), torch.zeros_like(Q)
    R.rbe_real_forces(ctx, P, Q, F)
    R.rbe_forces_vjp(ctx, P, Q, g, gp, gq, R.RBE_PART_REAL)
    R.rbe_set_k(ctx, np.array([[1], [0], [0]], np.int32))
    _, (e,) = R.rbe_energy(ctx, P, Q, allow_status=(R.RBE_OK, R.RBE_ERR_NOT_NEUTRAL, R.RBE_ERR_NONFINITE))
    return host(F), host(gp), host(gq), np.array([e["e_real"], e["e_lj"], e["virial"]])


@pytest.mark.parametrize("n, L", [(200, 7.0), (1500, 13.0), (6000, 13.0), (3000, 30.0)])
def test_particles_without_a_position(n, L):
    rng = np.random.default_rng(n)
    g = int(np.ceil(n ** (1 / 3)))
    ax = (np.arange(g) + 0.5) * L / g
    pos = np.stack(np.meshgrid(ax, ax, ax, indexing="ij")).reshape(3, -1)[:, rng.permutation(g ** 3)[:n]]
    pos = pos + (rng.random((3, n)) - 0.5) * 0.2 * L / g
    q, G = rng.normal(size=n), rng.normal(size=(3, n))
    ref = _run(pos, q, G, L)
    bad = pos.copy()
    lost = [3, n // 2, n - 1]
    bad[0, lost[0]] = np.nan
    bad[1, lost[1]] = np.inf
    bad[:, lost[2]] = np.nan
    keep = np.setdiff1d(np.arange(n), lost)
    want = _run(pos[:, keep], q[keep], G[:, keep], L)
    got = _run(bad, q, G, L)
    assert rel_l2(got[0][:, keep], want[0]) <= 1e-12
    assert rel_l2(got[1][:, keep], want[1]) <= 1e-12
    assert rel_l2(got[2][keep], want[2]) <= 1e-12
    assert rel_l2(got[3], want[3]) <= 1e-12
    assert np.isfinite(ref[0]).all()
