"""The exact-basis condensation with its rows' bands split in two segments
(launches short of workgroups) and whole.

Directions of one float64 Jacobi sweep against the oracle where the second
segment is absent (128 free vertices, one chunk), nearly empty (130), as long as
the first (256) and ragged (260, and 255 in 2D).  Tolerance 1e-9 of the largest
direction, that of the other float64 sweep tests.

One step of a single bar, split, against the same bar six times in one batch,
whole: the same sums in another order, so the positions after three iterations
agree to 1e-11 of the largest move in float64 and to 1e-5 of it with float32
local arithmetic (a hundred times 2^-24, for directions whose rounding the
condition of the 3 x 3 systems amplifies)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from ccscenes import stretch2d, tet_bar
from oracle import solvers as S
from oracle.basis import basis_matrix, exact_basis
from oracle.fem import Problem
from oracle.timestep import predictor

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


@pytest.fixture(scope="module")
def cg():
    import paper_2510_12053_amd.ccgpu as cg
    cg.lib()
    return cg


@pytest.mark.parametrize("size", [(9, 4, 4), (14, 5, 2), (17, 4, 4), (14, 5, 4), 17], ids=str)
def test_directions_float64(cg, size):
    ctx = cg.cc_create(0)
    if size == 17:
        s = stretch2d(n=17)
    else:
        s = tet_bar(*size, E=1e6, length=tuple(0.1 * (np.array(size) - 1)))
    p = Problem.from_scene(s)
    mid = cg.cc_mesh_upload(ctx, s.X, s.elems, s.fixed, s.E, s.nu, s.rho)
    cg.cc_subspace_build(ctx, mid, 0, s.dt, s.quasistatic)
    x0, v0 = s.initial_state()
    xh = predictor(p, x0, v0, s.targets(1))
    x = xh + 1e-3 * np.random.default_rng(3).normal(size=xh.shape)
    x[p.fixed] = xh[p.fixed]
    ranks = np.unique(np.linspace(0, p.free.size - 1, 12).astype(int))
    Um = basis_matrix(p, *exact_basis(p, verts=p.free[ranks]))
    H, g = p.hessian(x), p.gradient(x)
    Ur = S._basis_at(p, Um, x, S.Params(method=S.CC))
    want, _ = S.local_directions(p, Ur, H, g, ranks, S.CC)
    par = cg.cc_params_default(method=cg.METHOD_CC, gravity=s.gravity, quasistatic=s.quasistatic)
    dx = cg.cc_probe_sweep(ctx, mid, _t(x), _t(p.x_tilde), s.dt, par)[2].cpu().numpy()[p.free[ranks]]
    assert np.abs(dx - want).max() <= 1e-9 * np.abs(want).max()
    cg.cc_destroy(ctx)


@pytest.mark.parametrize("prec,size,tol", [(0, (21, 6, 6), 1e-11), (1, (29, 9, 7), 1e-5)])
def test_split_step_equals_whole(cg, prec, size, tol):
    ctx = cg.cc_create(0)
    s = tet_bar(*size, E=1e6, length=tuple(0.1 * (np.array(size) - 1)))
    mids = [cg.cc_mesh_upload(ctx, s.X, s.elems, s.fixed, s.E, s.nu, s.rho) for _ in range(6)]
    for m in mids:
        cg.cc_subspace_build(ctx, m, 0, s.dt, False)
    free = ~np.asarray(s.fixed, dtype=bool)
    x0, v0 = (np.array(a) for a in s.initial_state())
    v0[free] += 0.3 * np.random.default_rng(5).normal(size=v0[free].shape)
    par = cg.cc_params_default(method=cg.METHOD_CC, precision=prec, gravity=s.gravity, max_iters=3,
                               corotate=prec)
    x, v = _t(x0), _t(v0)
    cg.cc_step(ctx, mids[0], x, v, None, s.dt, par, 0.0)
    xs, vs = [_t(x0) for _ in mids], [_t(v0) for _ in mids]
    cg.cc_step_batch(ctx, mids, xs, vs, None, s.dt, par, 0.0)
    moved = float((x - _t(x0)).abs().max())
    for y in xs:
        assert float((x - y).abs().max()) <= tol * moved
    cg.cc_destroy(ctx)
