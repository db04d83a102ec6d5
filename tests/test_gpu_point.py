"""Rotations, element Hessians and gradient of a sweep in one launch against the
same kernels one by one (as they are launched while they are timed): two
iterations of a corotated Jacobi sweep, a coloured sweep with Hessians per
colour, and one with Hessians per sweep, of a single mesh and of a batch of two
whose colour counts differ, in both precisions.

Tolerance: the same terms in the same order, so float64 agrees to 1e-12 of the
largest move, and float32 local arithmetic, in case a product is contracted in
one place and not in the other, to 1e-5 of it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from ccscenes import rod_impulse, tet_bar

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


@pytest.fixture(scope="module")
def cg():
    import paper_2510_12053_amd.ccgpu as cg
    cg.lib()
    return cg


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 1e-5)])
@pytest.mark.parametrize("sweep,refresh,corot", [(0, 0, 1), (1, 0, 1), (1, 0, 0), (1, 1, 1)])
def test_one_launch_equals_single_kernels(cg, sweep, refresh, corot, prec, tol, batch):
    scenes = [tet_bar(7, 4, 3, E=1e6, length=(0.6, 0.3, 0.2)), rod_impulse(nx=9, E=1e4, length=0.2)]
    if not batch:
        scenes = scenes[:1]
    ctx = cg.cc_create(0)
    mids = []
    for s in scenes:
        mids.append(cg.cc_mesh_upload(ctx, s.X, s.elems, s.fixed, s.E, s.nu, s.rho))
        cg.cc_subspace_build(ctx, mids[-1], 0, s.dt, False)
    par = cg.cc_params_default(method=cg.METHOD_CC, precision=prec, sweep=sweep, hess_refresh=refresh, corotate=corot,
                               gravity=scenes[0].gravity, max_iters=2)
    rng = np.random.default_rng(9)
    x0 = [np.array(s.initial_state()[0]) for s in scenes]
    v0 = [np.where(np.asarray(s.fixed, dtype=bool)[:, None], 0.0, 0.2 * rng.normal(size=x.shape))
          for s, x in zip(scenes, x0)]
    got = []
    for timed in (False, True):
        xs, vs = [_t(x) for x in x0], [_t(v) for v in v0]
        if timed:
            cg.cc_profile_enable(ctx, 63)
        if batch:
            cg.cc_step_batch(ctx, mids, xs, vs, None, scenes[0].dt, par, 0.0)
        else:
            cg.cc_step(ctx, mids[0], xs[0], vs[0], None, scenes[0].dt, par, 0.0)
        if timed:
            cg.cc_profile_enable(ctx, 0)
        got.append(xs)
    for x, y, a in zip(*got, x0):
        moved = float((x - _t(a)).abs().max())
        assert moved > 0 and float((x - y).abs().max()) <= tol * moved
    cg.cc_destroy(ctx)
