"""A single mesh's line search that goes through many halvings: a stiff bar with a
one-ring patch basis, two of whose eight sweeps find no lower energy in twenty
halvings and fall back to coordinate descent.

The gradient is taken at the points that are mostly accepted (a full step, a first
halving) and at the accepted one, not at every trial point: at most three times an
iteration, six times one that falls back.  Positions, energy and iterations equal
those of the batched path, whose search is another one: the same float64 sums in
another order, 1e-11 of the bar's length and 1e-12 of the energy."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from ccscenes import tet_bar

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def test_failing_sweeps_take_few_gradients():
    import paper_2510_12053_amd.ccgpu as cg
    size = (13, 5, 5)
    s = tet_bar(*size, E=1e7, length=tuple(0.05 * (np.array(size) - 1)))
    free = ~np.asarray(s.fixed, dtype=bool)
    rng = np.random.default_rng(5)
    x0, v0 = (np.array(a) for a in s.initial_state())
    x0[free] += 0.005 * rng.normal(size=x0[free].shape)
    ctx = cg.cc_create(0)
    mid = cg.cc_mesh_upload(ctx, s.X, s.elems, s.fixed, s.E, s.nu, s.rho)
    cg.cc_subspace_build(ctx, mid, 1, s.dt, False)
    par = cg.cc_params_default(method=cg.METHOD_CC, gravity=s.gravity, max_iters=8)
    xb, vb = _t(x0), _t(v0)
    cg.cc_step_batch(ctx, [mid], [xb], [vb], None, s.dt, par, 0.0)
    want = cg.cc_step_info(ctx, mid)
    for timed in (False, True):
        x, v = _t(x0), _t(v0)
        if timed:
            cg.cc_profile_enable(ctx, 63)
        _, it, _ = cg.cc_step(ctx, mid, x, v, None, s.dt, par, 0.0)
        info = cg.cc_step_info(ctx, mid)
        assert it == 8 and info["sweep_fallbacks"] == want["sweep_fallbacks"] > 0
        assert info["halvings"] == want["halvings"]
        assert abs(info["energy"] - want["energy"]) <= 1e-12 * abs(want["energy"])
        assert float((x - xb).abs().max()) <= 1e-11 * 0.6
    gradients, energies = (cg.cc_profile_read(ctx, k)[1] for k in (cg.K_GRADIENT, cg.K_ENERGY))
    cg.cc_profile_enable(ctx, 0)
    failed = info["sweep_fallbacks"]
    assert energies > 20 * failed
    assert gradients <= 1 + 3 * (it - failed) + 6 * failed
    cg.cc_destroy(ctx)
