"""The matrix-core condensation of single meshes, in its three configurations: a
61x11x11 bar (ten vertices per workgroup, rows split in two segments), a 36x15x15
one (five, eight waves) and a 19x19x19 cube (five, sixteen waves): one Jacobi
sweep's CC directions against the oracle on sampled vertices, with and without
corotation.  Tolerance: 1e-4 of the largest direction, that of float32 local
arithmetic in the other sweep tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from ccscenes import tet_bar
from oracle import solvers as S
from oracle.basis import basis_matrix, exact_basis
from oracle.fem import Problem
from oracle.timestep import predictor

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


@pytest.mark.parametrize("size", [(61, 11, 11), (36, 15, 15), (19, 19, 19)], ids=str)
def test_directions_against_oracle(size):
    import paper_2510_12053_amd.ccgpu as cg
    ctx = cg.cc_create(0)
    s = tet_bar(*size, E=1e6, length=tuple(0.1 * (np.array(size) - 1)))
    p = Problem.from_scene(s)
    mid = cg.cc_mesh_upload(ctx, s.X, s.elems, s.fixed, s.E, s.nu, s.rho)
    cg.cc_subspace_build(ctx, mid, 0, s.dt, False)
    x0, v0 = s.initial_state()
    xh = predictor(p, x0, v0 + 0.3, s.targets(1))
    x = xh + 0.005 * np.random.default_rng(3).normal(size=xh.shape)
    x[p.fixed] = xh[p.fixed]
    m = p.free.size
    rng = np.random.default_rng(17)
    ranks = np.unique(np.concatenate([[0, m - 1], rng.choice(m, 8, replace=False)]))
    Um = basis_matrix(p, *exact_basis(p, verts=p.free[ranks]))
    H, g = p.hessian(x), p.gradient(x)
    for corot in (0, 1):
        par = cg.cc_params_default(method=cg.METHOD_CC, precision=cg.FP32_MIXED, gravity=s.gravity, corotate=corot)
        _, _, dx = cg.cc_probe_sweep(ctx, mid, _t(x), _t(p.x_tilde), s.dt, par)
        Ur = S._basis_at(p, Um, x, S.Params(method=S.CC, corotate=bool(corot)))
        dxo, _ = S.local_directions(p, Ur, H, g, ranks, S.CC)
        assert np.max(np.abs(dx.cpu().numpy()[p.free[ranks]] - dxo)) <= 1e-4 * np.max(np.abs(dxo))
    cg.cc_destroy(ctx)
