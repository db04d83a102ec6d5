"""The matrix-core condensation of float32 3D exact bases (the automatic choice
of cc_step, cc_probe_sweep and cc_step_batch): one Jacobi sweep's CC directions
against the oracle on sampled vertices, with and without corotation.

The sizes cover its three configurations and the edges of their tiles: 4 and 8
free vertices (fewer than a workgroup's five, fewer band rows than a chunk's
first), 64 and 128 (whole chunks), 65 and 180, a rod without held vertices, the
41x11x11 bar (enough rows for ten vertices per workgroup; its band fills the
192-position ring) and a 17x17x17 cube (a band too wide for two workgroups per
CU).  Tolerance: 1e-4 of the largest direction, that of float32 local
arithmetic in the other sweep tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from ccscenes import rod_impulse, tet_bar
from oracle import solvers as S
from oracle.basis import basis_matrix, exact_basis
from oracle.fem import Problem
from oracle.timestep import predictor

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SIZES = [(2, 2, 2), (3, 2, 2), (5, 4, 4), (9, 4, 4), (14, 5, 2), (6, 6, 6), "rod", (41, 11, 11), (17, 17, 17)]


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


@pytest.fixture(scope="module")
def cg():
    import paper_2510_12053_amd.ccgpu as cg
    cg.lib()
    return cg


@pytest.mark.parametrize("size", SIZES, ids=str)
def test_directions_against_oracle(cg, size):
    ctx = cg.cc_create(0)
    if size == "rod":
        s = rod_impulse(E=1e4)
    else:
        n = np.array(size) - 1
        s = tet_bar(*size, E=1e6, length=tuple(0.1 * n))
    p = Problem.from_scene(s)
    mid = cg.cc_mesh_upload(ctx, s.X, s.elems, s.fixed, s.E, s.nu, s.rho)
    cg.cc_subspace_build(ctx, mid, 0, s.dt, False)
    x0, v0 = s.initial_state()
    xh = predictor(p, x0, v0 + 0.3, s.targets(1))
    x = xh + 0.005 * np.random.default_rng(3).normal(size=xh.shape)
    x[p.fixed] = xh[p.fixed]
    m = p.free.size
    rng = np.random.default_rng(17)
    ranks = np.unique(np.concatenate([[0, m - 1], rng.choice(m, min(m, 14), replace=False)]))
    Um = basis_matrix(p, *exact_basis(p, verts=p.free[ranks]))
    H, g = p.hessian(x), p.gradient(x)
    for corot in (0, 1):
        par = cg.cc_params_default(method=cg.METHOD_CC, precision=cg.FP32_MIXED, gravity=s.gravity, corotate=corot)
        _, _, dx = cg.cc_probe_sweep(ctx, mid, _t(x), _t(p.x_tilde), s.dt, par)
        Ur = S._basis_at(p, Um, x, S.Params(method=S.CC, corotate=bool(corot)))
        dxo, _ = S.local_directions(p, Ur, H, g, ranks, S.CC)
        assert np.max(np.abs(dx.cpu().numpy()[p.free[ranks]] - dxo)) <= 1e-4 * np.max(np.abs(dxo))
    cg.cc_destroy(ctx)
