"""Batches whose meshes do not share a condensation launch, or not the kernel that
each would take alone.

  few:    three small bars beside a short one with a wide section: too few rows for
          the tiles, the band kernel for all;
  many:   four 41x11x11 bars, which fill the chip, beside it: two launches, tiles
          for the bars;
  cube:   a 17x17x17 cube, for whose launch the band kernel is the better one,
          beside two small bars: the band kernel for all;
  both:   the cube and four 41x11x11 bars: the band kernel and the tiles;
  wide:   a 19x19x19 cube, for which the tiles are the better ones, beside two small
          bars: one launch in its configuration;
  tiny:   two 41x11x11 bars and six of 4 to 180 free vertices: one launch of ten
          vertices per workgroup;
  mid:    two 25x15x15 bars and the six: one launch of five vertices per workgroup;
  long:   a mesh with a row of more than eight upper blocks (no tile records)
          beside two small bars: the band kernel for all.

One Jacobi or coloured sweep (the band kernel, except for twelve 41x11x11 bars) at
full steps, corotated, float32 local arithmetic, from the predictor, against the same sweep of
each mesh by itself in float64.  Tolerance: 1e-4 of the largest displacement, that
of float32 local arithmetic in the other sweep tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from ccscenes import tet_bar

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def _bar(*size, **kw):
    s = tet_bar(*size, E=1e6, **dict(dict(length=tuple(0.1 * (np.array(size) - 1))), **kw))
    return s.X, s.elems, np.asarray(s.fixed, dtype=bool)


def _star(*shape):
    """A bar whose middle vertex is joined to the whole surface of the eight cells
    around it: 26 neighbours."""
    X, el, fixed = _bar(*shape)
    nx, ny, nz = shape
    hub = (nx // 2) + nx * ((ny // 2) + ny * (nz // 2))
    i, j, k = hub % nx, hub // nx % ny, hub // (nx * ny)
    at = np.arange(len(X))
    ai, aj, ak = at % nx, at // nx % ny, at // (nx * ny)
    near = (abs(ai - i) <= 1) & (abs(aj - j) <= 1) & (abs(ak - k) <= 1)
    keep = ~np.all(near[el], axis=1)                 # the eight cells around the hub go ...
    faces = {}
    for t in el[~keep]:
        for a in range(4):
            f = tuple(np.delete(t, a))
            faces.setdefault(tuple(sorted(f)), []).append(f)
    star = [(hub, *f[0]) for key, f in faces.items() if len(f) == 1]   # ... and their surface is joined to it
    star = np.array(star, dtype=np.int32)
    D = X[star[:, 1:]] - X[star[:, :1]]
    flip = np.linalg.det(D) < 0
    star[flip, 2], star[flip, 3] = star[flip, 3].copy(), star[flip, 2].copy()
    return X, np.concatenate([el[keep], star]).astype(np.int32), fixed


WIDE = ((4, 17, 17), dict(length=(1.05, 1.0, 1.0)))
TINY = lambda: [_bar(*d) for d in [(2, 2, 2), (3, 2, 2), (5, 4, 4), (9, 4, 4), (14, 5, 2), (6, 6, 6)]]
SETS = {
    "few": lambda: [_bar(7, 4, 4), _bar(*WIDE[0], **WIDE[1]), _bar(12, 5, 3), _bar(9, 6, 6)],
    "many": lambda: [_bar(41, 11, 11)] * 2 + [_bar(*WIDE[0], **WIDE[1])] + [_bar(41, 11, 11)] * 2,
    "cube": lambda: [_bar(7, 4, 4), _bar(17, 17, 17), _bar(9, 6, 6)],
    "both": lambda: [_bar(41, 11, 11)] * 3 + [_bar(17, 17, 17), _bar(41, 11, 11)],
    "wide": lambda: [_bar(7, 4, 4), _bar(19, 19, 19), _bar(9, 6, 6)],
    "tiny": lambda: [_bar(41, 11, 11)] * 2 + TINY(),
    "mid": lambda: [_bar(25, 15, 15)] * 2 + TINY(),
    "long": lambda: [_bar(7, 4, 4), _star(9, 5, 5), _bar(9, 6, 6)],
}


@pytest.fixture(scope="module")
def cg():
    import paper_2510_12053_amd.ccgpu as cg
    cg.lib()
    return cg


@pytest.mark.parametrize("name,sweep", [(n, w) for n in SETS for w in (0, 1)] + [("twelve", 1)])
def test_batch_against_float64_of_each_mesh(cg, name, sweep):
    meshes = SETS[name]() if name in SETS else [_bar(41, 11, 11)] * 12
    dt = 1.0 / 60
    ctx = cg.cc_create(0)
    mids = []
    for X, el, fixed in meshes:
        mids.append(cg.cc_mesh_upload(ctx, X, el, fixed, 1e6, 0.45, 1000.0))
        cg.cc_subspace_build(ctx, mids[-1], 0, dt, False)
    rng = np.random.default_rng(11)
    x0 = [X.copy() for X, _, _ in meshes]
    v0 = [np.where(fixed[:, None], 0.0, 0.3 * rng.normal(size=X.shape)) for X, _, fixed in meshes]
    par = [cg.cc_params_default(method=cg.METHOD_CC, precision=p, sweep=sweep, corotate=1, max_iters=1, line_search=0,
                                gravity=(0.0, -9.81, 0.0)) for p in (cg.FP64, cg.FP32_MIXED)]
    xs, vs = [_t(x) for x in x0], [_t(v) for v in v0]
    cg.cc_step_batch(ctx, mids, xs, vs, None, dt, par[1], 0.0)
    for m, x, v, got in zip(mids, x0, v0, xs):
        want, vr = _t(x), _t(v)
        cg.cc_step(ctx, m, want, vr, None, dt, par[0], 0.0)
        moved = float((want - _t(x + dt * v)).abs().max())
        assert moved > 0 and float((got - want).abs().max()) <= 1e-4 * moved
    cg.cc_destroy(ctx)
