"""Row counts at which the network kernels' grids change: one tile, one past
it, whole workgroups, more tiles than waves (each wave walks several), and
partial gradients that do not fill the sum's 16 slices.  Forward: every row
equals the same row's result in a batch of its own 16 (bit for bit: a row's
arithmetic does not depend on its place).  Gradient: the mean over a batch of
whole tiles equals the mean of its tiles' gradients (float32 sums, 1e-5)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from ccscenes import mlp_init

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def setup():
    import paper_2510_12053_amd.ccgpu as cg
    ctx = cg.cc_create(0)
    rng = np.random.default_rng(5)
    cg.cc_mlp_set(ctx, mlp_init(3) + 0.05 * rng.normal(size=cg.MLP_NPARAM))
    X = torch.tensor(rng.normal(size=(70000, 16)).astype(np.float32), device=DEV)
    T = torch.tensor(rng.normal(size=(70000, 3)).astype(np.float32), device=DEV)
    yield cg, ctx, X, T
    cg.cc_destroy(ctx)


@pytest.mark.parametrize("B", [1, 15, 17, 64, 65, 65536, 65537, 70000])
def test_forward_rows_do_not_depend_on_the_batch(setup, B):
    cg, ctx, X, _ = setup
    Y = cg.cc_mlp_forward(ctx, X[:B])
    for r0 in sorted({0, max(0, B // 2 // 16 * 16), (B - 1) // 16 * 16}):
        r1 = min(B, r0 + 16)
        assert torch.equal(Y[r0:r1], cg.cc_mlp_forward(ctx, X[r0:r1].contiguous()))


@pytest.mark.parametrize("tiles", [1, 2, 5, 17, 63])
def test_gradient_is_the_mean_of_its_tiles(setup, tiles):
    cg, ctx, X, T = setup
    idx = torch.arange(16 * tiles, dtype=torch.int32, device=DEV)
    g, loss = cg.cc_mlp_gradient(ctx, X, T, idx)
    parts = [cg.cc_mlp_gradient(ctx, X, T, idx[16 * k:16 * k + 16].contiguous()) for k in range(tiles)]
    ref = sum(p[0].double() for p in parts) / tiles
    # a tile's gradient scales its output error by 1 / rows before the bfloat16
    # products: for tile counts that are no powers of two the two roundings differ
    tol = 1e-5 if tiles & (tiles - 1) == 0 else 1e-2
    assert float((g.double() - ref).norm()) <= tol * float(ref.norm())
    assert abs(loss - np.mean([p[1] for p in parts])) <= 1e-5 * loss
