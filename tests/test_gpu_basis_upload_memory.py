"""Host memory of cc_subspace_upload for a dense basis: its own copies are the sorted
rows and the band layout in float64 and the band layout once in float32, 20 bytes
for each of the basis's values, and no second float32 copy (24).  A 14x9x9 bar
(1,053 free vertices, 10 million values), resident memory sampled during the call;
22 bytes a value, and the basis arrives as it was."""
import threading
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from ccscenes import tet_bar

pytestmark = pytest.mark.gpu


def _rss():
    with open("/proc/self/statm") as f:
        return int(f.read().split()[1]) * 4096


def test_dense_upload_holds_one_float32_copy():
    import paper_2510_12053_amd.ccgpu as cg
    s = tet_bar(14, 9, 9, E=1e6, length=(1.3, 0.8, 0.8))
    ctx = cg.cc_create(0)
    mid = cg.cc_mesh_upload(ctx, s.X, s.elems, s.fixed, s.E, s.nu, s.rho)
    cg.cc_subspace_build(ctx, mid, 0, s.dt, False)
    ptr, idx, U = cg.cc_subspace_download(ctx, mid, s.n, 3)
    cg.cc_subspace_upload(ctx, mid, ptr, idx, U, s.dt)      # the runtime's staging buffers
    peak, done = [_rss()], threading.Event()

    def sample():
        while not done.is_set():
            peak[0] = max(peak[0], _rss())
            time.sleep(5e-4)
    start = peak[0]
    t = threading.Thread(target=sample)
    t.start()
    cg.cc_subspace_upload(ctx, mid, ptr, idx, U, s.dt)
    done.set()
    t.join()
    values = 9 * 1053 ** 2
    assert peak[0] - start <= 22 * values
    back = cg.cc_subspace_download(ctx, mid, s.n, 3)
    np.testing.assert_array_equal(back[2], U)
    cg.cc_destroy(ctx)
