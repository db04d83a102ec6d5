"""Device memory of a mesh before it has a dense basis: the buffers that only the
dense condensation reads (tile records, their index arrays, segment sums; 600 bytes
a free vertex) come with the first dense basis.  The 81x21x21 beam, 34,839 free
vertices: the second and third uploads, which allocate the same buffers without the
context's first ones, take 300 MB (8,300 to 8,400 bytes a vertex with the
allocator's 2 MiB steps; 8,640 is half way to what those buffers would add)."""
import pytest

torch = pytest.importorskip("torch")

from ccscenes import twist_beam

pytestmark = pytest.mark.gpu


def test_upload_holds_no_dense_buffers():
    import paper_2510_12053_amd.ccgpu as cg
    s = twist_beam()
    ctx = cg.cc_create(0)
    used = []
    for _ in range(3):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        cg.cc_mesh_upload(ctx, s.X, s.elems, s.fixed, s.E, s.nu, s.rho)
        used.append(free - torch.cuda.mem_get_info()[0])
    cg.cc_destroy(ctx)
    assert max(used[1:]) <= 8640 * s.n
