"""Direction records against the node records they copy, at row lengths around
the kernel's chunk of 256 cells."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(2, 2, 2), (7, 5, 3), (256, 3, 4), (257, 4, 3), (258, 3, 3), (515, 2, 3)])
def test_direction_records(n):
    import torch

    import paper_1609_00724_amd as q
    g = np.random.default_rng(sum(n))
    b = [torch.from_numpy(g.standard_normal(n[::-1]).astype(np.float32)).cuda() for _ in range(3)]
    f = q.field_init(*b, (0, 0, 0), (1, 1, 1)).add_cell_dirs()
    torch.cuda.synchronize()
    nx, ny, nz = n
    nodes = f.ws.view(torch.float32)[:4 * nx * ny * nz].reshape(nz, ny, nx, 4)
    want = torch.stack([nodes[c:nz - 1 + c, b_:ny - 1 + b_, a:nx - 1 + a, :3]
                        for c in (0, 1) for b_ in (0, 1) for a in (0, 1)], 3)
    got = f.dirs_ws.view(torch.float32)[:want.numel()].reshape(want.shape)
    assert torch.equal(got, want)


# rows of one layer together: whole groups and a remainder, the longest row that
# still pairs (128 cells), the shortest (1), and long rows in equal stretches
@pytest.mark.parametrize("n", [(2, 300, 3), (3, 129, 2), (9, 40, 3), (18, 33, 3), (86, 8, 3), (129, 6, 3), (130, 4, 3), (771, 3, 3)])
def test_direction_records_of_short_and_uneven_rows(n):
    test_direction_records(n)
