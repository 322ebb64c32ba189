"""Every stencil tile of two dimensions is computed exactly once, whatever the
grid: the blocks take the tiles of an XCD's share in groups of 32, rotated
against each other, and a group past the share's end in order.

Tile counts (64 x 16 nodes) of 8, 31, 32, 33, 63, 64 and 65 a share, shares that
are no whole number of tiles, and more tiles than blocks (2048 x 2048).  Bound:
the operator's 25 coefficients sum to 52 in magnitude, and a value passes
through fewer than 64 roundings.
"""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1704_08897_amd import bhx  # noqa: E402


@pytest.fixture(scope="module")
def handle():
    with bhx.Handle(0) as h:
        yield h


@pytest.mark.parametrize("nx,ny,bx,by", [
    (64, 1024, 0, 0), (256, 992, 1, 0), (256, 1024, 2, 1), (256, 1056, 0, 0), (1008, 504, 1, 1),
    (1024, 512, 0, 2), (1040, 488, 2, 0), (900, 333, 1, 2), (1023, 777, 2, 2), (2048, 2048, 0, 1)])
def test_operator_at_tile_group_edges(handle, nx, ny, bx, by):
    rng = np.random.default_rng(nx + 3 * ny)
    phi = -(rng.random((ny, nx)) - 0.7)
    x = rng.normal(size=(ny, nx))
    known = O.known_mask(phi)
    ref = np.where(known, 0.0, O.stencil_padded(np.where(known, 0.0, x), bx, by))
    dphi, dx = (torch.from_numpy(a).to("cuda:0") for a in (phi, x))
    out = torch.full_like(dx, 7.0)
    assert bhx.debug_apply(handle, 0, dphi, dx, out, bc=bhx.BC(bx, by)) == bhx.OK
    got = out.cpu().numpy()
    assert not got[known].any()
    assert np.abs(got - ref).max() <= 64 * np.finfo(float).eps * np.abs(x).max() * 52
