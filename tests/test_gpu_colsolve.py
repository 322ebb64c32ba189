"""The recursive column solve of the preconditioner, at the edges of its lane
segments, against the oracle's spectral form.

A lane holds 1, 2, 4, ... rows of a column (64 lanes a column, or 16 in the
wide items), so lengths around powers of two change the segment length and
whether the last segment is short.  Rounding the recursions' pole rho = 1 - d
changes the lowest mode's gain d^-4 by 4 eps / (2 d) at most, d >= pi / 2048:
3e-13; the bound leaves ten times that for the sums and the x transform.
"""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)
import oracle as O  # noqa: E402

try:
    import torch
    HAS_GPU = torch.cuda.is_available()
except Exception:
    HAS_GPU = False
pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not HAS_GPU, reason="needs a GPU")]
if HAS_GPU:
    from paper_1704_08897_amd import bhx

BOUND = {0: 3e-12, 1: 2e-4}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.fixture(scope="module")
def handle():
    with bhx.Handle(0) as h:
        yield h


def check(handle, shape, rules, prec, known_share):
    rng = np.random.default_rng(sum(shape) + 10 * sum(rules))
    phi = -(rng.random(shape) - (1 - known_share))
    r = rng.normal(size=shape)
    known = O.known_mask(phi)
    out = dev(np.zeros(shape))
    if len(shape) == 2:
        ref = O.spectral_preconditioner(r, known, *rules)
        s = bhx.debug_apply(handle, 1, dev(phi), dev(r), out, bc=bhx.BC(*rules), precision=prec)
    else:
        ref = O.spectral_preconditioner_3d(r, known, *rules)
        s = bhx.debug_apply3d(handle, 1, dev(phi), dev(r), out, bc=bhx.BC3(*rules),
                              precision=prec)
    assert s == bhx.OK
    assert O.relative_l2(out.cpu().numpy(), ref) <= BOUND[prec]


@pytest.mark.parametrize("ny", [4, 5, 63, 64, 65, 127, 129, 255, 257, 512, 513, 1000, 1025, 2047])
@pytest.mark.parametrize("nx,bx", [(4, 0), (37, 1), (64, 2), (2048, 0)])
def test_columns_2d(handle, nx, bx, ny):
    for by in (0, 1, 2):
        check(handle, (ny, nx), (bx, by), 0, 0.3)


@pytest.mark.parametrize("ny", [2048, 2049, 3000, 4093])
def test_long_columns_fp32(handle, ny):
    for by in (0, 1):
        check(handle, (ny, 24), (0, by), 1, 0.3)


@pytest.mark.parametrize("nz", [4, 15, 16, 17, 33, 127, 128, 257, 512])
def test_columns_3d_wide(handle, nz):
    """At least 4096 columns: the 16-lane items."""
    for rules in ((0, 1, 0), (1, 1, 1), (0, 0, 2), (2, 1, 1)):
        check(handle, (nz, 64, 65), rules, 0, 0.5)


@pytest.mark.parametrize("shape,rules", [((4095, 24), (0, 2)), ((4095, 24), (1, 2)),
                                         ((4095, 24), (2, 2)), ((24, 4095), (2, 0)),
                                         ((4095, 5, 6), (0, 1, 2)), ((4095, 5, 6), (2, 2, 2)),
                                         ((4, 4095, 6), (1, 2, 0)), ((6, 4, 4095), (2, 0, 1))])
def test_longest_dirichlet_axis_fp32(handle, shape, rules):
    """4095 nodes, the one FP32 Dirichlet length above 2047 (an odd extension of
    8192 points): as the last axis, whose lanes hold 64 rows, and as the others."""
    check(handle, shape, rules, 1, 0.3)
