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


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("ny", [4, 15, 16, 17, 31, 33, 63, 65, 127, 128, 129, 255, 257, 511, 512])
def test_columns_2d_wide(handle, ny, prec):
    """The 32-column items of shared launches (rows = -1) at the edges of their
    16-lane segments.  The first iterate of the solve is a multiple of the
    preconditioned right-hand side: compared by direction, at most twice the
    operator's bound apart.  37 and 64 columns: a partly and a fully used item."""
    for nx, bx in ((37, 1), (64, 0), (65, 2)):
        for by in (0, 1, 2):
            rng = np.random.default_rng(ny + 10 * nx + by)
            phi = -(rng.random((ny, nx)) - 0.7)
            F = rng.normal(size=(ny, nx))
            known = O.known_mask(phi)
            b = np.zeros((ny, nx))
            b[~known] = O.rhs(F, known, bx, by)
            z = O.spectral_preconditioner(b, known, bx, by)[~known]
            G = dev(F)
            s, st = bhx.extend_ex(handle, dev(phi), G, bc=bhx.BC(bx, by), tol=1e-14,
                                  opts=bhx.default_opts(maxit=1, rows=-1, precision=prec))
            assert s == bhx.NOT_CONVERGED and st.iterations == 1
            x = G.cpu().numpy()[~known]
            d = x / np.linalg.norm(x) - z / np.linalg.norm(z)
            assert np.linalg.norm(d) <= 2 * BOUND[prec], (nx, bx, by)


@pytest.mark.parametrize("nz", [4, 17, 128, 129, 512])
def test_columns_3d_wide_fp32(handle, nz):
    for rules in ((0, 1, 0), (1, 1, 1), (0, 0, 2), (2, 1, 1)):
        check(handle, (nz, 64, 65), rules, 1, 0.5)


@pytest.mark.parametrize("prec,by", [(0, 0), (0, 1), (0, 2), (1, 0), (1, 1), (1, 2)])
@pytest.mark.parametrize("rows", [0, -1])
def test_batch_across_column_classes(handle, rows, prec, by, monkeypatch):
    """An instance alone and in a batch whose longest column takes the launch to
    another kernel class (edges at 512 nodes of 8-column items, 128 of 32-column
    ones, 2048 in FP32): the same bits."""
    monkeypatch.setenv("BHX_SHAPE_KERNELS", "0")
    sides = [(45, 60), (75, 128), (90, 129), (50, 512), (41, 513), (33, 1300)]
    if prec == 1:
        sides.append((20, 4095 if by == 2 else 3000))
    ins = []
    for nx, ny in sides:
        y, x = np.meshgrid(np.linspace(-1, 1, ny), np.linspace(-1, 1, nx), indexing="ij")
        ins.append((dev(np.hypot(x, y) - 0.5), dev(np.cos(2 * x) + np.sin(y))))
    o = bhx.default_opts(maxit=24, rows=rows, precision=prec)
    bc = bhx.BC(0, by)
    alone = []
    for phi, F in ins:
        G = F.clone()
        s, _ = bhx.extend_ex(handle, phi, G, h=0.01, bc=bc, tol=1e-14, opts=o)
        assert s == bhx.NOT_CONVERGED
        alone.append(G)
    outs = [F.clone() for _, F in ins]
    k = len(ins)
    s, _ = bhx.extend_batched(handle, [p for p, _ in ins], outs, [0.01] * k, [bc] * k,
                              [1e-14] * k, opts=o)
    assert s == bhx.NOT_CONVERGED
    for a, b in zip(alone, outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("sides", [[(20, 4095)], [(20, 4095), (45, 60)], [(45, 60), (33, 1300)]])
def test_profiled_launches_across_column_classes(handle, sides):
    """The column pass of a 4095-node FP32 Dirichlet axis is a launch beside the
    other columns': the profile counts and times the two as one pass."""
    ins = [(dev(np.hypot(*np.meshgrid(np.linspace(-1, 1, ny), np.linspace(-1, 1, nx),
                                      indexing="ij")) - 0.5), dev(np.ones((ny, nx))))
           for nx, ny in sides]
    k = len(ins)
    o = bhx.default_opts(maxit=8, chunk=8, precision=1, profile=4)
    s, sts = bhx.extend_batched(handle, [p for p, _ in ins], [F for _, F in ins], [0.01] * k,
                                [bhx.BC(0, 2)] * k, [1e-14] * k, opts=o)
    assert s == bhx.NOT_CONVERGED
    assert sts[0].pass_launches[2] == 8 and sts[0].pass_ms[2] > 0
    assert all(st.iterations == 8 for st in sts)
