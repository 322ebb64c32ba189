"""Bluestein cores of the 1-D transforms at the edges of their lengths, against
the oracle's scipy transforms.

Sine transforms through the odd extension: a core of 2^L points serves axes of
up to 2^L / 3 nodes (85/86, 170/171, ... change the length; past 1365 nodes the
chirp-z form takes over).  Bounds as in the generic parity tests: 1e-11 in FP64,
2e-4 in FP32.
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

BOUND = {0: 1e-11, 1: 2e-4}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.fixture(scope="module")
def handle():
    with bhx.Handle(0) as h:
        yield h


def check(handle, shape, rules, prec):
    rng = np.random.default_rng(sum(shape) + 10 * sum(rules))
    phi = -(rng.random(shape) - 0.6)
    r = rng.normal(size=shape)
    known = O.known_mask(phi)
    out = dev(np.zeros(shape))
    if len(shape) == 2:
        ref = O.spectral_preconditioner(r, known, *rules)
        # transform 1: the FFT form, whatever the size
        s = bhx.debug_apply(handle, 1, dev(phi), dev(r), out, bc=bhx.BC(*rules),
                            precision=prec | (1 << 4))
    else:
        ref = O.spectral_preconditioner_3d(r, known, *rules)
        s = bhx.debug_apply3d(handle, 1, dev(phi), dev(r), out, bc=bhx.BC3(*rules),
                              precision=prec)
    assert s == bhx.OK
    assert O.relative_l2(out.cpu().numpy(), ref) <= BOUND[prec]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [5, 21, 22, 42, 43, 85, 86, 170, 171, 341, 342, 682, 683, 1365,
                               1366])
def test_sine_core_lengths(handle, n, prec):
    for ny in (7, 40):
        check(handle, (ny, n), (2, 0), prec)


@pytest.mark.parametrize("n", [21, 22, 85, 86, 341, 342, 1023])
def test_sine_core_lengths_3d(handle, n):
    """Along y of three dimensions, both sides of an edge."""
    check(handle, (5, n, 9), (0, 2, 1), 0)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [33, 63, 65, 100, 127, 129, 255, 257, 300, 511, 513, 1000, 1023,
                               1025, 1231, 2047])
def test_core_lengths(handle, n, prec):
    """Both ends of every core length, Neumann and periodic rows; few and many
    lines (short and long work items)."""
    for ny, rules in ((5, (0, 1)), (40, (1, 0)), (130, (0, 0))):
        check(handle, (ny, n), rules, prec)


@pytest.mark.parametrize("rules", [(0, 0), (1, 1), (2, 2)])
def test_batch_gives_the_single_solves_bits(handle, rules):
    """Schedules of 4, 8 and 16 points: an instance alone and beside a longer
    one, which takes the launch to another kernel family."""
    sizes = [(75, 70), (150, 90), (300, 180), (700, 100)]
    ins = []
    for nx, ny in sizes:
        y, x = np.meshgrid(np.linspace(-1, 1, ny), np.linspace(-1, 1, nx), indexing="ij")
        ins.append((dev(np.hypot(x, y) - 0.5), dev(np.cos(2 * x) + np.sin(y))))
    alone = []
    for phi, F in ins:
        G = F.clone()
        s, _ = bhx.extend_ex(handle, phi, G, h=0.01, bc=bhx.BC(*rules), tol=1e-10)
        assert s == bhx.OK
        alone.append(G)
    outs = [F.clone() for _, F in ins]
    k = len(ins)
    s, _ = bhx.extend_batched(handle, [p for p, _ in ins], outs, [0.01] * k,
                              [bhx.BC(*rules)] * k, [1e-10] * k)
    assert s == bhx.OK
    for a, b in zip(alone, outs):
        assert torch.equal(a, b)
