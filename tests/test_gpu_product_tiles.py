"""GPU parity of the throughput product kernel on operands that drive its per-tile and
per-step decisions, bitwise against the CPU oracle.

The few-wavefront kernel takes every grid of up to 2048 blocks of 16 x 16 outputs at some
format, number of components and kind of operands, so small products do not reach the
throughput kernel.  Here a small product's rows and columns repeat until the grid has more
blocks than that.  An output depends on its row and its column alone: the oracle computes
the small product once, and every repetition is compared with it."""
import numpy as np
import pytest

from paper_2207_08867_amd import inputs
from test_gpu_elementwise import assert_bits, to_dev, to_host
from test_gpu_matmul_f16_paths import blocky, cancelling, spread, straddle
from test_gpu_overflow import operands as overflowing
from test_gpu_seq import FORMATS, KINDS, operand

pytestmark = pytest.mark.gpu

EDGE = 741  # 47^2 = 2209 blocks, a last one of five rows or columns


@pytest.fixture(scope="module")
def mcf():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2207_08867_amd as m

    m.lib()
    return m


def repeated(x, axis):
    return np.ascontiguousarray(np.take(x, np.arange(EDGE) % x.shape[axis], axis=axis))


def check_repeated(got, want, what):
    assert_bits(got, repeated(repeated(want, -2), -1), what)


def products(mcf, orc, A, B, nc, kinds, what):
    A, B = A if kinds[0] else A[:1], B if kinds[1] else B[:1]
    got = to_host(mcf.mc_matmul(to_dev(repeated(A, 1)), to_dev(repeated(B, 2)), nc=nc, a_mc=kinds[0], b_mc=kinds[1]))
    check_repeated(got, orc.matmul(A, B, nc=nc, a_mc=kinds[0], b_mc=kinds[1]), f"{what} nc={nc} {kinds}")


@pytest.mark.parametrize("nc", [2, 3, 4])
@pytest.mark.parametrize("kinds", KINDS)
@pytest.mark.parametrize("what", ["spread", "straddle", "cancelling", "blocky"])
def test_f16_decisions(mcf, orc, nc, kinds, what):
    """Exact low products in some tiles only, accumulators on both sides of the last term's
    limit, zero terms before non-zero ones, steps that cancel, unordered components."""
    g = np.random.default_rng(1100 + nc)
    if what == "spread":
        A, B = spread(g, (70, 300), nc, 0), spread(g, (300, 45), nc, 1)
    elif what == "straddle":
        A, B = straddle(g, (48, 200), nc), straddle(g, (200, 33), nc)
    elif what == "cancelling":
        A, B = cancelling(g, 40, 36, 65, nc)
    else:
        A, B = blocky(g, (64, 256), nc, (-3, 1), (-3, 1)), blocky(g, (256, 48), nc, (-3, 1), (-3, 1))
    products(mcf, orc, A, B, nc, kinds, what)


@pytest.mark.parametrize("dt", FORMATS)
@pytest.mark.parametrize("nc", [2, 3, 4])
@pytest.mark.parametrize("kinds", KINDS)
def test_holes(mcf, orc, dt, nc, kinds):
    """Zero values, components, rows and columns, powers of two (the terms' general form)."""
    g = np.random.default_rng(1120 + nc)
    for K in (19, 64):
        products(mcf, orc, operand(g, (61, K), nc, dt, True), operand(g, (K, 53), nc, dt, True), nc, kinds, f"{dt} K={K}")


@pytest.mark.parametrize("dt", [np.float16, np.float32])
@pytest.mark.parametrize("nc", [2, 3])
@pytest.mark.parametrize("kinds", KINDS)
@pytest.mark.parametrize("K,kpos", [(1, 0), (37, 0), (37, 18), (37, 36)])
def test_overflow(mcf, orc, dt, nc, kinds, K, kpos):
    """An infinite leading component with NaNs behind it from the first, a middle or the last step."""
    A, B = overflowing(dt, nc, K, kpos)
    products(mcf, orc, A, B, nc, kinds, f"{dt} K={K} at {kpos}")


@pytest.mark.parametrize("dt", FORMATS)
@pytest.mark.parametrize("nc", [2, 3, 4])
def test_linear(mcf, orc, dt, nc):
    """MC-Linear with and without a bias, dense and with holes."""
    g = np.random.default_rng(1140 + nc)
    for holes in (False, True):
        x, W = operand(g, (61, 77), 1, dt, holes)[0], operand(g, (53, 77), nc, dt, holes)
        for b in (None, operand(g, (1, 53), nc, dt, False)[:, 0]):
            got = to_host(mcf.mc_linear_fwd(to_dev(repeated(x, 0)), to_dev(repeated(W, 1)),
                                            None if b is None else to_dev(repeated(b, 1))))
            check_repeated(got, orc.linear(x, W, b, nc=nc), f"{dt} nc={nc} holes={holes} bias={b is not None}")


@pytest.mark.parametrize("dt", FORMATS)
@pytest.mark.parametrize("nc", [2, 3, 4])
@pytest.mark.parametrize("kinds", KINDS)
def test_addmm(mcf, orc, dt, nc, kinds):
    """alpha A B + beta Y, operands with holes."""
    g = np.random.default_rng(1160 + nc)
    A, B = operand(g, (61, 37), nc if kinds[0] else 1, dt, True), operand(g, (37, 53), nc if kinds[1] else 1, dt, True)
    Y = operand(g, (61, 53), nc, dt, True)
    got = to_host(mcf.mc_addmm(to_dev(repeated(A, 1)), to_dev(repeated(B, 2)), to_dev(repeated(repeated(Y, 1), 2)),
                               nc=nc, alpha=0.5, beta=-1.75, a_mc=kinds[0], b_mc=kinds[1]))
    want = orc.addmm(A, B, Y, 0.5, -1.75, nc=nc, a_mc=kinds[0], b_mc=kinds[1])
    check_repeated(got, want, f"{dt} nc={nc} {kinds}")
