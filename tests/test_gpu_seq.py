"""GPU parity of the few-wavefront sequential product (and of mm_kernel just above the grid
sizes it takes) against the oracle, bitwise: block shapes of 8, 16 and 32 columns with edges on
both sides, reduction lengths around its LDS tile (128 bytes of steps), its test group and its
16-byte loads, aligned and unaligned rows, every operand kind and component count, and
operands whose zeros send wavefronts through its stricter test and the general step."""
import numpy as np
import pytest

from paper_2207_08867_amd import inputs
from test_gpu_elementwise import assert_bits, to_dev, to_host

pytestmark = pytest.mark.gpu

FORMATS = [np.float16, np.float32, np.float64]
KINDS = [(True, True), (True, False), (False, True)]


@pytest.fixture(scope="module")
def mcf():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2207_08867_amd as m

    m.lib()
    return m


def operand(g, shape, planes, dt, holes):
    """Components of every size; holes: zero low components, zero leading components, zero
    values, powers of two, a zero row and a zero column."""
    x = inputs.expansion(g, shape, planes, np.float64 if dt == np.float64 else dt, 0.3)
    if holes:
        pick = g.random(shape)
        for c in range(1, planes):
            x[c][pick < 0.2 / c] = 0
        x[0][(pick > 0.2) & (pick < 0.25)] = 0
        x[:, (pick > 0.3) & (pick < 0.6)] = 0
        two = (pick > 0.6) & (pick < 0.7)
        x[:, two] = 0
        x[0][two] = 0.25
        x[..., shape[-2] // 2, :] = 0
        x[..., shape[-1] // 3] = 0
    return x.astype(dt)


@pytest.mark.parametrize("dt", FORMATS)
@pytest.mark.parametrize("nc", [1, 2, 3, 4])
@pytest.mark.parametrize("kinds", KINDS)
@pytest.mark.parametrize("holes", [False, True])
def test_products(mcf, orc, dt, nc, kinds, holes):
    g = np.random.default_rng(900 + nc)
    # 8, 16 and 32 columns; K around 16, 32 and 64 steps (binary64, binary32, binary16 tiles)
    for M, N, K in ((33, 50, 16), (9, 32, 17), (40, 24, 31), (16, 17, 32), (64, 64, 33), (5, 70, 63), (70, 5, 64),
                    (37, 40, 65), (1, 96, 130), (31, 1, 3), (2, 2, 1)):
        A = operand(g, (M, K), nc if kinds[0] else 1, dt, holes)
        B = operand(g, (K, N), nc if kinds[1] else 1, dt, holes)
        got = to_host(mcf.mc_matmul(to_dev(A), to_dev(B), nc=nc, a_mc=kinds[0], b_mc=kinds[1]))
        want = orc.matmul(A, B, nc=nc, a_mc=kinds[0], b_mc=kinds[1])
        assert_bits(got, want, f"{dt.__name__} nc={nc} {kinds} holes={holes} {M}x{N}x{K}")


@pytest.mark.parametrize("dt", FORMATS)
@pytest.mark.parametrize("nc", [1, 2, 3])
def test_linear_and_batches(mcf, orc, dt, nc):
    g = np.random.default_rng(920 + nc)
    for T, I, O, holes in ((7, 130, 50, False), (33, 64, 32, True)):
        x = operand(g, (T, I), 1, dt, holes)[0]
        W, b = operand(g, (O, I), nc, dt, holes), operand(g, (1, O), nc, dt, False)[:, 0]
        want = orc.linear(x, W, b, nc=nc)
        assert_bits(to_host(mcf.mc_linear_fwd(to_dev(x), to_dev(W), to_dev(np.ascontiguousarray(b)))), want,
                    f"linear {T}x{I}x{O}")
    # batches: planes and batch strides that are and are not multiples of 16 bytes
    for B, M, N, K in ((3, 9, 10, 33), (2, 16, 8, 64)):
        A = np.stack([operand(g, (M, K), nc, dt, False) for _ in range(B)], 1)
        Y = np.stack([operand(g, (K, N), 1, dt, False) for _ in range(B)], 1)
        assert_bits(to_host(mcf.mc_bmm(to_dev(A), to_dev(Y), nc=nc, b_mc=False)),
                    orc.matmul_batched(A, Y, nc=nc, b_mc=False), f"batched {B}x{M}x{N}x{K}")


@pytest.mark.parametrize("dt", FORMATS)
@pytest.mark.parametrize("nc", [2, 3, 4])
@pytest.mark.parametrize("kinds", KINDS)
def test_ragged_above_the_limit(mcf, orc, dt, nc, kinds):
    """mm_kernel's edge tiles (2210 tiles: more than 8 per CU)."""
    M, N, K = 531, 1037, 19
    g = np.random.default_rng(940 + nc)
    A = operand(g, (M, K), nc if kinds[0] else 1, dt, False)
    B = operand(g, (K, N), nc if kinds[1] else 1, dt, False)
    rows, cols = np.divmod(g.integers(0, M * N, 4000), N)
    rows[:40], cols[40:80] = M - 1, N - 1
    got = to_host(mcf.mc_matmul(to_dev(A), to_dev(B), nc=nc, a_mc=kinds[0], b_mc=kinds[1]))[:, rows, cols]
    assert_bits(got, orc.matmul(A, B, nc=nc, a_mc=kinds[0], b_mc=kinds[1], rows=rows, cols=cols), f"{dt} {nc} {kinds}")


def test_one_component_beyond_one_launch(mcf):
    """2^32 + 2^16 outputs of one component: more lanes than one launch holds along x.  K = 1,
    so every output is the rounded product of two values."""
    import torch

    M, N = 65536, 65537
    g = torch.Generator(device="cuda")
    g.manual_seed(960)
    a = (torch.rand(M, generator=g, device="cuda") + 0.5).half()
    b = (torch.rand(N, generator=g, device="cuda") + 0.5).half()
    out = mcf.mc_matmul(a[None, :, None], b[None, None, :], nc=1)[0]
    for r in range(0, M, 4096):
        assert torch.equal(out[r : r + 4096], a[r : r + 4096, None] * b[None, :]), r


@pytest.mark.parametrize("dt", FORMATS)
@pytest.mark.parametrize("kinds", KINDS)
def test_neighbours_stay_out(mcf, orc, dt, kinds):
    """A 16-byte piece that crosses the end of a row or column reads what is stored next: with
    infinities and NaNs in every second row of A and column of B, the other outputs keep the
    oracle's bits, at rows and columns of every remainder and of fewer elements than a piece."""
    g = np.random.default_rng(970)
    for M, N, K in ((6, 9, 33), (5, 46, 17), (3, 3, 3), (9, 2, 70), (4, 15, 1), (33, 23, 31)):
        A = operand(g, (M, K), 2 if kinds[0] else 1, dt, False)
        B = operand(g, (K, N), 2 if kinds[1] else 1, dt, False)
        A[:, 1::2, :], B[:, :, 1::2] = np.inf, np.nan
        got = to_host(mcf.mc_matmul(to_dev(A), to_dev(B), nc=2, a_mc=kinds[0], b_mc=kinds[1]))[:, ::2, ::2]
        want = orc.matmul(np.ascontiguousarray(A[:, ::2]), np.ascontiguousarray(B[:, :, ::2]), nc=2, a_mc=kinds[0],
                          b_mc=kinds[1])
        assert_bits(np.ascontiguousarray(got), want, f"{dt.__name__} {kinds} {M}x{N}x{K}")


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("nc", [2, 3])
@pytest.mark.parametrize("kinds", KINDS)
@pytest.mark.parametrize("zeros", [1, 2, 5])
def test_zero_terms_by_chance(mcf, orc, dt, nc, kinds, zeros):
    """Dense operands with a zero term in one, two and five groups of steps of one row and one
    column: wavefronts that go back to the first test after one, and stay with the other after two."""
    M, N, K = 37, 41, 130
    g = np.random.default_rng(980 + nc)
    A = operand(g, (M, K), nc if kinds[0] else 1, dt, False)
    B = operand(g, (K, N), nc if kinds[1] else 1, dt, False)
    for i in range(zeros):
        A[:, 5, 19 + 21 * i] = 0
        B[:, 30 + 21 * i, 7] = 0
    got = to_host(mcf.mc_matmul(to_dev(A), to_dev(B), nc=nc, a_mc=kinds[0], b_mc=kinds[1]))
    want = orc.matmul(A, B, nc=nc, a_mc=kinds[0], b_mc=kinds[1])
    assert_bits(got, want, f"{dt.__name__} nc={nc} {kinds} zeros={zeros}")
