"""Precision of the products on the bf16 matrix cores where the cut into pieces is hardest, against the float64 entry
points column by column (a small column beside large ones has to be right too)."""
import numpy as np
import pytest

from paper_2106_00003_amd import binding, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL_Y, TOL_G = 1e-5, 1e-4


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    binding.set_kernel(binding.KERNEL_AUTO)
    yield
    binding.set_kernel(binding.KERNEL_AUTO)
    binding.release()


@pytest.fixture(autouse=True)
def _library_defaults(_forms_by_range):
    binding.set_rotation_form(binding.FORM_AUTO)


def rel(got, want):
    return float((got - want).norm() / want.norm())


def worst_column(got, want):
    """Largest relative error of a column that is not zero; a column that is has to come out as zeros."""
    err, norm = (got.to(want.dtype) - want).norm(dim=0), want.norm(dim=0)
    assert float(got.abs()[:, norm == 0].sum()) == 0.0
    return float((err[norm > 0] / norm[norm > 0]).max())


def operands(n, B, seed):
    data = inputs.make_custom(n, B, seed=seed)
    return (torch.from_numpy(data[k]).cuda() for k in ("theta", "X", "G"))


# operands as small, or as large, as float32 still holds with all its bits: each product and contraction tile, the tiled
# sweeps with both kinds of stages, sweeps
@pytest.mark.parametrize("scale", [1e-37, 1e-36, 1e-33, 2e37])
@pytest.mark.parametrize("n,B", [(34, 4100), (64, 65536), (254, 2111), (258, 40001), (1006, 70), (1006, 1100), (1024, 16400),
                                 (3002, 40), (256, 256)])
def test_operands_near_the_ends_of_the_range(n, B, scale):
    print(f"[precision] n={n} B={B} scale={scale}", flush=True)
    th, x, g = operands(n, B, 4000 + n)
    for xs, gs in ((scale, 1.0), (1.0, scale), (scale, 1.0 / scale)):
        xx, gg = (x.clamp(-4, 4) * xs).contiguous(), (g.clamp(-4, 4) * gs).contiguous()
        y = binding.givens_forward(th, xx)
        want_y = binding.givens_forward(th.double(), xx.double())
        assert worst_column(y, want_y) <= TOL_Y
        dx, dth = binding.givens_backward(th, y, gg)
        want_dx, want_dth = binding.givens_backward(th.double(), y.double(), gg.double())
        assert worst_column(dx, want_dx) <= TOL_G
        if xs * gs < 1e30:                                  # (sums over the batch stay in float32's range)
            assert rel(dth, want_dth) <= TOL_G


# every column of a size of its own, some zero, a few values far below their column
@pytest.mark.parametrize("n,B", [(64, 40000), (258, 40001), (1006, 70), (1024, 64), (1024, 4096)])
def test_columns_of_different_sizes(n, B):
    th, x, _ = operands(n, B, 4100 + n)
    sizes = torch.tensor([1.0, 1e-36, 0.0, 1e30, 1e-20, 1e-37], device="cuda")
    x = x.clamp(-4, 4) * sizes[torch.arange(B, device="cuda") % sizes.numel()]
    x[:: 7] *= 1e-6
    x[0, : 6] = 0.0
    want = binding.givens_forward(th.double(), x.double())
    assert worst_column(binding.givens_forward(th, x), want) <= TOL_Y
    assert worst_column(binding.givens_forward_transposed(th, x), binding.givens_forward_transposed(th.double(), x.double())) <= TOL_Y
    u = binding.givens_build(th, n)
    assert worst_column(binding.givens_apply_packed(binding.givens_pack(u), x), want) <= TOL_Y
    buf = x.clone()
    assert worst_column(binding.givens_forward(th, buf, Y=buf), want) <= TOL_Y


@pytest.mark.parametrize("n,B", [(30, 4096), (256, 4096)])
def test_small_complex_operands(n, B):
    gen = torch.Generator(device="cuda").manual_seed(4200 + n)
    th, ph = ((torch.rand(n * (n - 1) // 2, device="cuda", generator=gen) * 2 - 1) * np.pi for _ in range(2))
    x, g = (torch.randn(n, B, dtype=torch.complex64, device="cuda", generator=gen) for _ in range(2))
    wide = [t.double() for t in (th, ph)]
    for xs, gs in ((1e-36, 1.0), (1.0, 1e-36)):
        xx, gg = x * xs, g * gs
        y = binding.givens_unitary_forward(th, ph, xx)
        assert worst_column(y, binding.givens_unitary_forward(*wide, xx.to(torch.complex128))) <= TOL_Y
        dx, dth, dph = binding.givens_unitary_backward(th, ph, y, gg)
        want = binding.givens_unitary_backward(*wide, y.to(torch.complex128), gg.to(torch.complex128))
        assert worst_column(dx, want[0]) <= TOL_G and rel(dth, want[1]) <= TOL_G and rel(dph, want[2]) <= TOL_G


def patterns(count):
    """Values whose pieces are awkward: every bit pattern near the middle between two bf16 values and near the end of the
    middle piece (where a cut leading piece leaves the largest remainders), and random ones."""
    high = np.array([0x3f80, 0x3f81, 0x3fc0, 0x3ffe, 0x3fff, 0x4000, 0xbf80, 0x2f80], dtype=np.uint32)
    low = np.array([0xff7f, 0x7fff, 0x8000, 0x8001, 0xfeff, 0xff80, 0xffff, 0x7f7f, 0x8080, 0x0001], dtype=np.uint32)
    values = ((high[:, None] << np.uint32(16)) | low[None, :]).ravel()
    random = np.random.default_rng(5).integers(0x3f800000, 0x40000000, size=max(0, count - values.size), dtype=np.uint32)
    return torch.from_numpy(np.concatenate([values, random])[:count].view(np.float32).copy()).cuda()


# One product per result: six piece products, three left out (2^-24 of the product), and the sums: the last one at most
# 2^-23 (the matrix instructions do not round every sum to nearest), those before it on terms 2^-7 of it and smaller.
ONE_PRODUCT = (2.0 ** -24 + 2.0 ** -23) * (1 + 2.0 ** -5)


@pytest.mark.parametrize("B", [200, 20000])
def test_one_product_of_every_pattern(B):
    n = 256
    u, x = patterns(n), patterns(B)
    matrix = torch.diag(u)
    operand = x.repeat(n, 1).contiguous()
    want = u.double()[:, None] * x.double()[None, :]
    got = binding.givens_apply_packed(binding.givens_pack(matrix), operand)
    assert float(((got.double() - want) / want).abs().max()) <= ONE_PRODUCT


# with all angles zero and one column, dtheta of a pair (i, j), i < n/2 <= j, is the product y_i g_j; both tile sizes
@pytest.mark.parametrize("n,B", [(96, 200), (1024, 16384)])
def test_contraction_of_every_pattern(n, B):
    y, g = torch.zeros(n, B, device="cuda"), torch.zeros(n, B, device="cuda")
    y[: n // 2, 5] = patterns(n // 2)
    g[n // 2:, 5] = patterns(n // 2)
    theta = torch.zeros(n * (n - 1) // 2, device="cuda")
    _, dth = binding.givens_backward_ex(theta, y, g, reduction=binding.REDUCTION_GRAM)
    assert binding.last_reduction() == binding.REDUCTION_GRAM
    pairs = torch.from_numpy(binding.rr_schedule(n).reshape(-1, 2).astype(np.int64)).cuda()
    across = (pairs[:, 0] < n // 2) & (pairs[:, 1] >= n // 2)
    want = y[pairs[across, 0], 5].double() * g[pairs[across, 1], 5].double()
    assert float(((dth[across].double() - want) / want).abs().max()) <= ONE_PRODUCT


# Sums over many columns, of one sign and of both: the error of a slice's sum is a walk of six roundings per 16 columns
# of at most 2^-23 each, relative to sums that are 1/sqrt(3) of the last one in the mean square, so 2^-23 sqrt(6 4096 / 16)
# / sqrt(3) / 2 = 1.3e-6 for roundings spread evenly; sums of one sign gather half of that and no drift.
@pytest.mark.parametrize("n,B", [(64, 300000), (1024, 131072), (2048, 65536)])
def test_long_contractions(n, B):
    gen = torch.Generator(device="cuda").manual_seed(4300 + n)
    theta = torch.zeros(n * (n - 1) // 2, device="cuda")
    pairs = torch.from_numpy(binding.rr_schedule(n).reshape(-1, 2).astype(np.int64)).cuda()
    across = (pairs[:, 0] < n // 2) & (pairs[:, 1] >= n // 2)
    i, j = pairs[across, 0], pairs[across, 1] - n // 2
    for draw, most in ((torch.rand, 6e-7), (torch.randn, 1.8e-6)):
        y, g = torch.zeros(n, B, device="cuda"), torch.zeros(n, B, device="cuda")
        y[: n // 2], g[n // 2:] = (draw(n // 2, B, device="cuda", generator=gen) for _ in range(2))
        _, dth = binding.givens_backward_ex(theta, y, g, want_dx=False, reduction=binding.REDUCTION_GRAM)
        c = sum(y[: n // 2, k: k + 8192].double() @ g[n // 2:, k: k + 8192].double().T for k in range(0, B, 8192))
        assert rel(dth[across], c[i, j]) <= most
