"""The dense products behind wide batches (float32 operands cut into bf16 pieces on the matrix cores): the contraction
C = Y G^T at the edges of its tiles, steps and slices.  Compared with the float64 entry points, which are held to 1e-12
against the oracle elsewhere and run the sweep itself whatever the batch."""
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
    binding.release()


def rel(got, want):
    return float((got.double() - want).norm() / want.norm())


# 64 x 64 tiles: one row more and less than a tile, one column more and less than a step, a last slice that is short;
# 256 x 128 tiles: full ones, ragged ones, an unaligned row length
@pytest.mark.parametrize("n,B", [(2, 4), (62, 257), (64, 8192), (66, 4097), (130, 2049), (192, 6000), (1024, 16384),
                                 (1030, 16385), (1152, 7999)])
def test_gram_contraction_at_the_edges_of_its_tiles(n, B):
    data = inputs.make_custom(n, B, seed=1300 + n)
    print(f"[products] gram n={n} B={B}", flush=True)
    th, y, g = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X", "G"))
    dx, dth = binding.givens_backward_ex(th, y, g, reduction=binding.REDUCTION_GRAM)
    assert binding.last_reduction() == binding.REDUCTION_GRAM
    want_dx, want_dth = binding.givens_backward(th.double(), y.double(), g.double())
    assert rel(dx, want_dx) <= TOL_G and rel(dth, want_dth) <= TOL_G
    again = binding.givens_backward_ex(th, y, g, reduction=binding.REDUCTION_GRAM)[1]
    assert torch.equal(again, dth)


# the tiles between: contractions of 128 x 128, products of 64 x 64, 128 x 64 and 128 x 128 with loads two steps ahead, odd and
# even numbers of steps, ragged in both directions
@pytest.mark.parametrize("n,B", [(288, 12001), (386, 9001), (768, 5000), (770, 5001), (800, 4999), (1002, 3001),
                                 (1056, 4501)])
def test_tiles_of_middle_sizes(n, B):
    data = inputs.make_custom(n, B, seed=1330 + n)
    print(f"[products] middle n={n} B={B}", flush=True)
    th, x, g = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X", "G"))
    want = binding.givens_forward(th.double(), x.double())
    y = binding.givens_forward(th, x)
    assert rel(y, want) <= TOL_Y and rel(y[-3:, -3:], want[-3:, -3:]) <= TOL_Y
    dx, dth = binding.givens_backward_ex(th, y, g, reduction=binding.REDUCTION_GRAM)
    want_dx, want_dth = binding.givens_backward(th.double(), want, g.double())
    assert rel(dx, want_dx) <= TOL_G and rel(dth, want_dth) <= TOL_G


# operands that start at an odd multiple of four bytes, row lengths of every remainder: both tile sizes
@pytest.mark.parametrize("n,B", [(66, 4097), (66, 4098), (514, 4099), (512, 4096)])
def test_gram_contraction_of_unaligned_operands(n, B):
    data = inputs.make_custom(n, B, seed=1350 + n)
    th, y, g = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X", "G"))
    shifted = [torch.empty(n * B + 1, device="cuda")[1:].view(n, B).copy_(t) for t in (y, g)]
    _, want = binding.givens_backward_ex(th, y, g, reduction=binding.REDUCTION_GRAM)
    _, got = binding.givens_backward_ex(th, *shifted, reduction=binding.REDUCTION_GRAM)
    assert torch.equal(got, want)
    _, want = binding.givens_backward(th.double(), y.double(), g.double())
    assert rel(got, want) <= TOL_G


# applications through U: below and above the batch where they begin, one column past a tile, one row past and short of
# the tiles of 64, 128 and 256 rows, both directions, odd sizes, results over their operands, no allocation
@pytest.mark.parametrize("n,B", [(132, 2048), (192, 2049), (254, 2111), (256, 16385), (258, 40001), (302, 2050),
                                 (514, 33000), (1024, 2048), (1026, 12345)])
def test_wide_batches_go_through_u(n, B):
    data = inputs.make_custom(n, B, seed=1400 + n)
    print(f"[products] wide n={n} B={B}", flush=True)
    th, x = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X"))
    want = binding.givens_forward(th.double(), x.double())
    y = binding.givens_forward(th, x)
    assert rel(y, want) <= TOL_Y
    assert rel(y[:, -3:], want[:, -3:]) <= TOL_Y
    back = binding.givens_forward_transposed(th, y)
    assert rel(back, x.double()) <= 3 * TOL_Y
    buf = x.clone()
    binding.givens_forward(th, buf, Y=buf)
    assert torch.equal(buf, y)
    if n <= binding.NOALLOC_MAX_N:
        other = torch.full_like(x, float("nan"))
        assert torch.equal(binding.givens_forward_noalloc(th, x, other), y)
        buf.copy_(x)
        assert torch.equal(binding.givens_forward_noalloc(th, buf, buf), y)
    token = binding.givens_prepare(th, n, directions=binding.PREPARE_FORWARD)
    assert torch.equal(binding.givens_forward_prepared(token, x), y)


def test_wide_restricted_batch_with_an_odd_number_of_rows():
    n, m, B = 257, 40, 4099
    data = inputs.make_restricted(n, m, B, seed=1500)
    th, x, g = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X", "G"))
    y = binding.givens_forward_restricted(th, x, m)
    dx, dth = binding.givens_backward_restricted(th, y, g, m)
    want_y = binding.givens_forward_restricted(th.double(), x.double(), m)
    want_dx, want_dth = binding.givens_backward_restricted(th.double(), want_y, g.double(), m)
    assert rel(y, want_y) <= TOL_Y and rel(dx, want_dx) <= TOL_G and rel(dth, want_dth) <= TOL_G


@pytest.mark.parametrize("scale", [1e-30, 1e30, 3.4e38])
def test_products_keep_the_range_of_float32(scale):
    """Operands near the ends of the exponent range: the leading piece may not overflow, the trailing ones may vanish
    only where float32 itself has no bits left.  A column of U has norm 1, so results are of the operand's size."""
    n, B = 256, 4096
    data = inputs.make_custom(n, B, seed=1600)
    th = torch.from_numpy(data["theta"]).cuda()
    x = torch.zeros(n, B, device="cuda")
    rows = torch.arange(B, device="cuda") % n
    x[rows, torch.arange(B, device="cuda")] = scale
    y = binding.givens_forward(th, x)
    want = binding.givens_forward(th.double(), x.double())
    assert torch.isfinite(y).all() and rel(y, want) <= TOL_Y


# complex operands: below and above the batch from which each direction goes through U, odd batches, sizes of both kernel
# families, results over their operands
@pytest.mark.parametrize("n,B", [(2, 1024), (16, 4097), (30, 4096), (66, 1023), (66, 1024), (128, 1025), (130, 4099),
                                 (256, 4096), (272, 5001)])
def test_wide_unitary_batches(n, B):
    gen = torch.Generator(device="cuda").manual_seed(1700 + n)
    print(f"[products] unitary n={n} B={B}", flush=True)
    th, ph = ((torch.rand(n * (n - 1) // 2, device="cuda", generator=gen) * 2 - 1) * np.pi for _ in range(2))
    x, g = (torch.randn(n, B, dtype=torch.complex64, device="cuda", generator=gen) for _ in range(2))
    y = binding.givens_unitary_forward(th, ph, x)
    dx, dth, dph = binding.givens_unitary_backward(th, ph, y, g)

    def far(got, want):
        return float((got.to(want.dtype) - want).norm() / want.norm())

    want_y = binding.givens_unitary_forward(th.double(), ph.double(), x.to(torch.complex128))
    want = binding.givens_unitary_backward(th.double(), ph.double(), want_y, g.to(torch.complex128))
    assert far(y, want_y) <= TOL_Y
    assert all(far(a, b) <= TOL_G for a, b in zip((dx, dth, dph), want))
    none, dth2, dph2 = binding.givens_unitary_backward(th, ph, y, g, want_dx=False)
    assert none is None and torch.equal(dth2, dth) and torch.equal(dph2, dph)
    buf = x.clone()
    binding.givens_unitary_forward(th, ph, buf, Y=buf)
    assert torch.equal(buf, y)
    buf = g.clone()
    binding.givens_unitary_backward(th, ph, y, buf, dX=buf)
    assert torch.equal(buf, dx)


# the reduction a caller chooses, on both sides of the batch from which AUTO contracts, in both families; float64 has the sweep
@pytest.mark.parametrize("n,B", [(6, 3), (30, 200), (64, 1024), (128, 40), (144, 1024)])
def test_unitary_reductions_that_are_chosen(n, B):
    gen = torch.Generator(device="cuda").manual_seed(1750 + n)
    th, ph = ((torch.rand(n * (n - 1) // 2, device="cuda", generator=gen) * 2 - 1) * np.pi for _ in range(2))
    y, g = (torch.randn(n, B, dtype=torch.complex64, device="cuda", generator=gen) for _ in range(2))
    want = binding.givens_unitary_backward(th.double(), ph.double(), y.to(torch.complex128), g.to(torch.complex128))
    wide = B >= 4 * n and B >= 1024
    gram, sweep = binding.REDUCTION_GRAM, binding.REDUCTION_TWO_STAGE
    try:
        for chosen, runs in ((binding.REDUCTION_AUTO, gram if wide else sweep), (gram, gram), (sweep, sweep)):
            binding.set_reduction(chosen)
            got = binding.givens_unitary_backward(th, ph, y, g)
            assert binding.last_reduction() == runs and binding.last_product() == (runs == gram)
            for a, b in zip(got, want):
                assert float((a.to(b.dtype) - b).norm() / b.norm()) <= TOL_G
            binding.givens_unitary_backward(th.double(), ph.double(), y.to(torch.complex128), g.to(torch.complex128))
            assert binding.last_reduction() == sweep
    finally:
        binding.set_reduction(binding.REDUCTION_AUTO)


# the kernel for few columns: one column, one past its 32, contractions that do not fill its eight parts, the last size
# before the tiled kernels and the first after it
@pytest.mark.parametrize("n,B", [(1, 1), (2, 33), (31, 5), (33, 64), (130, 31), (257, 1), (514, 100), (1002, 64),
                                 (1024, 1536), (1024, 1537), (520, 4000)])
def test_packed_matrix_applied_to_few_columns(n, B):
    gen = torch.Generator(device="cuda").manual_seed(1800 + n)
    u, x = torch.randn(n, n, device="cuda", generator=gen), torch.randn(n, B, device="cuda", generator=gen)
    packed = binding.givens_pack(u)
    want = (u.double().cpu() @ x.double().cpu()).cuda()
    got = binding.givens_apply_packed(packed, x)
    # float32 operands and sums of n products: a few units in the last place
    assert rel(got, want) <= 1e-6
    with pytest.raises(binding.GivensError):
        binding.givens_apply_packed(packed, x, Y=x)


def test_packed_matrices_of_another_size_are_refused():
    x = torch.randn(1000, 40, device="cuda")
    u = torch.randn(1002, 1002, device="cuda")
    packed = binding.givens_pack(u)
    for matrix in (packed, packed.clone(), packed[:binding.lib().givens_packed_bytes(1000)].clone()[:-16]):
        with pytest.raises(ValueError):
            binding.givens_apply_packed(matrix, x)
    # a longer buffer, and views and copies of the right size, do
    longer = torch.empty(packed.numel() + 4096, dtype=torch.uint8, device="cuda")
    same = binding.givens_pack(u, packed=longer)
    y = torch.randn(1002, 40, device="cuda")
    want = binding.givens_apply_packed(packed, y)
    for matrix in (same, longer, longer[:packed.numel()], packed.clone()):
        assert torch.equal(binding.givens_apply_packed(matrix, y), want)
    with pytest.raises(ValueError):
        binding.givens_apply_packed(longer[8: 8 + packed.numel()], y)
    assert len({binding.lib().givens_packed_bytes(n) for n in range(1, 1200)}) == 1199


def test_layers_in_evaluation_keep_their_own_matrix():
    from paper_2106_00003_amd import layer
    nets = [layer.OrthogonalLinear(n, m) for n, m in ((130, None), (130, None), (129, 20))]
    xs = [torch.randn(net.n, 40, device="cuda") for net in nets]

    def check():
        with torch.no_grad():
            for net, x in zip(nets, xs):
                want = layer.givens_apply(net.theta.double(), x.double(), net.m)
                assert rel(net(x), want) <= TOL_Y

    check()
    check()
    with torch.no_grad():
        nets[1].theta.mul_(0.5)
    check()
    # a recorded evaluation reads the matrix of its time, also after the layer has gone on
    net, x = nets[0], xs[0]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.no_grad(), torch.cuda.stream(side):
        want = net(x).clone()
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            out = net(x)
    with torch.no_grad():
        net.theta.add_(0.1)
        net(x)
    for _ in range(3):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
