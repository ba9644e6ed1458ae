"""Tiled sweeps: forced on sizes at the edges of the pieces (one piece, a last piece of one index, sizes that fill the
pieces, both column splits of the gradient's stages), with odd sizes, restricted parametrisations and batches around the
kernels' blocks of 32 columns, against the float64 entry points."""
import numpy as np
import pytest

from paper_2106_00003_amd import binding, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# the float32 sweeps that the tiles stand in for are allowed 1e-5 and 1e-4; their own rounding is below 1e-6 at these sizes
TOL_Y, TOL_G = 2e-6, 4e-6


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    yield
    binding.set_kernel(binding.KERNEL_AUTO)
    binding.release()


def far(got, want):
    return float((got - want).norm() / want.norm())


def check(n, m, B, seed):
    print(f"[tiles] n={n} m={m} B={B}", flush=True)
    data = inputs.make_restricted(n, m, B, seed=seed)
    th, x, g = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X", "G"))
    want_y = binding.givens_forward_restricted(th.double(), x.double(), m)
    want_dx, want_dth = binding.givens_backward_restricted(th.double(), want_y, g.double(), m)
    try:
        binding.set_kernel(binding.KERNEL_TILES)
        y = binding.givens_forward_restricted(th, x, m)
        assert binding.last_kernel() == binding.KERNEL_TILES
        dx, dth = binding.givens_backward_restricted(th, y, g, m)
        assert binding.last_reduction() == binding.REDUCTION_GRAM
        assert far(y, want_y) <= TOL_Y and far(dx, want_dx) <= TOL_G and far(dth, want_dth) <= TOL_G
        again = binding.givens_backward_restricted(th, y, g, m, want_dx=False)[1]
        assert torch.equal(again, dth)
        buf = x.clone()
        assert torch.equal(binding.givens_forward_restricted(th, buf, m, Y=buf), y)
        buf = g.clone()
        binding.givens_backward_restricted(th, y, buf, m, dX=buf)
        assert torch.equal(buf, dx)
        if n % 2 == 0 and m == n - 1:
            back = binding.givens_forward_transposed(th, y)
            assert far(back, x.double()) <= 2 * TOL_Y
            u = binding.givens_build(th, n)
            assert far(u @ x, want_y) <= 2 * TOL_Y
    finally:
        binding.set_kernel(binding.KERNEL_AUTO)


@pytest.mark.parametrize("n,B", [(8, 1), (10, 40), (126, 33), (128, 31), (130, 64), (252, 65), (254, 7), (256, 500),
                                 (382, 3), (504, 129), (1006, 20), (258, 3000)])
def test_every_pair_free(n, B):
    check(n, n - 1, B, 3000 + n)


@pytest.mark.parametrize("n,m,B", [(9, 3, 5), (127, 126, 33), (129, 1, 40), (257, 20, 64), (300, 50, 40), (301, 299, 70),
                                   (515, 100, 1300), (640, 3, 2100)])
def test_restricted_and_odd_sizes(n, m, B):
    check(n, m, B, 3100 + n)


# stages that launch the tiles with a free pair only, in both calls, in the forward call and in the gradient (tile_choice.hpp)
@pytest.mark.parametrize("n,m,B", [(2901, 60, 300), (1001, 60, 1000), (2050, 41, 1000), (2901, 300, 40)])
def test_restricted_stages_that_leave_tiles_out(n, m, B):
    check(n, m, B, 3150)


def test_more_pieces_than_the_narrow_stages_take():
    check(3100, 3099, 48, 3200)


@pytest.mark.parametrize("scale", [1.0, 1e4, 1e6, 1e20])
def test_large_angles(scale):
    n, B = 200, 50
    gen = torch.Generator(device="cuda").manual_seed(3300)
    th = torch.randn(n * (n - 1) // 2, device="cuda", generator=gen) * scale
    x = torch.randn(n, B, device="cuda", generator=gen)
    want = binding.givens_forward(th.double(), x.double())
    try:
        binding.set_kernel(binding.KERNEL_TILES)
        assert far(binding.givens_forward(th, x), want) <= TOL_Y
    finally:
        binding.set_kernel(binding.KERNEL_AUTO)


# upstream gradients with infinities and NaN: dX of the other columns does not change, in stages of both kinds, with the operand swept
# and with the product
@pytest.mark.parametrize("n,B", [(258, 70), (258, 600), (1006, 90), (2050, 40)])
def test_infinities_and_nan_in_the_backward_call(n, B):
    print(f"[tiles] infinities n={n} B={B}", flush=True)
    data = inputs.make_custom(n, B, seed=3600 + n)
    th, y, g = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X", "G"))
    bad = g.clone()
    bad[1, 0], bad[n - 1, B // 2], bad[n // 2, B - 1] = float("nan"), float("inf"), -float("inf")
    clean = torch.ones(B, dtype=torch.bool, device="cuda")
    clean[[0, B // 2, B - 1]] = False
    try:
        binding.set_kernel(binding.KERNEL_TILES)
        want, _ = binding.givens_backward(th, y, g)
        dx, dth = binding.givens_backward(th, y, bad)
        again, plain = binding.givens_backward(th, y, g)
    finally:
        binding.set_kernel(binding.KERNEL_AUTO)
    assert torch.equal(dx[:, clean], want[:, clean]) and not torch.isfinite(dx[:, ~clean]).all(dim=0).any()
    assert not torch.isfinite(dth).all() and torch.equal(again, want) and torch.isfinite(plain).all()


# ... with restricted parametrisations, where most pairs of tiles have one that does not rotate: an angle's gradient is finite only where
# the float64 sweep's is
@pytest.mark.parametrize("n,m,B", [(401, 60, 90), (700, 90, 40), (1001, 200, 2100), (2901, 100, 33)])
def test_infinities_and_nan_in_restricted_backward_calls(n, m, B):
    print(f"[tiles] infinities n={n} m={m} B={B}", flush=True)
    data = inputs.make_restricted(n, m, B, seed=3650 + n)
    th, y, g = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X", "G"))
    for row, value in ((1, float("nan")), (n - 1, float("inf")), (n // 2, -float("inf"))):
        bad = g.clone()
        bad[row, B // 2] = value
        clean = torch.ones(B, dtype=torch.bool, device="cuda")
        clean[B // 2] = False
        try:
            binding.set_kernel(binding.KERNEL_TILES)
            want, plain = binding.givens_backward_restricted(th, y, g, m)
            dx, dth = binding.givens_backward_restricted(th, y, bad, m)
            again, plain_again = binding.givens_backward_restricted(th, y, g, m)
        finally:
            binding.set_kernel(binding.KERNEL_AUTO)
        wide = binding.givens_backward_restricted(th.double(), y.double(), bad.double(), m)[1]
        assert torch.equal(dx[:, clean], want[:, clean]) and not torch.isfinite(dx[:, B // 2]).all()
        assert not (torch.isfinite(dth) & ~torch.isfinite(wide)).any() and not torch.isfinite(dth).all()
        assert torch.equal(again, want) and torch.equal(plain_again, plain) and torch.isfinite(plain).all()


def test_calls_that_tiles_do_not_take():
    th = torch.zeros(15, device="cuda")
    try:
        binding.set_kernel(binding.KERNEL_TILES)
        for call in (lambda: binding.givens_forward(th, torch.zeros(6, 3, device="cuda")),
                     lambda: binding.givens_forward(th.double(), torch.zeros(6, 3, device="cuda").double()),
                     lambda: binding.givens_prepare(th, 6)):
            with pytest.raises(binding.GivensError) as err:
                call()
            assert err.value.code == -5
    finally:
        binding.set_kernel(binding.KERNEL_AUTO)


@pytest.fixture
def library_defaults():
    """Sizes take the tiles by themselves where no rotation form is chosen."""
    binding.set_rotation_form(binding.FORM_AUTO)
    yield
    binding.set_rotation_form(binding.FORM_RANGE)


# a size of every kind that the rule tells apart, on both sides of its batch: whether the forward and the backward call run
# as tiles, and whether each multiplies
@pytest.mark.parametrize("n,B,forward,backward,product", [
    (398, 500, False, False, False), (402, 1, False, False, False), (514, 400, True, False, False),
    (514, 500, True, True, False), (514, 2048, True, True, True), (706, 20, True, True, False),
    (1002, 300, True, False, False), (1002, 700, True, True, False), (1006, 40, True, True, False),
    (1024, 900, False, False, False), (1024, 1000, False, True, False), (1024, 2100, False, True, True),
    (1280, 1280, False, False, False), (1022, 700, False, True, False), (2050, 64, True, False, False),
    (898, 898, True, True, False), (896, 896, False, False, False), (2048, 1950, False, False, False)])
def test_sizes_around_the_rule(library_defaults, n, B, forward, backward, product):
    sizes_around_the_rule(n, B, forward, backward, product)


# sizes with a carousel shape, none of one wavefront: both sides of the batch and of 1e9 updates; 3, 5 and 7 slots
@pytest.mark.parametrize("n,B,forward,backward,product", [
    (696, 696, False, False, False), (780, 3, True, False, False), (780, 702, True, True, False), (770, 230, False, False, False),
    (770, 231, False, True, False), (690, 690, False, False, False), (904, 150, True, False, False), (904, 151, True, True, False),
    (904, 2048, True, True, True), (1002, 301, True, True, False), (1280, 213, True, False, False), (1280, 214, True, True, False),
    (1280, 1221, True, True, False), (1280, 1222, False, False, False), (2048, 342, True, True, False), (4096, 119, True, False, False)])
def test_sizes_without_a_shape_of_one_wavefront(library_defaults, n, B, forward, backward, product):
    sizes_around_the_rule(n, B, forward, backward, product)


# two and three slots, whose backward sweeps are the fastest: both sides of each line
@pytest.mark.parametrize("n,B,forward,backward,product", [
    (900, 271, True, False, False), (900, 359, True, False, False), (900, 360, True, True, False), (956, 382, True, False, False),
    (964, 289, True, False, False), (964, 290, True, True, False), (1060, 264, True, False, False), (1060, 265, True, True, False),
    (1196, 298, True, False, False), (1204, 201, True, True, False), (702, 526, True, False, False), (702, 527, True, True, False),
    (894, 268, True, False, False), (894, 671, True, True, False), (942, 376, True, False, False), (942, 377, True, True, False),
    (966, 290, False, True, False), (978, 293, True, False, False), (978, 294, True, True, False)])
def test_sizes_of_two_and_three_slots(library_defaults, n, B, forward, backward, product):
    sizes_around_the_rule(n, B, forward, backward, product)


def sizes_around_the_rule(n, B, forward, backward, product):
    data = inputs.make_custom(n, B, seed=3500 + n)
    th, x, g = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X", "G"))
    y = binding.givens_forward(th, x)
    assert (binding.last_kernel() == binding.KERNEL_TILES) == forward and binding.last_product() == product
    dx, dth = binding.givens_backward(th, y, g)
    assert (binding.last_kernel() == binding.KERNEL_TILES) == backward and binding.last_product() == product
    assert binding.last_reduction() == (binding.REDUCTION_GRAM if backward or B >= 2 * n else binding.REDUCTION_TWO_STAGE)
    want_y = binding.givens_forward(th.double(), x.double())
    assert binding.last_kernel() != binding.KERNEL_TILES and not binding.last_product()
    want_dx, want_dth = binding.givens_backward(th.double(), want_y, g.double())
    assert far(y, want_y) <= 1e-5 and far(dx, want_dx) <= 1e-4 and far(dth, want_dth) <= 1e-4


def test_routes_and_graph_replay(library_defaults):
    """A size that takes the tiles by itself, plain and through autograd, and recorded into a graph."""
    from paper_2106_00003_amd import layer
    n, B = 1006, 1100
    data = inputs.make_custom(n, B, seed=3400)
    th, x, g = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X", "G"))
    assert not binding.givens_prepare_pays(n, None, B) and binding.givens_prepare_pays(256, None, B)
    y, dx, dth = torch.empty_like(x), torch.empty_like(x), torch.empty_like(th)

    def run():
        binding.givens_forward(th, x, Y=y)
        binding.givens_backward(th, y, g, dX=dx, dtheta=dth)

    run()
    want = [t.clone() for t in (y, dx, dth)]
    thg, xg = th.clone().requires_grad_(True), x.clone().requires_grad_(True)
    out = layer.givens_apply(thg, xg)
    out.backward(g)
    assert torch.equal(out.detach(), want[0]) and torch.equal(xg.grad, want[1]) and torch.equal(thg.grad, want[2])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        run()
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            run()
    for _ in range(3):
        for t in (y, dx, dth):
            t.fill_(float("nan"))
        filler = (x @ x.T).sum()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.isfinite(filler) and all(torch.equal(a, b) for a, b in zip((y, dx, dth), want))
