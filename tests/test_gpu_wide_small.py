"""Smallest matrices on wide batches: every size of the range, odd ones and restricted parametrisations among them, batches on both
sides of what the product takes narrow and of whole tiles and slices, in place, the transpose, graphs, against float64."""
import pytest

from paper_2106_00003_amd import binding

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.set_kernel(binding.KERNEL_AUTO)
    yield
    binding.release()


def rel(got, want):
    return float((got.double() - want).norm() / want.norm())


def problem(n, m, B, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    th = (torch.rand(binding.num_angles(n, m), device="cuda", generator=gen) * 2 - 1) * 3.1
    return th, *(torch.randn(n, B, device="cuda", generator=gen) for _ in range(2))


def check(n, m, B):
    th, x, g = problem(n, m, B, 11 * n + B)
    want_y = binding.givens_forward_restricted(th.double(), x.double(), m)
    want_dx, want_dth = binding.givens_backward_restricted(th.double(), want_y, g.double(), m)
    y = binding.givens_forward_restricted(th, x, m)
    assert binding.last_kernel() == binding.KERNEL_COLUMN
    dx, dth = binding.givens_backward_restricted(th, y, g, m)
    assert binding.last_kernel() == binding.KERNEL_COLUMN and binding.last_reduction() == binding.REDUCTION_GRAM and binding.last_product()
    assert rel(y, want_y) <= 1e-5 and rel(dx, want_dx) <= 1e-4 and rel(dth, want_dth) <= 1e-4
    buf = x.clone()
    assert torch.equal(binding.givens_forward_restricted(th, buf, m, Y=buf), y)
    buf = g.clone()                                                # in place: the calls of the other sizes
    again_dx, again_dth = binding.givens_backward_restricted(th, y, buf, m, dX=buf)
    assert rel(again_dx, dx.double()) <= 1e-6 and rel(again_dth, dth.double()) <= 2e-6
    assert rel(binding.givens_backward_restricted(th, y, g, m, want_dx=False)[1], dth.double()) <= 2e-6


@pytest.mark.parametrize("n", range(16, 67))
def test_every_size(n):
    check(n, n - 1, 2048 + 37 * n)


@pytest.mark.parametrize("n,m,B", [(64, 63, 2048), (64, 63, 24576), (64, 63, 24577), (62, 61, 24609), (33, 32, 49153), (63, 5, 30000),
                                   (17, 1, 65536), (48, 20, 40001), (64, 30, 65535)])
def test_batches_and_restricted(n, m, B):
    check(n, m, B)


# calls that take the kernels of the other sizes: without allocations, on prepared tables, dX in the place of G, no dX
@pytest.mark.parametrize("n,m,B", [(n, n - 1, B) for n in range(16, 65) for B in (2 * n + 2, 2048 + 11 * n)] +
                         [(64, 20, 700), (63, 5, 4000), (33, 8, 30000), (48, 47, 24577)])
def test_every_way_to_a_result_gives_the_same_bits(n, m, B):
    th, x, g = problem(n, m, B, 7 * n + B)
    y = binding.givens_forward_restricted(th, x, m)
    dx, dth = binding.givens_backward_restricted(th, y, g, m)
    token = binding.givens_prepare(th, n, m, binding.PREPARE_FORWARD | binding.PREPARE_BACKWARD_WIDE, batch=B)
    assert torch.equal(binding.givens_forward_prepared(token, x), y)
    pdx, pdth = binding.givens_backward_prepared(token, y, g, th.numel())
    assert torch.equal(pdx, dx) and torch.equal(pdth, dth)
    buf = g.clone()
    idx, idth = binding.givens_backward_restricted(th, y, buf, m, dX=buf)
    assert torch.equal(idx, dx) and torch.equal(idth, dth)
    assert torch.equal(binding.givens_backward_restricted(th, y, g, m, want_dx=False)[1], dth)
    if n % 2 == 0 and m == n - 1:
        assert torch.equal(binding.givens_forward_noalloc(th, x, torch.empty_like(x)), y)


# infinities and NaN in the upstream gradient, and in an angle: the other columns of dX do not change, and what the float64 sweep
# cannot tell is not finite here
@pytest.mark.parametrize("n,m,B", [(64, 63, 3000), (40, 39, 24600), (33, 32, 130), (16, 15, 5000), (63, 9, 2500)])
def test_infinities_and_nan_in_the_backward_call(n, m, B):
    th, x, g = problem(n, m, B, 13 * n)
    y = binding.givens_forward_restricted(th, x, m)
    want, plain = binding.givens_backward_restricted(th, y, g, m)
    for row, value in ((1, float("nan")), (n - 1, float("inf")), (n // 2, -float("inf"))):
        bad = g.clone()
        bad[row, B // 2] = value
        clean = torch.ones(B, dtype=torch.bool, device="cuda")
        clean[B // 2] = False
        dx, dth = binding.givens_backward_restricted(th, y, bad, m)
        wide = binding.givens_backward_restricted(th.double(), y.double(), bad.double(), m)[1]
        assert torch.equal(dx[:, clean], want[:, clean]) and not torch.isfinite(dx[:, B // 2]).all()
        assert not (torch.isfinite(dth) & ~torch.isfinite(wide)).any() and not torch.isfinite(dth).all()
    for value in (float("nan"), float("inf")):
        bad = th.clone()
        bad[th.numel() // 2] = value
        got = binding.givens_forward_restricted(bad, x, m), *binding.givens_backward_restricted(bad, y, g, m)
        wide = binding.givens_forward_restricted(bad.double(), x.double(), m), *binding.givens_backward_restricted(bad.double(), y.double(), g.double(), m)
        assert all(not (torch.isfinite(a) & ~torch.isfinite(b)).any() for a, b in zip(got, wide))
    again = binding.givens_backward_restricted(th, y, g, m)
    assert torch.equal(again[0], want) and torch.equal(again[1], plain) and torch.isfinite(plain).all()


def test_gram_form_chosen_for_a_narrow_batch():
    th, x, g = problem(40, 39, 7, 5)
    want_y = binding.givens_forward(th.double(), x.double())
    want_dx, want_dth = binding.givens_backward(th.double(), want_y, g.double())
    dx, dth = binding.givens_backward_ex(th, want_y.float(), g, reduction=binding.REDUCTION_GRAM)
    assert rel(dx, want_dx) <= 1e-4 and rel(dth, want_dth) <= 1e-4


@pytest.mark.parametrize("n,B", [(16, 5000), (50, 30000), (64, 3000)])
def test_transposed_and_recorded(n, B):
    th, x, g = problem(n, n - 1, B, n)
    y, dx, dth = torch.empty_like(x), torch.empty_like(x), torch.empty_like(th)

    def step():
        binding.givens_forward(th, x, Y=y)
        binding.givens_backward(th, y, g, dX=dx, dtheta=dth)

    step()
    assert rel(binding.givens_forward_transposed(th, y), x.double()) <= 3e-5
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        step()
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for seed in range(3):                                          # replays on new values, eager work between them
        new = problem(n, n - 1, B, 100 + seed)
        for old, value in zip((th, x, g), new):
            old.copy_(value)
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in (y, dx, dth)]
        step()
        assert all(torch.equal(a, b) for a, b in zip(got, (y, dx, dth)))


# through autograd: the plain calls, which are the faster ones here
@pytest.mark.parametrize("n,m,B", [(40, None, 3000), (64, None, 130), (33, 8, 2500)])
def test_autograd_takes_the_plain_calls(n, m, B):
    from paper_2106_00003_amd import layer
    th, x, g = problem(n, n - 1 if m is None else m, B, n + B)
    y = binding.givens_forward_restricted(th, x, n - 1 if m is None else m)
    dx, dth = binding.givens_backward_restricted(th, y, g, n - 1 if m is None else m)
    thg, xg = th.clone().requires_grad_(True), x.clone().requires_grad_(True)
    before = binding.givens_prepare(th, n, m)                      # (tokens count the calls)
    out = layer.givens_apply(thg, xg, m)
    out.backward(g)
    assert binding.givens_prepare(th, n, m) == before + 1
    assert torch.equal(out.detach(), y) and torch.equal(xg.grad, dx) and torch.equal(thg.grad, dth)
