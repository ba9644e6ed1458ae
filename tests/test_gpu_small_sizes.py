"""Sizes up to 128 run one wavefront per strip of columns, every even n with its own number of blocks before the unrolled
ones: both sweeps against the oracle, at the batches where strips get wider, and the calls that share the route."""
import numpy as np
import pytest

from oracle import c_oracle as C
from oracle import givens_oracle as O
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


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def far(got, want):
    return float((got - want).norm() / want.norm())


@pytest.mark.parametrize("B", [1, 5, 300])
def test_every_even_size_up_to_132(B):
    for n in range(2, 133, 2):
        data = inputs.make_custom(n, B, seed=2000 + n)
        th, x, g = (dev(data[k]) for k in ("theta", "X", "G"))
        y = binding.givens_forward(th, x)
        want_y = C.forward(data["theta"], data["X"])
        assert O.rel_fro(y.cpu().numpy(), want_y) <= TOL_Y, n
        want_dth, want_dx, _ = C.reverse_sweep(data["theta"], want_y, data["G"])
        for reduction in (binding.REDUCTION_TWO_STAGE, binding.REDUCTION_GRAM):
            dx, dth = binding.givens_backward_ex(th, y, g, reduction=reduction)
            assert O.rel_fro(dx.cpu().numpy(), want_dx) <= TOL_G, (n, reduction)
            assert O.rel_fro(dth.cpu().numpy(), want_dth) <= TOL_G, (n, reduction)
        back = binding.givens_forward_transposed(th, y)
        assert O.rel_fro(back.cpu().numpy(), data["X"]) <= 2 * TOL_Y, n


# strips of 1, 2, 4 and 8 columns forward (1, 2, 4 reverse), a last strip that is not full, column kernel and product
@pytest.mark.parametrize("n", [16, 30, 32, 58, 128])
@pytest.mark.parametrize("B", [257, 1025, 2047, 2049, 4097, 16385])
def test_strip_widths_of_small_sizes(n, B):
    data = inputs.make_custom(n, B, seed=2200 + n)
    th, x, g = (dev(data[k]) for k in ("theta", "X", "G"))
    y = binding.givens_forward(th, x)
    want_y = binding.givens_forward(th.double(), x.double())
    assert far(y, want_y) <= TOL_Y
    want_dx, want_dth = binding.givens_backward(th.double(), want_y, g.double())
    for reduction in (binding.REDUCTION_TWO_STAGE, binding.REDUCTION_GRAM):
        dx, dth = binding.givens_backward_ex(th, y, g, reduction=reduction)
        assert far(dx, want_dx) <= TOL_G and far(dth, want_dth) <= TOL_G
    token = binding.givens_prepare(th, n, directions=binding.PREPARE_FORWARD | binding.PREPARE_BACKWARD)
    assert torch.equal(binding.givens_forward_prepared(token, x), y)
    _, dth = binding.givens_backward_prepared(token, y, g, th.numel())
    assert far(dth, want_dth) <= TOL_G
    buf = x.clone()
    assert torch.equal(binding.givens_forward(th, buf, Y=buf), y)
    assert torch.equal(binding.givens_forward_noalloc(th, x, torch.empty_like(x)), y)


@pytest.mark.parametrize("n,m,B", [(17, 5, 40), (33, 32, 7), (126, 20, 300), (127, 126, 50)])
def test_small_restricted_and_odd_sizes(n, m, B):
    data = inputs.make_restricted(n, m, B, seed=2400 + n)
    th, x, g = (dev(data[k]) for k in ("theta", "X", "G"))
    y = binding.givens_forward_restricted(th, x, m)
    dx, dth = binding.givens_backward_restricted(th, y, g, m)
    want_y = binding.givens_forward_restricted(th.double(), x.double(), m)
    want_dx, want_dth = binding.givens_backward_restricted(th.double(), want_y, g.double(), m)
    assert far(y, want_y) <= TOL_Y and far(dx, want_dx) <= TOL_G and far(dth, want_dth) <= TOL_G
