"""The entry point that allocates nothing (givens_forward_noalloc) against givens_forward, through the
C ABI: two calls in a row, the second on a smaller problem, so that whatever the first call left in the
library's static device array is there when the second runs.  The two entry points launch the same
kernels on the same inputs, so the outputs must agree bit for bit (which is inside the fp32 tolerance
of 1e-5 on Y that both are held to against the oracle; that comparison is made here as well).
"""
import numpy as np
import pytest

from oracle import c_oracle as C
from oracle import givens_oracle as O
from paper_2106_00003_amd import binding, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL_Y = 1e-5


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    binding.set_kernel(binding.KERNEL_AUTO)
    yield
    binding.release()


def _both(n, B, seed, dist):
    data = inputs.make_custom(n, B, seed=seed, theta_dist=dist)
    th, X = data["theta"], data["X"]
    print(f"[noalloc] n={n} B={B} seed={seed} {dist}", flush=True)
    th_d, x_d = torch.from_numpy(th).cuda(), torch.from_numpy(X).cuda()
    y_new = torch.full_like(x_d, float("nan"))
    binding.givens_forward_noalloc(th_d, x_d, y_new)
    family = binding.last_kernel()
    torch.cuda.synchronize()
    y_ref = binding.givens_forward(th_d, x_d)
    assert binding.last_kernel() == family
    torch.cuda.synchronize()
    assert torch.equal(y_new, y_ref)
    err = O.rel_fro(y_new.cpu().numpy(), C.forward(th, X))
    print(f"[noalloc] n={n} B={B}: identical to givens_forward, Y err vs oracle {err:.3e}", flush=True)
    assert err <= TOL_Y


def test_two_calls_in_a_row_second_smaller():
    _both(1024, 300, 401, "uniform")       # largest n the static array takes; carousel family, lifted form
    _both(256, 77, 402, "normal0.1")       # smaller: scaled form, tables shorter than what the array holds
    _both(64, 130, 403, "uniform")         # column family
    _both(130, 9, 404, "uniform")          # LDS strip family


def test_in_place_and_repeated():
    data = inputs.make_custom(512, 64, seed=405)
    th_d, x_d = torch.from_numpy(data["theta"]).cuda(), torch.from_numpy(data["X"]).cuda()
    want = binding.givens_forward(th_d, x_d)
    for _ in range(3):
        buf = x_d.clone()
        binding.givens_forward_noalloc(th_d, buf, buf)
        torch.cuda.synchronize()
        assert torch.equal(buf, want)


def test_sizes_beyond_the_static_array_are_rejected():
    n = binding.NOALLOC_MAX_N + 2
    th_d = torch.zeros(n * (n - 1) // 2, device="cuda")
    x_d = torch.ones(n, 4, device="cuda")
    y_d = torch.zeros_like(x_d)
    with pytest.raises(binding.GivensError) as info:
        binding.givens_forward_noalloc(th_d, x_d, y_d)
    assert info.value.code == -5
    torch.cuda.synchronize()
    assert float(y_d.abs().max()) == 0.0   # nothing was launched


# under the library's defaults, where some sizes take the tiles by themselves: their smallest, sizes without a carousel
# shape, with one of 3, 5 and 7 slots, and the largest; narrow, below and above the batch that goes through U
@pytest.mark.parametrize("n", [402, 514, 882, 998, 1002, 1006, 1010, 1022, 1024])
def test_equal_under_the_library_defaults(n):
    binding.set_rotation_form(binding.FORM_AUTO)
    binding.set_kernel(binding.KERNEL_AUTO)
    for B in (1, 33, 700, 2047, 2100):
        data = inputs.make_custom(n, B, seed=410 + n)
        th, x = (torch.from_numpy(data[k]).cuda() for k in ("theta", "X"))
        print(f"[noalloc] defaults n={n} B={B}", flush=True)
        want = binding.givens_forward(th, x)
        family = binding.last_kernel()
        y = torch.full_like(x, float("nan"))
        binding.givens_forward_noalloc(th, x, y)
        assert binding.last_kernel() == family
        assert torch.equal(y, want)
        buf = x.clone()
        binding.givens_forward_noalloc(th, buf, buf)
        assert torch.equal(buf, want)


def test_the_range_check_after_calls_without_one():
    """The flag words take turns among the calls that make a range check, whatever runs between them."""
    n, B = 512, 40
    th, x = torch.empty(n * (n - 1) // 2, device="cuda"), torch.randn(n, B, device="cuda")
    y = torch.empty_like(x)
    for large, small in ((3.0, 0.1), (3.0, 0.1)):
        for between in (0, 1, 2):
            th.fill_(large)
            binding.set_rotation_form(binding.FORM_RANGE)
            binding.givens_forward_noalloc(th, x, y)
            assert binding.last_rotation_form() == binding.FORM_LIFTED
            binding.set_rotation_form(binding.FORM_STANDARD)
            for _ in range(between):
                binding.givens_forward_noalloc(th, x, y)
            binding.set_rotation_form(binding.FORM_RANGE)
            th.fill_(small)
            binding.givens_forward_noalloc(th, x, y)
            assert binding.last_rotation_form() == binding.FORM_SCALED
