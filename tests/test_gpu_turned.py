"""Forward sweeps that read their coefficient table in the order of their lanes: batches on both sides of every line of the
rule, strips and workgroups that are partly filled, against the sweeps on prepared tables (which keep the order of the angles;
a strip's arithmetic does not depend on either, so the bits are the same) and against the float64 entry points."""
import pytest

from paper_2106_00003_amd import binding

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.set_kernel(binding.KERNEL_AUTO)     # (with a rotation form chosen: no tiles)
    yield
    binding.set_rotation_form(binding.FORM_RANGE)
    binding.release()


def rel(got, want):
    return float((got - want).norm() / want.norm())


# one wavefront per strip (528: 33 lanes, 1024: all), then strips of 2, 3 and 8 wavefronts (test_launch_choice.py: which are turned)
@pytest.mark.parametrize("n,B", [(528, 512), (528, 513), (528, 768), (528, 771), (1024, 1021), (1024, 1024), (1024, 1025),
                                 (1024, 1537), (768, 1535), (1008, 2007), (1040, 1041), (1040, 1561), (1536, 30), (3072, 257), (4096, 131)])
@pytest.mark.parametrize("form,scale", [(binding.FORM_STANDARD, 2.0), (binding.FORM_RANGE, 2.0), (binding.FORM_RANGE, 0.1)])
def test_forward(n, B, form, scale):
    binding.set_rotation_form(form)
    gen = torch.Generator(device="cuda").manual_seed(n + B)
    th = (torch.rand(n * (n - 1) // 2, device="cuda", generator=gen) * 2 - 1) * scale
    x = torch.randn(n, B, device="cuda", generator=gen)
    y = binding.givens_forward(th, x)
    token = binding.givens_prepare(th, n, None, binding.PREPARE_FORWARD)
    assert torch.equal(y, binding.givens_forward_prepared(token, x))
    assert rel(y.double(), binding.givens_forward(th.double(), x.double())) <= 1e-5
    assert rel(binding.givens_forward_transposed(th, y), x) <= 3e-5
    xr = x[:-1].contiguous()                                        # the added row of an odd problem
    count = binding.num_angles(n - 1, n // 3)
    yr = binding.givens_forward_restricted(th[:count], xr, n // 3)
    assert rel(yr.double(), binding.givens_forward_restricted(th[:count].double(), xr.double(), n // 3)) <= 1e-5


@pytest.mark.parametrize("n,B", [(528, 528), (1024, 1024)])
def test_build(n, B):
    binding.set_rotation_form(binding.FORM_STANDARD)
    gen = torch.Generator(device="cuda").manual_seed(n)
    th = (torch.rand(n * (n - 1) // 2, device="cuda", generator=gen) * 2 - 1) * 3
    u = binding.givens_build(th, n)
    assert rel(u.double(), binding.givens_build(th.double(), n)) <= 1e-5


# strips of 2 and 4 floats, one and four of them per workgroup (both sides of each line), and of two wavefronts
@pytest.mark.parametrize("n,B", [(128, 1), (144, 5), (512, 1023), (1024, 9), (1024, 1024), (1024, 1025), (640, 2047), (1024, 4090),
                                 (1024, 4097), (1040, 33), (128, 511), (272, 512), (272, 513), (336, 1280), (336, 1281), (512, 2048),
                                 (528, 2049), (784, 3072), (784, 3073)])
def test_unitary_forward(n, B):
    gen = torch.Generator(device="cuda").manual_seed(n + B)
    th, ph = ((torch.rand(n * (n - 1) // 2, device="cuda", generator=gen) * 2 - 1) * 3 for _ in range(2))
    x = torch.randn(n, B, device="cuda", generator=gen, dtype=torch.complex64)
    y = binding.givens_unitary_forward(th, ph, x)
    assert binding.last_kernel() == binding.KERNEL_CAROUSEL
    last = x[:, -min(B, 3):].contiguous()                            # columns do not interact
    if B < 4 * n:                                                    # (wider ones are multiplied)
        assert torch.equal(binding.givens_unitary_forward(th, ph, last), y[:, -min(B, 3):])
    few = x[:, -min(B, 70):].to(torch.complex128).contiguous()
    assert rel(y[:, -min(B, 70):].to(torch.complex128), binding.givens_unitary_forward(th.double(), ph.double(), few)) <= 1e-5


# through autograd: sizes whose plain calls are turned take those
@pytest.mark.parametrize("n,B", [(528, 520), (528, 64), (768, 1600)])
def test_autograd(n, B):
    from paper_2106_00003_amd import layer
    gen = torch.Generator(device="cuda").manual_seed(n * B)
    th = ((torch.rand(n * (n - 1) // 2, device="cuda", generator=gen) * 2 - 1) * 3).requires_grad_(True)
    x, g = torch.randn(n, B, device="cuda", generator=gen).requires_grad_(True), torch.randn(n, B, device="cuda", generator=gen)
    with torch.no_grad():
        y = binding.givens_forward(th.detach(), x.detach())
        dx, dth = binding.givens_backward(th.detach(), y, g)
    before = binding.givens_prepare(th.detach(), n)
    out = layer.givens_apply(th, x)
    out.backward(g)
    assert binding.givens_prepare(th.detach(), n) == before + (1 if B > 512 else 2)
    assert torch.equal(out.detach(), y) and torch.equal(x.grad, dx) and torch.equal(th.grad, dth)
