"""The library's own defaults (GIVENS_FORM_AUTO), under which sizes take the tiles, and batches the product, by themselves:
plain, restricted, prepared, transposed, in place and through autograd, against the float64 entry points."""
import numpy as np
import pytest

from paper_2106_00003_amd import binding

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL_Y, TOL_G = 1e-5, 1e-4


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    binding.set_kernel(binding.KERNEL_AUTO)
    binding.set_reduction(binding.REDUCTION_AUTO)
    yield
    binding.release()


@pytest.fixture(autouse=True)
def _library_defaults(_forms_by_range):
    binding.set_rotation_form(binding.FORM_AUTO)


def rel(got, want):
    return float((got.double() - want).norm() / want.norm())


def _cases():
    rng = np.random.default_rng(20210689)
    sizes = [401, 402, 514, 515, 700, 706, 882, 898, 901, 930, 1001, 1002, 1006, 1022, 1023, 1024, 1030, 1278, 1280, 1302,
             2049, 2050, 300, 129]
    out = []
    for idx, n in enumerate(sizes * 2):
        B = int(rng.choice([1, 5, 33, 64, 257, n // 2 + 1, (3 * n) // 4, n, 2 * n, 2500]))
        m = int(rng.integers(1, n)) if rng.random() < 0.4 else n - 1
        out.append((idx, n, min(B, 1500) if n > 1400 else B, m, ["uniform", "small", "huge"][int(rng.integers(0, 3))]))
    return out


@pytest.mark.parametrize("idx,n,B,m,angles", _cases())
def test_random_problems(idx, n, B, m, angles):
    from paper_2106_00003_amd import layer
    gen = torch.Generator(device="cuda").manual_seed(9000 + idx)
    count = binding.num_angles(n, m)
    th = torch.randn(count, device="cuda", generator=gen) * {"uniform": 1.8, "small": 0.1, "huge": 1e4}[angles]
    x, g = (torch.randn(n, B, device="cuda", generator=gen) for _ in range(2))
    print(f"[defaults] case {idx}: n={n} B={B} m={m} angles={angles}", flush=True)
    want_y = binding.givens_forward_restricted(th.double(), x.double(), m)
    want_dx, want_dth = binding.givens_backward_restricted(th.double(), want_y, g.double(), m)
    y = binding.givens_forward_restricted(th, x, m)
    dx, dth = binding.givens_backward_restricted(th, y, g, m)
    assert rel(y, want_y) <= TOL_Y and rel(dx, want_dx) <= TOL_G and rel(dth, want_dth) <= TOL_G
    buf = x.clone()
    assert torch.equal(binding.givens_forward_restricted(th, buf, m, Y=buf), y)
    buf = g.clone()
    assert torch.equal(binding.givens_backward_restricted(th, y, buf, m, dX=buf)[0], dx)
    token = binding.givens_prepare(th, n, m, directions=binding.PREPARE_FORWARD | binding.PREPARE_BACKWARD_WIDE, batch=B)
    assert rel(binding.givens_forward_prepared(token, x), want_y) <= TOL_Y
    pdx, pdth = binding.givens_backward_prepared(token, y, g, count)
    assert rel(pdx, want_dx) <= TOL_G and rel(pdth, want_dth) <= TOL_G
    if n % 2 == 0 and m == n - 1:
        back = binding.givens_forward_transposed(th, y)
        assert rel(back, x.double()) <= 3 * TOL_Y
    thg, xg = th.clone().requires_grad_(True), x.clone().requires_grad_(True)
    out = layer.givens_apply(thg, xg, m)
    out.backward(g)
    assert rel(out.detach(), want_y) <= TOL_Y and rel(xg.grad, want_dx) <= TOL_G and rel(thg.grad, want_dth) <= TOL_G


# a column of its own: infinities and NaN stay in it, on every route (tiles, product of every tile, sweep, packed and kept)
@pytest.mark.parametrize("n,B", [(6, 3), (64, 40000), (256, 64), (258, 40001), (514, 70), (1006, 64), (1006, 2100), (1024, 2100)])
def test_infinities_and_nan_stay_in_their_columns(n, B):
    from paper_2106_00003_amd import layer
    gen = torch.Generator(device="cuda").manual_seed(9100 + n)
    net = layer.OrthogonalLinear(n)
    x = torch.randn(n, B, device="cuda", generator=gen)
    bad = x.clone()
    bad[1, 0], bad[n - 1, B // 2], bad[n // 2, B - 1] = float("nan"), float("inf"), -float("inf")
    clean = torch.ones(B, dtype=torch.bool, device="cuda")
    clean[[0, B // 2, B - 1]] = False
    th = net.theta.detach()
    packed = binding.givens_pack(binding.givens_build(th, n))
    with torch.no_grad():
        net(x), net(x)
        for call in (lambda t: binding.givens_forward(th, t), lambda t: binding.givens_forward_transposed(th, t),
                     lambda t: binding.givens_apply_packed(packed, t), net):
            want, got = call(x), call(bad)
            assert torch.equal(got[:, clean], want[:, clean])
            assert not torch.isfinite(got[:, ~clean]).all(dim=0).any()
