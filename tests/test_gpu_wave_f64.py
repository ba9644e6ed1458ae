"""Float64 sweeps on one wavefront per strip: every kind of size (one to eight slots per lane, blocks before the unrolled
ones), both sides of each strip width, odd and restricted sizes, against the oracle and the LDS kernels they stand in for."""
import numpy as np
import pytest

from oracle import c_oracle as C
from oracle import givens_oracle as O
from paper_2106_00003_amd import binding, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    binding.set_kernel(binding.KERNEL_AUTO)
    yield
    binding.set_kernel(binding.KERNEL_AUTO)
    binding.release()


def far(got, want):
    return float((got - want).norm() / want.norm())


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("B", [1, 7])
def test_every_even_size_up_to_136(B):
    for n in range(2, 137, 2):
        data = inputs.make_custom(n, B, seed=4000 + n, dtype=np.float64)
        th, x, g = (dev(data[k]) for k in ("theta", "X", "G"))
        y = binding.givens_forward(th, x)
        want_y = C.forward(data["theta"], data["X"])
        want_dth, want_dx, _ = C.reverse_sweep(data["theta"], want_y, data["G"])
        dx, dth = binding.givens_backward(th, y, g)
        for got, want in ((y, want_y), (dx, want_dx), (dth, want_dth)):
            assert O.rel_fro(got.cpu().numpy(), want) <= TOL, n
        assert O.rel_fro(binding.givens_forward_transposed(th, y).cpu().numpy(), data["X"]) <= TOL, n


@pytest.mark.parametrize("n,B", [(64, 256), (64, 513), (64, 4099), (140, 257), (256, 512), (252, 1025), (504, 513),
                                 (512, 1024), (512, 4097), (528, 300), (1024, 70), (1008, 520), (32, 128), (32, 129),
                                 (260, 1026), (32, 9001), (1024, 2401)])
def test_strip_widths_against_the_lds_kernels(n, B):
    print(f"[wave64] n={n} B={B}", flush=True)
    data = inputs.make_custom(n, B, seed=4200 + n, dtype=np.float64)
    th, x, g = (dev(data[k]) for k in ("theta", "X", "G"))

    def run():
        y = binding.givens_forward(th, x)
        dx, dth = binding.givens_backward(th, y, g)
        return y, dx, dth, binding.givens_build(th, n), binding.givens_forward_transposed(th, x)

    got = run()
    binding.set_kernel(binding.KERNEL_LDS)
    want = run()
    binding.set_kernel(binding.KERNEL_AUTO)
    assert all(far(a, b) <= TOL for a, b in zip(got, want))
    buf = x.clone()
    assert torch.equal(binding.givens_forward(th, buf, Y=buf), got[0])
    buf = g.clone()
    assert torch.equal(binding.givens_backward(th, got[0], buf, dX=buf)[0], got[1])


# wavefronts of eight lanes with slots and fewer, whose other lanes stay on but one; nine, where none does: batches past the ones that
# take one kernel per call, strips of every width.  Beyond it the rows of other strips, sums and angles are as they should be.
@pytest.mark.parametrize("n,B", [(n, B) for n in (10, 12, 14, 16, 18) for B in (1025, 2049, 4099)] + [(16, 9001), (13, 3000), (15, 5000)])
def test_few_lanes_with_slots(n, B):
    data = inputs.make_restricted(n, n - 1, B, seed=4250 + n)
    th, x, g = (dev(data[k]).double() for k in ("theta", "X", "G"))

    def run():
        y = binding.givens_forward_restricted(th, x, n - 1)
        return (y, *binding.givens_backward_restricted(th, y, g, n - 1))

    got = run()
    binding.set_kernel(binding.KERNEL_LDS)
    want = run()
    binding.set_kernel(binding.KERNEL_AUTO)
    assert all(far(a, b) <= TOL for a, b in zip(got, want))


# one kernel per call: strips that end with the batch, just past it and far before it, the largest batch and the next; both sides of
# the sizes that take it.  Angles of 0 among the free ones, bypassed pairs, and odd sizes.  No more than some hundred roundings of
# 1.1e-16 lie between the two, so 1e-12 has room.
@pytest.mark.parametrize("n,m,B", [(2, 1, 128), (2, 1, 129), (8, 7, 32), (8, 7, 33), (7, 3, 64), (8, 7, 1024), (8, 7, 1025),
                                   (15, 14, 17), (16, 5, 16), (16, 15, 1024), (18, 17, 14), (18, 17, 15), (24, 23, 21), (23, 9, 22),
                                   (24, 2, 1024), (26, 25, 9), (26, 25, 10), (31, 30, 8), (32, 31, 8), (32, 31, 17), (32, 6, 16)])
def test_smallest_problems_in_one_kernel(n, m, B):
    print(f"[small64] n={n} m={m} B={B}", flush=True)
    data = inputs.make_restricted(n, m, B, seed=4600 + n)
    th, x, g = (dev(data[k]).double() for k in ("theta", "X", "G"))
    th[::3] = 0.0

    def run():
        y = binding.givens_forward_restricted(th, x, m)
        out = [y, *binding.givens_backward_restricted(th, y, g, m), binding.givens_build_restricted(th, n, m)]
        if n % 2 == 0 and m == n - 1:
            out.append(binding.givens_forward_transposed(th, x))
        return out

    got = run()
    binding.set_kernel(binding.KERNEL_LDS)
    want = run()
    binding.set_kernel(binding.KERNEL_AUTO)
    assert all(far(a, b) <= TOL for a, b in zip(got, want))
    buf = x.clone()
    assert torch.equal(binding.givens_forward_restricted(th, buf, m, Y=buf), got[0])
    buf = g.clone()
    dx, dth = binding.givens_backward_restricted(th, got[0], buf, m, dX=buf)
    assert torch.equal(dx, got[1]) and torch.equal(dth, got[2])


# both sides of the batch up to which a strip has a row of sums of its own, and single slots, where none has: dX has the
# same arithmetic, dtheta its sums in another order
@pytest.mark.parametrize("n,B", [(1024, 102), (1024, 103), (768, 136), (768, 137), (512, 205), (512, 206), (264, 256), (264, 257),
                                 (128, 1), (128, 6), (64, 127), (40, 3), (1024, 98), (1024, 99), (768, 174), (768, 175), (704, 168),
                                 (704, 169), (512, 219), (512, 220), (176, 128), (176, 129), (180, 256), (180, 257)])
def test_strips_with_and_without_a_row_of_their_own(n, B):
    data = inputs.make_restricted(n, n - 1, B, seed=4700 + n)
    th, y, g = (dev(data[k]).double() for k in ("theta", "X", "G"))
    got = binding.givens_backward(th, y, g)
    binding.set_kernel(binding.KERNEL_LDS)
    want = binding.givens_backward(th, y, g)
    binding.set_kernel(binding.KERNEL_AUTO)
    assert all(far(a, b) <= TOL for a, b in zip(got, want))


@pytest.mark.parametrize("n,m,B", [(11, 4, 9), (129, 128, 30), (255, 20, 300), (511, 510, 40), (512, 7, 600)])
def test_restricted_and_odd_sizes(n, m, B):
    data = inputs.make_restricted(n, m, B, seed=4400 + n)
    th, x, g = (dev(data[k]).double() for k in ("theta", "X", "G"))

    def run():
        y = binding.givens_forward_restricted(th, x, m)
        return (y, *binding.givens_backward_restricted(th, y, g, m))

    got = run()
    binding.set_kernel(binding.KERNEL_LDS)
    want = run()
    binding.set_kernel(binding.KERNEL_AUTO)
    assert all(far(a, b) <= TOL for a, b in zip(got, want))


# Infinities and NaN stay in the columns and the angles they reach, in one kernel per call (n <= 32), in strips of their own and in
# strips that share a row of sums: where the LDS kernels' results are finite the values are close, elsewhere neither is finite.
@pytest.mark.parametrize("n,B", [(2, 9), (8, 4), (15, 40), (16, 200), (24, 700), (32, 8), (32, 2000), (64, 64), (64, 513), (200, 129),
                                 (512, 1025), (1008, 70), (1024, 800)])
def test_infinities_and_nan_stay_where_they_belong(n, B):
    print(f"[wave64] infinities n={n} B={B}", flush=True)
    data = inputs.make_restricted(n, n - 1, B, seed=4700 + n)
    th, x, g = (dev(data[k]).double() for k in ("theta", "X", "G"))
    y = binding.givens_forward_restricted(th, x, n - 1)
    bad_x, bad_g = x.clone(), g.clone()
    bad_x[0, 0], bad_x[n - 1, B // 2], bad_x[n // 2, B - 1] = float("nan"), float("inf"), -float("inf")
    bad_g[n // 2, 1], bad_g[n - 1, B - 1] = float("inf"), float("nan")

    def run():
        return [binding.givens_forward_restricted(th, bad_x, n - 1), *binding.givens_backward_restricted(th, y, bad_g, n - 1)]

    got = run()
    binding.set_kernel(binding.KERNEL_LDS)
    want = run()
    binding.set_kernel(binding.KERNEL_AUTO)
    for a, b in zip(got, want):
        finite = torch.isfinite(b)
        assert torch.equal(torch.isfinite(a), finite) and not finite.all()
        if finite.any():
            assert far(a[finite], b[finite]) <= TOL
