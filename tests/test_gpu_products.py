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
