"""The filter on few elements and thin grids, where one thread per element sums the
window. There the weighted sum of a constant and the sum of the weights are the same
sums, so a uniform design stays exactly uniform. On both sides of the rule that
chooses between the forms each agrees with sums by shifts of the grid within 1e-13 (as in
tests/test_gpu_filter.py)."""
import numpy as np
import pytest

import oracle as O
from tests.test_gpu_filter import _by_shifts

pytestmark = pytest.mark.gpu


def _both(nx, ny, r, beta, chi, grad):
    import torch

    from paper_2411_19030_amd import _pt
    f = _pt.make_filter(nx, ny, r, beta, 0.5)
    c, g = torch.tensor(chi, device="cuda"), torch.tensor(grad, device="cuda")
    fil, phys, work, gc = (torch.empty_like(c) for _ in range(4))
    _pt.pt_filter_projection(f, c, fil, phys)
    _pt.pt_filter_projection_backward(f, fil, g, work, gc)
    torch.cuda.synchronize()
    return fil.cpu().numpy(), phys.cpu().numpy(), gc.cpu().numpy()


@pytest.mark.parametrize("nx,ny,r", [(100, 100, 0.03), (64, 64, 0.05), (199, 150, 0.03),
                                     (2000, 10, 0.05), (16384, 1, 0.01), (300, 12, 0.8)])
def test_uniform_design_stays_uniform_on_few_elements(gpu, nx, ny, r):
    fil, _, _ = _both(nx, ny, r, 32.0, np.ones(nx * ny), np.ones(nx * ny))
    assert np.all(fil == 1.0)


# forward and backward by one thread per element; forward so, backward by tiles; both by tiles
@pytest.mark.parametrize("nx,ny,r", [(2000, 10, 0.05), (64, 64, 0.05), (64, 64, 0.2),
                                     (256, 256, 0.03), (5, 700, 0.1)])
def test_both_sides_of_the_rule(gpu, nx, ny, r):
    rng = np.random.default_rng(nx + 7 * ny)
    chi, grad = rng.uniform(0.0, 1.0, nx * ny), rng.standard_normal(nx * ny)
    fil, phys, gc = _both(nx, ny, r, 8.0, chi, grad)
    num, W = _by_shifts(nx, ny, r, chi)
    o_fil = num / W
    o_phys = O.design.projection(o_fil, 8.0, 0.5)
    o_gc, _ = _by_shifts(nx, ny, r, O.design.projection_deriv(o_fil, 8.0, 0.5) * grad / W)
    for a, b in ((fil, o_fil), (phys, o_phys), (gc, o_gc)):
        assert np.abs(a - b).max() <= 1e-13 * np.abs(b).max()
