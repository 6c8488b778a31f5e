"""The coarse end of the V-cycle (one work-group, levels in LDS) at the sizes where its split over
threads changes: one, two, four and eight indices of its first level per thread, rows that are no
power of two, odd coarsest grids, two and three levels."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import dirichlet as dr
from oracle import iterative as it

pytestmark = pytest.mark.gpu

# (nz, ny, nx): half the cells of the tail's first level are 256, 864, 2048, 1680, 3840 and 6720
# (FP64 starts the last one a level lower, its LDS budget holding fewer cells)
SHAPES = [(8, 8, 8), (12, 12, 12), (16, 16, 16), (14, 20, 12), (16, 24, 20), (20, 28, 24)]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1306_3159_amd import native
    native.load_library()
    return torch.device("cuda:0")


def cycle(dev, shape, r, alpha, **kw):
    from paper_1306_3159_amd import BlobRD
    S = BlobRD(shape, torch.zeros((0, 3), dtype=torch.float64, device=dev), **kw)
    z = S.vcycle(torch.as_tensor(r, device=dev), alpha).cpu().numpy()
    S.close()
    return z


@pytest.mark.parametrize("alpha", [0.0, 0.7])
@pytest.mark.parametrize("shape", SHAPES)
def test_tail_periodic(dev, shape, alpha):
    """Against the oracle's cycle: FP64 to rounding (a few hundred operations a cell), FP32 within
    100 units in the last place of the field's largest value."""
    print("[case] tail periodic", shape, alpha, flush=True)
    from paper_1306_3159_amd import FP64, MIXED
    r = np.random.default_rng(11).standard_normal(shape)
    if alpha == 0.0:
        r -= r.mean()
    ref = it.vcycle(r, alpha)
    big = np.abs(ref).max()
    assert np.max(np.abs(cycle(dev, shape, r, alpha, precision=FP64) - ref)) < 1e-12 * big
    assert np.max(np.abs(cycle(dev, shape, r, alpha, precision=MIXED) - ref)) < 1e-5 * big


@pytest.mark.parametrize("alpha", [0.0, 0.7])
@pytest.mark.parametrize("shape", SHAPES)
def test_tail_box(dev, shape, alpha):
    """The box cycle is symmetric (it preconditions CG) and cuts the residual several times; FP32
    agrees with FP64 within 100 units in the last place of the field's largest value."""
    print("[case] tail box", shape, alpha, flush=True)
    from paper_1306_3159_amd import BOUNDARY_DIRICHLET, FP64, MIXED
    rng = np.random.default_rng(12)
    a, b = rng.standard_normal(shape), rng.standard_normal(shape)
    kw = dict(boundary=BOUNDARY_DIRICHLET, boundary_value=1.0)
    va, vb = (cycle(dev, shape, v, alpha, precision=FP64, **kw) for v in (a, b))
    assert abs(np.sum(va * b) - np.sum(a * vb)) < 1e-12 * np.linalg.norm(va) * np.linalg.norm(b)
    assert np.linalg.norm(a - dr.apply_A0(va, alpha)) < 0.25 * np.linalg.norm(a)
    assert np.max(np.abs(cycle(dev, shape, a, alpha, precision=MIXED, **kw) - va)) < 1e-5 * np.abs(va).max()
