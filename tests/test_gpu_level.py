"""A level of the V-cycle in two launches (pre-smoothing, residual and restriction; correction and
post-smoothing) against its per-step launches, where the split changes: vectors of two and four
cells, one to four vectors per thread, tiles of 4 x 4 and 8 x 8 rows, rows that are no power of two,
levels right above the coarse tail."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# (nz, ny, nx): 24^3 has its tail right below; 36-cell rows take vectors of two; 72 x 56 x 40 and
# 64^3 two vectors per thread in FP32; 96 x 112 x 80 8 x 8 tiles and three
SHAPES = [(24, 24, 24), (20, 28, 36), (40, 56, 72), (64, 64, 64), (80, 112, 96)]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1306_3159_amd import native
    native.load_library()
    return torch.device("cuda:0")


@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_two_launch_level(dev, monkeypatch, shape, prec, box):
    """One V-cycle: bitwise equal in the periodic cell; in a box, whose transfers are summed in
    another order, to 1e-13 (FP64) and 100 units in the last place (FP32) of the largest value.
    And a reactive solve, whose CG takes the closing sweep of the finest level apart."""
    print("[case] two-launch level", shape, prec, box, flush=True)
    from paper_1306_3159_amd import BOUNDARY_DIRICHLET, BlobRD
    rng = np.random.default_rng(21)
    r = torch.as_tensor(rng.standard_normal(shape), device=dev)
    f = torch.as_tensor(1.0 + 0.5 * rng.standard_normal(shape), device=dev)
    nz, ny, nx = shape
    q = torch.as_tensor(rng.uniform(4.0, 16.0, (3, 3)), device=dev)
    kappa = torch.ones(3, dtype=torch.float64, device=dev)
    kw = dict(boundary=BOUNDARY_DIRICHLET, boundary_value=1.0) if box else {}
    out, rc = {}, {}
    for mode in ("1", "0"):
        monkeypatch.setenv("BLOB_RD_BLOCKED", mode)
        S = BlobRD(shape, q, kappa, precision=prec, rtol=1e-10, **kw)
        z = [S.vcycle(r, alpha).cpu().numpy() for alpha in (0.0, 0.4)]
        c, st = S.solve_reactive(f)
        out[mode] = z + [c.cpu().numpy()]
        rc[mode] = st["rc"]
        S.close()
    assert rc["1"] == rc["0"]  # (1e-10 is below the residual's rounding floor on the largest grid)
    for a, b in zip(out["1"], out["0"]):
        if box:
            assert np.max(np.abs(a - b)) < (1e-5 if prec else 1e-13 if a is not out["1"][2] else 1e-8) * np.abs(b).max()
        else:
            assert np.array_equal(a, b)
