"""A large level of the V-cycle in tiles cut on all axes (three half-sweeps in one launch, residual
with restriction) against its per-step launches: rows of whole and partial segments of eight
vectors, a last tile that reaches beyond the rows, two such levels above each other."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# (nz, ny, nx): rows too long for a level's two-launch form; 200 = 3.1 segments in FP32, 6.25 in
# FP64, where 100 x 20 x 16 below (3.1 segments, 2.5 tiles of rows) is such a level too
SHAPES = [(32, 40, 200), (32, 32, 256)]


@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_slab_level(monkeypatch, shape, prec, box):
    """One V-cycle: bitwise equal in the periodic cell; in a box, whose transfers are summed in
    another order, to 1e-13 (FP64) and 1e-5 (FP32) of the largest value. And a reactive solve, whose
    CG enters the cycle with no stored red sweep, to ten times its tolerance in the box."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1306_3159_amd import BOUNDARY_DIRICHLET, BlobRD
    print("[case] slab level", shape, prec, box, flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(31)
    r = torch.as_tensor(rng.standard_normal(shape), device=dev)
    f = torch.as_tensor(1.0 + 0.5 * rng.standard_normal(shape), device=dev)
    q = torch.as_tensor(rng.uniform(5.0, 11.0, (3, 3)), device=dev)
    kappa = torch.ones(3, dtype=torch.float64, device=dev)
    kw = dict(boundary=BOUNDARY_DIRICHLET, boundary_value=1.0) if box else {}
    out = {}
    for mode in ("1", "0"):
        monkeypatch.setenv("BLOB_RD_BLOCKED", mode)
        S = BlobRD(shape, q, kappa, precision=prec, rtol=1e-7, **kw)
        out[mode] = [S.vcycle(r, alpha).cpu().numpy() for alpha in (0.0, 0.4)]
        c, st = S.solve_reactive(f, alpha=0.4)
        assert st["rc"] == 0
        out[mode].append(c.cpu().numpy())
        S.close()
    for k, (a, b) in enumerate(zip(out["1"], out["0"])):
        if box:
            assert np.max(np.abs(a - b)) < (1e-6 if k == 2 else 1e-5 if prec else 1e-13) * np.abs(b).max()
        else:
            assert np.array_equal(a, b)
