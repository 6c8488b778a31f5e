"""Forms of the V-cycle's and the Krylov kernels that only some sizes take: tiles of a large level in more than
one group of planes and tiles that reach beyond the last plane or row, the box's coarse tail, GMRES columns
beyond those whose scalars are held in LDS, folded sums in a box."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import dirichlet as dr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1306_3159_amd import native
    native.load_library()
    return torch.device("cuda:0")


def no_blobs(dev):
    return torch.zeros((0, 3), dtype=torch.float64, device=dev)


# (nz, ny, nx): five planes of tiles (a group of four and one of one) in both precisions; in FP64 also 2.5
# planes of tiles with 3.1 segments a row, and 2.5 rows of tiles
@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("shape,prec", [((40, 24, 256), 0), ((40, 24, 256), 1), ((20, 16, 100), 0), ((16, 20, 96), 0)])
def test_tile_groups_and_partial_tiles(dev, monkeypatch, shape, prec, box):
    """One V-cycle against the per-step launches: bitwise in the periodic cell, in a box, whose transfers are
    summed in another order, to 1e-13 (FP64) and 1e-5 (FP32) of the largest value."""
    from paper_1306_3159_amd import BOUNDARY_DIRICHLET, BlobRD
    print("[case] tiles", shape, prec, box, flush=True)
    r = torch.as_tensor(np.random.default_rng(41).standard_normal(shape), device=dev)
    kw = dict(boundary=BOUNDARY_DIRICHLET) if box else {}
    out = {}
    for mode in ("1", "0"):
        monkeypatch.setenv("BLOB_RD_BLOCKED", mode)
        S = BlobRD(shape, no_blobs(dev), precision=prec, **kw)
        out[mode] = [S.vcycle(r, alpha).cpu().numpy() for alpha in (0.0, 0.4)]
        words = S.time_kernel("vcycle", reps=1)[1]
        out[mode].append(words)
        S.close()
    assert out["1"][2] < 0.75 * out["0"][2]  # the levels above the tail are indeed not in per-step launches
    for a, b in zip(out["1"][:2], out["0"][:2]):
        if box:
            assert np.max(np.abs(a - b)) < (1e-5 if prec else 1e-13) * np.abs(b).max()
        else:
            assert np.array_equal(a, b)


@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", [(24, 24, 24), (20, 28, 36), (40, 56, 72), (64, 64, 64), (80, 112, 96), (40, 24, 256)])
def test_solve_with_levels_in_few_launches(dev, monkeypatch, shape, prec, box):
    """Reactive solves with and without them both converge, to solutions c with |A c - f| <= rtol |f|; A's
    eigenvalues are at least alpha, so two of them differ by at most 2 rtol |f| / alpha."""
    from paper_1306_3159_amd import BOUNDARY_DIRICHLET, BlobRD
    print("[case] solves", shape, prec, box, flush=True)
    rng = np.random.default_rng(43)
    f = torch.as_tensor(1.0 + 0.5 * rng.standard_normal(shape), device=dev)
    q = torch.as_tensor(rng.uniform(5.0, 15.0, (3, 3)), device=dev)
    kappa = torch.ones(3, dtype=torch.float64, device=dev)
    kw = dict(boundary=BOUNDARY_DIRICHLET, boundary_value=0.0) if box else {}
    alpha, rtol, c = 0.4, 1e-8, []
    for mode in ("1", "0"):
        monkeypatch.setenv("BLOB_RD_BLOCKED", mode)
        S = BlobRD(shape, q, kappa, precision=prec, rtol=rtol, **kw)
        x, st = S.solve_reactive(f, alpha=alpha)
        assert st["rc"] == 0
        c.append(x)
        S.close()
    assert float((c[0] - c[1]).norm()) <= 2 * rtol / alpha * float(f.norm())
    if not box:
        assert torch.equal(c[0], c[1])


def axis_prolong(n):
    """1D interpolation from n/2 to n cells of a box: 3/4 and 1/4; next to a face, beyond which the coarse
    value is -u, 1/2 of the parent."""
    P = np.zeros((n, n // 2))
    for i in range(n):
        own, near = i // 2, i // 2 + (1 if i % 2 else -1)
        inside = 0 <= near < n // 2
        P[i, own] = 0.75 if inside else 0.5
        if inside:
            P[i, near] = 0.25
    return P


def along_axes(mats, v):
    for axis, m in enumerate(mats):
        v = np.moveaxis(np.tensordot(m, v, (1, axis)), 0, axis)
    return v


def box_cycle(f, alpha, h=1.0):
    """The V-cycle on alpha I - D L_0 with D = 1: red, black, red, black from zero, residual restricted by the
    transposed interpolation over 8, correction, black, red, black, red; exact on a grid that has an odd edge or
    one of at most four cells."""
    n = f.shape
    if any(s % 2 for s in n) or min(n) <= 4:
        return dr.solve_A0(f, alpha, 1.0, h)
    idx = np.indices(n)
    colour = idx.sum(0) % 2
    faces = sum((i == 0).astype(int) + (i == s - 1) for i, s in zip(idx, n))
    diag = alpha + (6.0 + faces) / h ** 2
    u = np.zeros(n)

    def sweep(c):
        v = u + (f - dr.apply_A0(u, alpha, 1.0, h)) / diag
        return np.where(colour == c, v, u)

    for c in (0, 1, 0, 1):
        u = sweep(c)
    P = [axis_prolong(s) for s in n]
    R = [p.T / 2.0 for p in P]
    u = u + along_axes(P, box_cycle(along_axes(R, f - dr.apply_A0(u, alpha, 1.0, h)), alpha, 2.0 * h))
    for c in (1, 0, 1, 0):
        u = sweep(c)
    return u


@pytest.mark.parametrize("alpha", [0.0, 0.7])
@pytest.mark.parametrize("shape", [(8, 8, 8), (12, 12, 12), (16, 16, 16), (14, 20, 12), (16, 24, 20), (20, 28, 24)])
def test_box_tail_against_plain_cycle(dev, shape, alpha):
    """The coarse tail in a box: FP64 to rounding (a few hundred operations a cell), FP32 within 100 units in the
    last place of the field's largest value, as the periodic tail against its oracle."""
    from paper_1306_3159_amd import BOUNDARY_DIRICHLET, BlobRD
    print("[case] box tail", shape, alpha, flush=True)
    r = np.random.default_rng(47).standard_normal(shape)
    ref = box_cycle(r, alpha)
    for prec, tol in ((0, 1e-12), (1, 1e-5)):
        S = BlobRD(shape, no_blobs(dev), precision=prec, boundary=BOUNDARY_DIRICHLET)
        z = S.vcycle(torch.as_tensor(r, device=dev), alpha).cpu().numpy()
        S.close()
        assert np.max(np.abs(z - ref)) < tol * np.abs(ref).max()


def test_gmres_columns_beyond_lds(dev):
    """Inner GMRES of the block preconditioner with 128 columns (scalars in LDS) and more (in memory). Here 120
    columns have reduced the residual to its rounding level (a Schur system of this kind takes some 40 to
    1e-8), so further ones change the result by rounding only."""
    import workloads as W
    from paper_1306_3159_amd import BlobRD
    print("[case] GMRES columns", flush=True)
    rng = np.random.default_rng(53)
    n, N = 32, 300
    q = torch.as_tensor(W.rsa_positions(rng, n, N, 3.0), device=dev)
    vg = torch.as_tensor(rng.standard_normal((n, n, n)), device=dev)
    vf = torch.as_tensor(rng.standard_normal(N), device=dev)
    S = BlobRD(n, q, gmres_restart=200)
    ref_g, ref_l = S.saddle_precond(vg, vf, alpha=0.3, m=120)
    for m in (127, 128, 129, 130, 192, 200):
        zg, zl = S.saddle_precond(vg, vf, alpha=0.3, m=m)
        assert float((zl - ref_l).norm() / ref_l.norm()) < 1e-9
        assert float((zg - ref_g).norm() / ref_g.norm()) < 1e-9
    S.close()


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("box", [False, True])
def test_folded_step_with_many_blobs(dev, prec, box):
    """CG's step is formed by the update up to 2048 blobs and by its own launch beyond, in the same order: one
    more blob of zero rate changes no bit of the solution."""
    from paper_1306_3159_amd import BOUNDARY_DIRICHLET, BlobRD
    print("[case] folded step", prec, box, flush=True)
    rng = np.random.default_rng(59)
    n, N = 40, 2049
    q = torch.as_tensor(rng.uniform(3.5, n - 3.5, (N, 3)), device=dev)
    kappa = torch.as_tensor(rng.uniform(0.5, 2.0, N), device=dev)
    kappa[-1] = 0.0
    f = torch.as_tensor(1.0 + 0.5 * rng.standard_normal((n, n, n)), device=dev)
    kw = dict(boundary=BOUNDARY_DIRICHLET, boundary_value=0.5) if box else {}
    c = []
    for k in (N - 1, N):
        S = BlobRD(n, q[:k].contiguous(), kappa[:k].contiguous(), precision=prec, **kw)
        x, st = S.solve_reactive(f)
        assert st["rc"] == 0 and st["outer_iters"] > 2
        c.append(x)
        S.close()
    assert torch.equal(c[0], c[1])
