"""CG's direction, product and steps of the solution in one launch: the solution holds every step
whatever the number of iterations (steps are taken two iterations at a time, the rest at the end),
for even and odd counts, one to several cell pairs per thread, both precisions, periodic and box."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", [(8, 8, 8), (20, 28, 36), (128, 128, 160)])
def test_solution_holds_every_step(shape, prec, box):
    """CG stops once the recurred residual is below half the tolerance; the residual of the returned
    solution, formed anew in FP64, differs from it by the rounding of A c (norm of A 12 D / h^2, some units
    in the last place), while a step missing from the solution would leave it several times above."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1306_3159_amd import BOUNDARY_DIRICHLET, BlobRD
    print("[case] CG steps", shape, prec, box, flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(5)
    f = torch.as_tensor(1.0 + 0.5 * rng.standard_normal(shape), device=dev)
    q = torch.as_tensor(rng.uniform(0.4, 0.6, (3, 3)) * min(shape), device=dev)
    kappa = torch.full((3,), 2.0, dtype=torch.float64, device=dev)
    kw = dict(boundary=BOUNDARY_DIRICHLET, boundary_value=1.0) if box else {}
    counts = set()
    for rtol in (1e-1, 1e-2, 1e-3, 1e-4, 1e-5, 1e-6, 1e-7, 1e-8):
        S = BlobRD(shape, q, kappa, precision=prec, rtol=rtol, **kw)
        for alpha in (0.0, 0.3):
            c, st = S.solve_reactive(f, alpha=alpha)
            slack = 20 * 2.0 ** -52 * 12.0 * float(c.norm() / f.norm())
            if slack >= 0.1 * rtol:
                continue  # near the floor that rounding sets
            assert st["rc"] == 0 and st["refinements"] == 0
            assert st["rel_resid"] <= 0.5 * rtol + slack
            counts.add(st["outer_iters"])
        S.close()
    assert {k % 2 for k in counts} == {0, 1}, counts


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,blobs", [(32, 1), (32, 64), (32, 1025), (64, 2048), (64, 2049)])
def test_sums_formed_by_the_next_pass(n, blobs, prec):
    """A solve alone lets CG's vector passes finish the reductions before them (up to 512 blocks, 2048
    blobs), a batch's rounds finish them in their own launches: the same bits either way."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1306_3159_amd import Batch, BlobRD
    print("[case] CG sums", n, blobs, prec, flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(9)
    shape = (n, n, n)
    f = torch.as_tensor(1.0 + 0.5 * rng.standard_normal(shape), device=dev)
    q = torch.as_tensor(rng.uniform(0.0, n, (blobs, 3)), device=dev)
    kappa = torch.as_tensor(rng.uniform(0.5, 2.0, blobs), device=dev)
    S = BlobRD(shape, q, kappa, precision=prec, rtol=1e-8)
    alone, st = S.solve_reactive(f)
    S.close()
    assert st["rc"] == 0
    spec = dict(shape=shape, q=q, kappa=kappa, precision=prec, rtol=1e-8, kind=0)
    B = Batch([spec, spec])
    c = [torch.zeros_like(f), torch.zeros_like(f)]
    B.solve([f, f], c, [None, None])
    assert torch.equal(c[0], alone) and torch.equal(c[1], alone)
