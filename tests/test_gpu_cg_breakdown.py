"""A CG solve that breaks down: it fails with an error, and later solves on the handle are as before it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,blobs", [(32, 1), (64, 64), (64, 2049)])
def test_breakdown_ends_the_solve(n, blobs):
    """A right-hand side beyond the range of the FP32 V-cycle makes z, and so beta, non-finite before the first
    step (the direction's launch finds it up to 512 blocks): the solve fails, alone and in a batch, and the
    handle then gives the same bits as before."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1306_3159_amd import Batch, BlobRD, BlobRDError
    print("[case] CG breakdown", n, blobs, flush=True)
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(11)
    shape = (n, n, n)
    f = torch.as_tensor(1.0 + 0.5 * rng.standard_normal(shape), device=dev)
    q = torch.as_tensor(rng.uniform(0.0, n, (blobs, 3)), device=dev)
    kappa = torch.as_tensor(rng.uniform(0.5, 2.0, blobs), device=dev)
    S = BlobRD(shape, q, kappa, precision=1, rtol=1e-8)
    before, st = S.solve_reactive(f)
    assert st["rc"] == 0
    for _ in range(2):
        with pytest.raises(BlobRDError):
            S.solve_reactive(f * 1e60)
        after, st = S.solve_reactive(f)
        assert st["rc"] == 0 and torch.equal(after, before)
    S.close()
    spec = dict(shape=shape, q=q, kappa=kappa, precision=1, rtol=1e-8, kind=0)
    B = Batch([spec])
    with pytest.raises(BlobRDError):
        B.solve([f * 1e60], [torch.zeros_like(f)], [None])
