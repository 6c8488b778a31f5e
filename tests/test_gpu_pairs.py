"""Set-up of a placement where its kernels change form: pair rows within one wave's lanes, over
several registers a lane, and beyond them (sorted by one lane); tiles with more candidate blobs
than are staged at once; a scan of fewer and of more bins than threads."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import exact as ex
from oracle import learned as LN

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1306_3159_amd import native
    native.load_library()
    return torch.device("cuda:0")


# blobs drawn without separation: in 24^3 a row holds about half of them, 20, 160 and 580 entries
@pytest.mark.parametrize("n,N", [(24, 40), (24, 300), (24, 1100), (96, 200)])
def test_pairs_and_spread(dev, n, N):
    """Whole numbers of the pair list equal; the spread against the oracle's to rounding."""
    print("[case] pairs", n, N, flush=True)
    from paper_1306_3159_amd import BlobRD, Net
    rng = np.random.default_rng(31)
    q = rng.uniform(0.0, n, (N, 3))
    S = BlobRD(n, torch.as_tensor(q, device=dev))
    net = Net(dev)
    S.precond_build(net)
    ptr, col, _ = S.precond_csr()
    optr, ocol = LN.pair_list(LN.wrap_positions(q, n), n)
    assert np.array_equal(ptr.cpu().numpy(), optr) and np.array_equal(col.cpu().numpy(), ocol)
    lam = rng.standard_normal(N)
    got = S.spread(torch.as_tensor(lam, device=dev)).cpu().numpy()
    ref = ex.spread(lam, q, (n, n, n), 1.0, 4)
    assert np.max(np.abs(got - ref)) < 1e-13 * np.abs(ref).max()
    net.close()
    S.close()
