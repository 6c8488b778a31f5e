"""The loss of the learned preconditioner on short and on long pair lists: one launch a call, or its products
over the whole GPU."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _setup(n, N, samples, seed):
    import os
    import paper_1306_3159_amd as rd
    from paper_1306_3159_amd import BlobRD, Net
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(seed)
    weights = np.load(os.path.join(os.path.dirname(rd.__file__), "weights", "precond_rsa256.npy"))
    net = Net(dev)
    net.set_params(torch.as_tensor(weights.astype(np.float32).ravel()))
    S = BlobRD(n, torch.as_tensor(rng.random((N, 3)) * n, device=dev), precision=1)
    nnz = S.precond_build(net)
    X = rng.standard_normal((samples, N))
    Y = rng.standard_normal((samples, N))
    net.zero_grad()
    return net, S, nnz, X - X.mean(1, keepdims=True), Y


@pytest.mark.parametrize("N,samples,short", [(1, 1, True), (700, 3, True), (1100, 3, False), (4000, 8, False)])
def test_loss_of_both_forms(N, samples, short):
    """Mean over the samples of |P W P y - x|^2 / |x|^2 in FP64 from W's own entries (some ten thousand of them):
    1e-12."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] loss", N, samples, flush=True)
    net, S, nnz, X, Y = _setup(96, N, samples, 61)
    assert (nnz <= 1 << 13) == short
    if N == 1:
        X = X + 1.0  # one blob: P y = 0, the loss is 1
    dev = torch.device("cuda:0")
    got = S.precond_loss_grad(net, torch.as_tensor(X, device=dev), torch.as_tensor(Y, device=dev))
    ptr, col, val = (v.cpu().numpy() for v in S.precond_csr())
    rows = np.repeat(np.arange(N), np.diff(ptr))
    want = 0.0
    for x, y in zip(X, Y):
        w = np.bincount(rows, val * (y - y.mean())[col], minlength=N)
        want += np.sum((w - w.mean() - x) ** 2) / np.sum(x ** 2) / samples
    assert got == pytest.approx(want, rel=1e-12)
    S.close()


def test_one_sample_of_a_dense_suspension():
    """One sample's loss and gradient over a long pair list (1.4 10^6 entries) takes less than 1.5 times the
    building of W from that list: 0.7 with the products over the whole GPU, 3 in one work-group."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] loss of a dense suspension", flush=True)
    net, S, nnz, X, Y = _setup(128, 20000, 1, 67)
    assert nnz > 10 ** 6
    dev = torch.device("cuda:0")
    X, Y = torch.as_tensor(X, device=dev), torch.as_tensor(Y, device=dev)

    def median(call):
        t = []
        for _ in range(9):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            call()
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return sorted(t)[4]

    loss, build = median(lambda: S.precond_loss_grad(net, X, Y)), median(lambda: S.precond_build(net))
    assert loss < 1.5 * build, (loss, build)
    S.close()
