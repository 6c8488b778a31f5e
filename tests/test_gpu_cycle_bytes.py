"""The bytes that blob_rd_time_kernel reports for a V-cycle are those of the launches it makes."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# Words a cell of a level, in its precision (a colour's array is half a word; coarse values 1/8):
# ten launches: three half-sweeps (the other colour, f, the own colour), red residual, restriction (coarse f and red u),
# red correction, four half-sweeps
PER_STEP = 3 * 1.5 + 2.0 + (0.5 + 0.125 + 0.0625) + (1.0 + 0.125) + 4 * 1.5
# two launches: f in, red and coarse f out; coarse u, red and f in, both colours out
TWO = (1.0 + 0.5 + 0.125) + (0.125 + 0.5 + 1.0 + 1.0)
# tiles: f in, red out; red and f in, coarse f out; red correction; red and f in, black out; closing red half-sweep
TILES = (1.0 + 0.5) + (0.5 + 1.0 + 0.125) + (1.0 + 0.125) + (0.5 + 1.0 + 0.5) + 1.5


@pytest.mark.parametrize("box", [False, True])
@pytest.mark.parametrize("shape,prec,routes", [
    ((64, 64, 64), 1, (TWO, TWO)),            # levels 64^3 and 32^3 above the tail at 16^3
    ((128, 128, 128), 1, (TILES, TWO, TWO)),
    ((64, 32, 128), 0, (TILES, TWO)),         # rows too long for two launches; the tail starts at 32 x 8 x 16
    ((16, 16, 16), 0, ()),                    # the whole cycle in the tail
])
def test_cycle_bytes(shape, prec, routes, box, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1306_3159_amd import BOUNDARY_DIRICHLET, BlobRD
    print("[case] V-cycle bytes", shape, prec, box, flush=True)
    dev = torch.device("cuda:0")
    n, e = shape[0] * shape[1] * shape[2], 4 if prec else 8
    kw = dict(boundary=BOUNDARY_DIRICHLET) if box else {}
    q = torch.tensor([[s / 2.0 for s in shape[::-1]]], dtype=torch.float64, device=dev)
    for blocked in ("1", "0"):
        monkeypatch.setenv("BLOB_RD_BLOCKED", blocked)
        S = BlobRD(shape, q, precision=prec, **kw)
        levels = routes if blocked == "1" else (PER_STEP,) * len(routes)
        # the entry reads the FP64 residual and writes f, and the first red sweep where a level-0 launch reads it:
        # the two-launch and tiled levels open from f
        entry = 8 + e * (1.0 if blocked == "1" and routes else 1.5)
        want = n * entry + sum(n / 8 ** l * e * w for l, w in enumerate(levels))
        for cold in (False, True):
            ms, got = S.time_kernel("vcycle", reps=3, cold=cold)
            assert ms > 0 and got == pytest.approx(want, rel=1e-12)
        S.close()
