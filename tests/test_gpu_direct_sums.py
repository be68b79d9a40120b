"""Dedispersion that reads every trial's samples where they are, at its edges: channels that
fill no group and no quarter, rows that end with the last sample read, trials and samples that
fill no tile, sums of many channels of the largest sample.  Whole numbers: every element of
the DM transform is the plain sum (tolerance 0)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27262_amd import spotlight
    return spotlight


# channels, trials, samples out, largest delay
EDGES = [(1, 1, 1, 0), (3, 2, 5, 3), (4, 16, 256, 1), (15, 17, 257, 700), (16, 5, 61, 1750), (17, 33, 511, 40),
         (67, 16, 769, 1700), (1030, 20, 300, 900), (4133, 3, 260, 1000)]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("nch,ndm,n_out,smax", EDGES)
def test_edges_equal_the_plain_sum(spl, nch, ndm, n_out, smax, mode):
    rng = np.random.default_rng(nch + n_out)
    D = rng.integers(0, smax + 1, size=(ndm, nch)).astype(np.int32)
    D[-1, -1] = smax   # the last channel's samples end the block
    p = spl.Plan(nch, 750.0, -0.05, 1e-3, n_out, widths=(1,), threshold=50.0, delays=D)
    n_in, n_dd = p.info["n_in"], p.info["n_dd"]
    pitch = (n_in + 15) // 16 * 16
    batch = spl.Batch([p, p], mode=mode)
    for b in range(2):
        batch.set_tiles(b, 4, 1)
    xs = [rng.integers(0, 256, size=(nch, pitch), dtype=np.uint8), np.full((nch, pitch), 255, np.uint8)]
    batch.run([torch.from_numpy(x).cuda() for x in xs], spl.new_candidates(1024))
    torch.cuda.synchronize()
    t = np.arange(n_dd)
    for b, x in enumerate(xs):
        want = np.stack([sum(x[c, D[d, c] + t].astype(np.int64) for c in range(nch)) for d in range(ndm)])
        got = batch.dm_transform(b)[:, :n_dd].cpu().numpy()
        assert np.array_equal(got, want), (b, np.argwhere(got != want)[:5])
