"""The shared-row dedispersion kernel at the edges of its tiles: trials, samples and channels
that fill no tile, rows staged in one to many items, blocks whose rows end with the last
sample read.  Whole numbers, so every element of the DM transform is the plain sum (tolerance
0)."""
import numpy as np
import pytest

from paper_2606_27262_amd import workloads as W
from test_shared_sums import steps_before_the_first

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27262_amd import spotlight
    return spotlight


# channels, band, trials, DM step, samples out, first DM, rising frequency
EDGES = {
    "one-trial-tile": (256, 550.0, 750.0, 64, 0.25, 1024, 0.0, False),
    "one-sample-over": (65, 550.0, 750.0, 65, 0.5, 1025, 0.0, False),
    "short-block": (203, 550.0, 750.0, 70, 0.5, 61, 0.0, False),
    "one-run": (16, 1100.0, 1300.0, 64, 0.25, 1500, 0.0, False),
    "last-run-overlaps": (333, 550.0, 750.0, 129, 0.25, 2047, 40.0, False),
    "rising-band": (333, 550.0, 750.0, 100, 0.5, 3000, 0.0, True),
    "carry-of-high-bytes": (1111, 1100.0, 1300.0, 66, 0.1, 1100, 10.0, False),
    "wide-rows": (2048, 550.0, 750.0, 70, 1.5, 1030, 0.0, False),
}


@pytest.mark.parametrize("name", EDGES)
def test_edges_equal_the_plain_sum(spl, name):
    nch, lo, hi, ndm, step, n_out, dm0, flip = EDGES[name]
    p = W.make_plan(nch, lo, hi, 1.31072e-3, n_out, dm0, dm0 + step * ndm, ndm, (1, 4))
    if flip:
        p["fch1"], p["foff"] = p["fch1"] + (nch - 1) * p["foff"], -p["foff"]
    check(spl, spl.Plan.from_dict(p))


def test_no_row_starts_before_the_block(spl):
    """Channels that would agree best on rows starting before the block's first sample."""
    check(spl, spl.Plan(64, 750.0, -200.0 / 64, 1e-3, 1500, widths=(1,), delays=steps_before_the_first()))


def check(spl, plan):
    nch, ndm = plan.info["nchans"], plan.info["ndm"]
    batch = spl.Batch([plan], hit_capacity=1 << 20)
    for dw, j in ((4, 2), (2, 2), (4, 1)):
        try:
            batch.set_tiles(0, dw, j, 0, waves=16)
            break
        except spl.SplError:
            continue
    assert batch.shared_delays() is not None, "the plan is meant to share its rows"
    n_in, n_dd = plan.info["n_in"], plan.info["n_dd"]
    rng = np.random.default_rng(nch)
    x = rng.integers(0, 256, size=(nch, n_in), dtype=np.uint8)
    x[rng.random(nch) < 0.3] = 255   # whole channels at the largest byte
    block = spl.upload_block(x, pitch=(n_in + 15) // 16 * 16)
    cands, stats = batch.run([block], spl.new_candidates(1 << 18))
    torch.cuda.synchronize()
    got = batch.dm_transform(0)[:, :n_dd].cpu().numpy()
    D = plan.delays()
    want = np.zeros((ndm, n_dd), np.int64)
    for d in range(ndm):
        for c in range(nch):
            want[d] += x[c, D[d, c]:D[d, c] + n_dd]
    assert np.array_equal(got, want)
