"""Blocks whose rows lie 256 MiB or more apart, which the shared-row dedispersion does not
address: searched by another kernel in the same launch sequence, whatever is under way, with
the tables left for the next block.  Whole numbers (tolerance 0)."""
import numpy as np
import pytest

from paper_2606_27262_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NCH, WIDE = 24, 1 << 28


@pytest.fixture(scope="module")
def spl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27262_amd import spotlight
    return spotlight


@pytest.fixture(scope="module")
def wide(spl):
    """Device memory of one block of wide rows (6 GiB; only the rows' starts are written)."""
    return torch.empty((NCH, WIDE), dtype=torch.uint8, device="cuda")


def transform(x, plan):
    D, n_dd = plan.delays(), plan.info["n_dd"]
    want = np.zeros((plan.info["ndm"], n_dd), np.int64)
    for d in range(want.shape[0]):
        for c in range(x.shape[0]):
            want[d] += x[c, D[d, c]:D[d, c] + n_dd]
    return want


@pytest.mark.parametrize("mode", [0, 1])
def test_wide_rows_between_short_ones(spl, wide, mode):
    # 70 trials and 1,101 samples: the last tiles are not full
    plan = spl.Plan.from_dict(W.make_plan(NCH, 1100.0, 1300.0, 1.31072e-3, 1100, 0.0, 17.5, 70, (1, 2)))
    n_in = plan.info["n_in"]
    rng = np.random.default_rng(3)
    xs = [rng.integers(0, 256, size=(NCH, n_in), dtype=np.uint8) for _ in range(3)]
    pitch = (n_in + 15) // 16 * 16
    short = [spl.upload_block(x, pitch=pitch) for x in xs]
    wide[:, :n_in].copy_(torch.from_numpy(xs[1]))
    batch = spl.Batch([plan, plan], mode=mode, hit_capacity=1 << 20)
    batch.set_tiles(0, 4, 2, 0, waves=16)
    tables = batch.shared_delays()
    assert tables is not None, "the plan is meant to share its rows"
    # eight searches enqueued one behind the other, nothing waited for between them
    blocks = [[short[0], short[2]], [short[0], wide], [wide, short[2]], [short[2], short[0]]] * 2
    which = [(0, 2), (0, 1), (1, 2), (2, 0)] * 2
    stream = torch.cuda.Stream()
    got = []
    cands, stats = spl.new_candidates(1 << 12), torch.zeros(spl.STATS_WORDS, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for b in blocks:
            batch.run(b, cands, stats)
            got.append([batch.dm_transform(k)[:, :plan.info["n_dd"]].clone() for k in range(2)])
    torch.cuda.synchronize()
    want = [transform(x, plan) for x in xs]
    for r, pair in enumerate(which):
        for k in range(2):
            assert np.array_equal(got[r][k].cpu().numpy(), want[pair[k]]), (r, k)
    again = batch.shared_delays()
    assert again is not None and np.array_equal(again, plan.delays())


def test_wide_rows_without_allocation(spl, wide):
    """The static-scratch run on wide rows, between runs of the batch's own workspace."""
    plan = spl.Plan.from_dict(W.make_plan(NCH, 1100.0, 1300.0, 1.31072e-3, 1100, 0.0, 17.5, 70, (1, 2), threshold=3.5))
    n_in = plan.info["n_in"]
    x = np.random.default_rng(4).integers(0, 256, size=(NCH, n_in), dtype=np.uint8)
    short = spl.upload_block(x, pitch=(n_in + 15) // 16 * 16)
    wide[:, :n_in].copy_(torch.from_numpy(x))
    batch = spl.Batch([plan], hit_capacity=1 << 16)
    batch.set_tiles(0, 4, 2, 0, waves=16)
    assert batch.shared_delays() is not None
    out = []
    for run, block in ((batch.run, short), (batch.run_static, wide), (batch.run, short)):
        stats = torch.zeros(spl.STATS_WORDS, dtype=torch.int64, device="cuda")
        cands, stats = run([block], spl.new_candidates(1 << 14), stats)
        torch.cuda.synchronize()
        out.append(spl.candidates_to_numpy(cands, stats))
    assert out[0].size > 0
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])


def test_autotuner_takes_wide_rows(spl, wide, tmp_path):
    plan = spl.Plan.from_dict(W.make_plan(NCH, 1100.0, 1300.0, 1.31072e-3, 1100, 0.0, 17.5, 70, (1, 2)))
    n_in = plan.info["n_in"]
    x = np.random.default_rng(5).integers(0, 256, size=(NCH, n_in), dtype=np.uint8)
    wide[:, :n_in].copy_(torch.from_numpy(x))
    batch = spl.Batch([plan], hit_capacity=1 << 16)
    batch.autotune([wide], cache_path=str(tmp_path / "tiles.txt"))
    batch.run([wide], spl.new_candidates(1 << 12))
    torch.cuda.synchronize()
    assert np.array_equal(batch.dm_transform(0)[:, :plan.info["n_dd"]].cpu().numpy(), transform(x, plan))
