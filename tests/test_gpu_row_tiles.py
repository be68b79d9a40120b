"""The row-staging dedispersion kernels at sums past 256 channels, where their 16-bit fields are
moved on: every compiled shape with one and two LDS buffers and one and two vectors a staged
row, on delays that no two channels share (so that the 16-wavefront shapes stage rows too),
with samples of the largest value throughout.  Whole numbers: every element of the DM
transform is the plain sum (tolerance 0)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NCH, NDM, N_OUT = 515, 70, 1100   # two moves and three channels; trials and samples that fill no tile
NARROW = {(2, 2, 8, 1), (4, 2, 4, 1), (4, 1, 8, 1), (4, 2, 8, 1), (8, 1, 4, 1), (8, 1, 8, 1), (4, 1, 16, 1), (4, 2, 16, 1),
          (2, 2, 16, 1), (4, 1, 16, 2), (4, 2, 16, 2), (2, 2, 16, 2)}
WIDE = {(2, 2, 8, 1), (4, 1, 8, 1), (4, 2, 8, 1), (2, 2, 16, 1), (2, 2, 16, 2)}   # two vectors a row


@pytest.fixture(scope="module")
def spl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27262_amd import spotlight
    return spotlight


@pytest.mark.parametrize("spread,shapes", [(90, NARROW), (1200, WIDE)], ids=["rows-to-1K", "rows-to-2K"])
def test_row_staged_shapes_past_256_channels(spl, spread, shapes):
    rng = np.random.default_rng(spread)
    D = rng.integers(0, spread + 1, size=(NDM, NCH)).astype(np.int32)
    D[-1, -1] = spread
    plan = spl.Plan(NCH, 750.0, -0.3, 1e-3, N_OUT, widths=(1,), threshold=50.0, delays=D)
    n_in, n_dd = plan.info["n_in"], plan.info["n_dd"]
    pitch = (n_in + 15) // 16 * 16
    xs = [rng.integers(0, 256, size=(NCH, pitch), dtype=np.uint8), np.full((NCH, pitch), 255, np.uint8)]
    xs[0][rng.random(NCH) < 0.3] = 255
    blocks = [torch.from_numpy(x).cuda() for x in xs]
    want = [np.zeros((NDM, n_dd), np.int64) for _ in xs]
    for b, x in enumerate(xs):
        for d in range(NDM):
            for c in range(NCH):
                want[b][d] += x[c, D[d, c]:D[d, c] + n_dd]
    ran = set()
    for mode in (spl.MODE_PLAIN_PER_BEAM, spl.MODE_PERSISTENT_GRAPH):
        batch = spl.Batch([plan, plan], mode=mode, hit_capacity=1 << 16)
        cands = spl.new_candidates(1024)
        for dw, j, nw, nbuf in sorted(shapes):
            for chunk in (0, 2, 8):
                try:
                    batch.set_tiles(0, dw, j, chunk, waves=nw, buffers=nbuf)
                except spl.SplError:
                    continue   # (eight channels of long rows pass the LDS)
                assert batch.shared_delays() is None, "the plan is meant to have no rows to share"
                batch.run(blocks, cands)
                torch.cuda.synchronize()
                for b in range(2):
                    got = batch.dm_transform(b)[:, :n_dd].cpu().numpy()
                    assert np.array_equal(got, want[b]), (dw, j, nw, nbuf, chunk, mode, b)
                ran.add((dw, j, nw, nbuf))
    assert ran == shapes
