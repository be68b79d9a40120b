"""Hit lists at the edges of their passes: rows of no, few (held one a lane) and many hits,
lists of no, one and many chunks, rows shorter than a block of the index, and a buffer that
the hits fill exactly.  Candidates bit for bit with the oracle's (tolerance 0)."""
import numpy as np
import pytest

from test_gpu_parity import _random_monotone_delays, compare, gpu_run, make_plan, oracle_run, spl  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n_out", [60, 64, 129, 4100])
@pytest.mark.parametrize("threshold", [0.5, 2.0, 3.3, 40.0])
def test_rows_and_chunks_of_every_size(spl, mode, n_out, threshold):  # noqa: F811
    rng = np.random.default_rng(n_out + mode)
    plans, blocks = [], []
    for ndm, stencils in ((37, ((1, 1), (5, 5))), (1, ((2, 70),)), (66, ((1, 1), (3, 64), (2, 2)))):
        D = _random_monotone_delays(rng, ndm, 9, 50)
        p = make_plan(spl, 9, ndm, n_out, (1, 4), threshold, delays=D, stencils=stencils)
        x = rng.integers(0, 256, size=(9, p.info["n_in"]), dtype=np.uint8)
        x[:, : x.shape[1] // 3] //= 4   # rows with hits bunched at one end
        plans.append(p)
        blocks.append(x)
    ref, rc = oracle_run(plans, blocks)
    n_hits = [r["hits"]["d"].size for r in ref]
    cap = max(1, max(n_hits) if mode == spl.MODE_PLAIN_PER_BEAM else sum(n_hits))   # a list a beam, or one
    g = gpu_run(spl, plans, blocks, mode=mode, hit_capacity=cap)
    compare(g, ref, rc)
