"""Plans whose shortest block row is longer than the shared-row dedispersion addresses are
tiled by row staging from the start."""
import numpy as np
import pytest

from paper_2606_27262_amd import spotlight as spl


@pytest.mark.parametrize("n_in,shared", [(5000, True), ((1 << 28) - 16, True), ((1 << 28) - 15, False), (1 << 28, False)])
def test_long_rows_are_staged(n_in, shared):
    d = np.repeat(np.arange(64, dtype=np.int32)[:, None], 32, axis=1)   # every channel alike
    plan = spl.Plan(32, 750.0, -1.0, 1e-3, n_in - 63, widths=(1,), delays=d)
    assert plan.info["n_in"] == n_in
    b = spl.Batch([plan], hit_capacity=1 << 16)
    b.set_tiles(0, 4, 2, 0, waves=16)
    got = b.shared_delays()
    assert (got is not None) == shared
    if shared:
        assert np.array_equal(got, d)
