"""Batches that the static scratch of spl_batch_run_static takes: the largest hit capacities
whose workspace fitted its 64 MiB when the limit was documented stay within it."""
import pytest

from paper_2606_27262_amd import spotlight as spl
from paper_2606_27262_amd import workloads as W


@pytest.mark.parametrize("mode", [spl.MODE_PLAIN_PER_BEAM, spl.MODE_PERSISTENT_GRAPH])
@pytest.mark.parametrize("beams,hits", [(1, 1079733), (40, 994112), (200, 642816)])
def test_static_scratch_takes_what_it_took(beams, hits, mode):
    plan = spl.Plan.from_dict(W.make_plan(64, 550.0, 750.0, 1e-3, 1000, 0.0, 20.0, 32, (1, 4)))
    b = spl.Batch([plan] * beams, hit_capacity=hits, mode=mode)
    assert b.workspace_bytes() <= spl.STATIC_SCRATCH_BYTES
