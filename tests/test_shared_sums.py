"""The shared-row tables of the dedispersion on the CPU: the delays they encode, decoded
channel by channel, equal the plan's, and plans without shared patterns are not routed
to them."""
import numpy as np
import pytest

from paper_2606_27262_amd import spotlight as spl
from paper_2606_27262_amd import workloads as W


def band(nch, f_lo, f_hi, ndm, step, tsamp=1.31072e-3, n_out=2048, flip=False, dm0=0.0):
    p = W.make_plan(nch, f_lo, f_hi, tsamp, n_out, dm0, dm0 + step * ndm, ndm, (1, 4, 16))
    if flip:   # the lowest frequency first: the delays fall along the channels
        p["fch1"] += (nch - 1) * p["foff"]
        p["foff"] = -p["foff"]
    return spl.Plan.from_dict(p)


PLANS = {
    "band4": lambda: spl.Plan.from_dict(W.plan_c2()),
    "fine-steps": lambda: band(1024, 550.0, 750.0, 200, 0.25),
    "high-dm": lambda: band(512, 550.0, 750.0, 130, 0.5, dm0=900.0),
    "one-tile": lambda: band(256, 550.0, 750.0, 17, 0.5),
    "odd-channels": lambda: band(203, 550.0, 750.0, 65, 0.5),
    "sixteen-channels": lambda: band(16, 550.0, 750.0, 64, 0.25),
    "rising-band": lambda: band(333, 550.0, 750.0, 100, 0.5, flip=True),
    "band3": lambda: spl.Plan.from_dict(W.plan_band3_c4()),
}


@pytest.mark.parametrize("name", PLANS)
def test_tables_encode_the_plans_delays(name):
    plan = PLANS[name]()
    b = spl.Batch([plan], hit_capacity=1 << 16)
    tried = 0
    for dw, j in ((4, 2), (2, 2), (4, 1)):
        try:
            b.set_tiles(0, dw, j, 0, waves=16)
        except spl.SplError:
            continue
        got = b.shared_delays()
        if got is not None:
            tried += 1
            assert np.array_equal(got, plan.delays())
    b.set_tiles(0, 4, 1, 0, waves=4)
    assert b.shared_delays() is None   # other shapes stage single channels
    assert tried > 0 or name in ("sixteen-channels", "band3", "one-tile")


def test_arbitrary_delay_tables():
    """Delay tables of no physical form: whatever is shared encodes them exactly."""
    rng = np.random.default_rng(5)
    shared = 0
    for k in range(24):
        nch, ndm = int(rng.integers(1, 120)), int(rng.integers(1, 150))
        base = rng.integers(0, 200, nch)[None, :] + rng.integers(0, 40, ndm)[:, None]
        noise = rng.integers(0, (1, 2, 3, 6)[k % 4], (ndm, nch)) * (rng.random((ndm, 1)) < 0.2)
        d = (base + noise).astype(np.int32)
        plan = spl.Plan(nch, 750.0, -200.0 / nch, 1e-3, 600, widths=(1, 3), delays=d)
        b = spl.Batch([plan], hit_capacity=1 << 16)
        b.set_tiles(0, 4, 2, 0, waves=16)
        got = b.shared_delays()
        if got is not None:
            shared += 1
            assert np.array_equal(got, d), k
    assert shared >= 6


def steps_before_the_first(nch=64, ndm=64):
    """Delays whose channels would agree best on rows that start before the block: every
    other channel steps from 1 to 5 over the trials, the ones between from 0 to 1."""
    d = np.zeros((ndm, nch), np.int32)
    d[:, 1::2] = (1 + np.arange(ndm) * 5 // ndm)[:, None]
    d[:, 2::2] = (np.arange(ndm) * 2 // ndm)[:, None]
    return d


def test_no_row_starts_before_the_block():
    """(a start before a row would be an offset that wraps)"""
    d = steps_before_the_first()
    plan = spl.Plan(64, 750.0, -200.0 / 64, 1e-3, 1500, widths=(1,), delays=d)
    b = spl.Batch([plan], hit_capacity=1 << 16)
    b.set_tiles(0, 4, 2, 0, waves=16)
    got = b.shared_delays()
    assert got is not None and np.array_equal(got, d)


@pytest.mark.parametrize("nch,f_lo,f_hi,ndm,step", [
    (2048, 300.0, 500.0, 900, 0.5),      # rows of 1-2 KB for the 64-trial tiles
    (4096, 300.0, 500.0, 640, 0.25),
    (1024, 550.0, 750.0, 600, 2.0),
    (777, 300.0, 500.0, 333, 0.3)])
def test_default_tiles_take_every_plan(nch, f_lo, f_hi, ndm, step):
    """Whatever the rule for default tiles picks, the batch is made."""
    for n_out in (3000, 8192):
        plan = band(nch, f_lo, f_hi, ndm, step, n_out=n_out)
        b = spl.Batch([plan], hit_capacity=1 << 16)
        got = b.shared_delays()
        assert got is None or np.array_equal(got, plan.delays())


def test_default_tiles_of_an_uneven_table():
    """Delays shared by every channel but one, whose spread only row tiles of fewer trials take."""
    d = np.repeat(np.arange(640, dtype=np.int32)[:, None] // 8, 1000, axis=1)
    d[:, 501] = np.arange(640) * 14
    plan = spl.Plan(1000, 750.0, -0.2, 1e-3, 9000, widths=(1,), delays=d)
    spl.Batch([plan], hit_capacity=1 << 16)


def test_plans_without_shared_patterns_stage_single_channels():
    plan = spl.Plan.from_dict(W.plan_c1())   # 88 samples from trial to trial at the lowest channel
    b = spl.Batch([plan], hit_capacity=1 << 16)
    assert b.shared_delays() is None
    rng = np.random.default_rng(1)
    d = rng.integers(0, 60, (64, 64)).astype(np.int32)
    plan = spl.Plan(64, 750.0, -1.0, 1e-3, 600, widths=(1,), delays=d)
    b = spl.Batch([plan], hit_capacity=1 << 16)
    b.set_tiles(0, 4, 2, 0, waves=16)
    assert b.shared_delays() is None
