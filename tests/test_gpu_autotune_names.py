"""The autotuner's choices: the shared-row kernel is timed, and cached, under the name that the
defaults give it, whatever the plan's spread; a choice cached for earlier kernels is not taken."""
import numpy as np
import pytest

from paper_2606_27262_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spl():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27262_amd import spotlight
    return spotlight


def band(spl):
    return spl.Plan.from_dict(W.make_plan(4096, 550.0, 750.0, 1.31072e-3, 8192, 0.0, 512.0, 1024, (1, 4)))


def uneven(spl):
    """Delays that all channels share but one, whose spread makes rows of 1.3 KB in 32-trial row
    tiles: 32 channels of such rows pass the LDS, 16 do not."""
    d = np.repeat(np.arange(640, dtype=np.int32)[:, None] // 8, 1000, axis=1)
    d[:, 501] = np.arange(640) * 25
    return spl.Plan(1000, 750.0, -0.2, 1e-3, 9000, widths=(1, 4), delays=d)


@pytest.mark.parametrize("make", [band, uneven])
def test_one_name_for_shared_rows(spl, tmp_path, make):
    plan = make(spl)
    first = spl.Batch([plan], hit_capacity=1 << 20)
    assert first.shared_delays() is not None, "the default of this plan is meant to be shared rows"
    block = torch.randint(0, 256, (plan.info["nchans"], (plan.info["n_in"] + 15) // 16 * 16), dtype=torch.uint8, device="cuda")
    cache = tmp_path / "tiles.txt"
    tuned = spl.Batch([plan], hit_capacity=1 << 20)
    tiles = tuned.autotune([block], cache_path=str(cache))[0]
    # (several times as fast as every row-staged shape here)
    assert tuned.shared_delays() is not None and tiles == first.tiles(0)
    sig, *fields = cache.read_text().split()
    # the line of a library whose shapes all staged rows: no kernel tag
    old = tmp_path / "old.txt"
    bare = sig.rsplit("-", 1)[0]
    old.write_text(f"{bare} 2 2 8 1 16 0.001\n")
    again = spl.Batch([plan], hit_capacity=1 << 20)
    assert again.autotune([block], cache_path=str(old))[0] == tiles
    lines = [line.split() for line in old.read_text().splitlines()]
    assert [line[0] for line in lines] == [bare, sig] and lines[1][1:6] == fields[:5]
