"""Scoring from snippets at every alignment that a 16-bit tensor can have, and in passes that
the candidates do not fill: the same images through the same arithmetic; only the order of
the fully connected layer's partial sums may differ, which can reorder a near-tied pooling
window now and then (the bounds of the test of passes against a single pass)."""
import numpy as np
import pytest

from oracle import cnn
from test_gpu_ranker import _random_params, _random_snippets

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1, 2, 4])
@pytest.mark.parametrize("n", [1, 33, 70])
def test_alignment_and_ragged_passes(n, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27262_amd import spotlight as spl
    params = cnn.flatten_params(_random_params(5)).astype(np.float32)
    bits, _ = _random_snippets(np.random.default_rng(5), 70)
    all_ = torch.from_numpy(bits.view(np.int16)).cuda()
    whole = spl.Ranker(max_batch=96)
    whole.set_weights(params)
    want = whole.score(all_).cpu().numpy()[:n]
    flat = torch.empty(n * 2 * 64 * 256 + 8, dtype=torch.int16, device="cuda")
    snip = flat[offset:offset + n * 2 * 64 * 256].view(n, 2, 64, 256)
    snip.copy_(all_[:n])
    r = spl.Ranker(max_batch=32)
    r.set_weights(params)
    got = r.score(snip).cpu().numpy()
    scale = max(1.0, np.abs(want).max())
    d = np.abs(got - want)
    assert np.median(d) <= 1e-4 * scale and d.max() <= 2e-2 * scale
