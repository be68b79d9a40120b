"""Scoring the same images from tensors of every 16-bit alignment and in passes that they do not
fill: the convolutions add each value in one fixed order, so every pooling decision is the same,
bit for bit; only the order in which FC1's 64 partial sums are added may differ."""
import numpy as np
import pytest

from oracle import cnn
from test_gpu_ranker import _random_params, _random_snippets

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 70


@pytest.fixture(scope="module")
def images():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    params = cnn.flatten_params(_random_params(5)).astype(np.float32)
    bits, x = _random_snippets(np.random.default_rng(5), N)
    p = cnn.unflatten_params(params.astype(np.float64))
    _, cache = cnn.forward(p, x)
    # An order of 64 additions errs by at most 64 * 2^-24 of the sum of the magnitudes (a tenth
    # more for the BF16 activations); two orders differ by twice that.  The output layer passes
    # that on, and adds its own 65 terms in one order, whose roundings follow their operands.
    h = 2 * 64 * 2.0 ** -24 * 1.1 * (np.abs(cache["f"]) @ np.abs(p["f1w"]).T)
    out = np.abs(p["f2w"][0])
    bound = h @ out + 65 * 2.0 ** -23 * 1.1 * (np.abs(cache["hr"]) @ out + abs(p["f2b"][0]))
    return params, torch.from_numpy(bits.view(np.int16)).cuda(), bound


@pytest.mark.parametrize("offset", [0, 1, 2, 3, 5])
@pytest.mark.parametrize("n", [1, 33, 70])
def test_decisions_are_the_same_bits(images, n, offset):
    from paper_2606_27262_amd import spotlight as spl
    params, all_, bound = images
    whole = spl.Ranker(max_batch=96)
    whole.set_weights(params)
    want = whole.score(all_).cpu().numpy()[:n]
    flat = torch.empty(n * 2 * 64 * 256 + 8, dtype=torch.int16, device="cuda")
    snip = flat[offset:offset + n * 2 * 64 * 256].view(n, 2, 64, 256)
    snip.copy_(all_[:n])
    for max_batch in (96, 32):
        r = spl.Ranker(max_batch=max_batch)
        r.set_weights(params)
        got = r.score(snip).cpu().numpy()
        first = (n - 1) // max_batch * max_batch   # of the last pass
        for layer in range(4):
            a, b = r.pool_args(layer)[:n - first], whole.pool_args(layer)[first:n]
            assert torch.equal(a, b), (max_batch, layer, int((a != b).sum()))
        d = np.abs(got.astype(np.float64) - want)
        print(f"n {n} offset {offset} passes of {max_batch}: max |diff| {d.max():.3g}, of the bound {np.max(d / bound[:n]):.3g}",
              flush=True)
        assert np.all(d <= bound[:n])
