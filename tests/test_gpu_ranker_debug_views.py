"""The ranker's debug views after a scoring pass that its candidates do not fill: the images past
them are zero images, whatever earlier passes left in the buffers."""
import numpy as np
import pytest

from oracle import cnn
from test_gpu_ranker import _random_params, _random_snippets

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("reweight", [False, True])
@pytest.mark.parametrize("n", [1, 31, 33, 63, 64 + 5])
def test_views_after_a_ragged_pass(n, reweight):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27262_amd import spotlight as spl
    nb = 64
    params = cnn.flatten_params(_random_params(11)).astype(np.float32)
    bits, _ = _random_snippets(np.random.default_rng(11), nb + 5)
    snip = torch.from_numpy(bits.view(np.int16)).cuda()
    r = spl.Ranker(max_batch=nb)
    r.set_weights(params)
    r.score(snip[:nb])                       # a full pass fills every image
    r.score(snip[:n])
    if reweight:                             # the views are of the pass, not of later weights
        r.set_weights(cnn.flatten_params(_random_params(12)).astype(np.float32))
    last = n % nb
    padded = torch.zeros((nb, 2, 64, 256), dtype=torch.int16, device="cuda")
    padded[:last] = snip[n - last:n]
    whole = spl.Ranker(max_batch=nb)
    whole.set_weights(params)
    whole.score(padded)
    torch.cuda.synchronize()
    for layer in range(4):
        assert torch.equal(r.pool_args(layer), whole.pool_args(layer)), layer
    # The products of FC1 are the same; the order in which the 64 partial sums of a value are
    # added may differ.  Each order errs by at most 64 * 2^-24 of the sum of magnitudes, and that
    # is bounded for a zero image by its activations (BF16: 2^-7 more at most, after four layers).
    p = cnn.unflatten_params(params.astype(np.float64))
    _, cache = cnn.forward(p, np.zeros((1, 2, 64, 256)))
    bound = 2 * 64 * 2.0 ** -24 * 1.1 * (np.abs(cache["f"]) @ np.abs(p["f1w"]).T).max()
    d = (r.fc_preact()[last:] - whole.fc_preact()[last:]).abs().max().item()
    print(f"n {n}: fc_preact of zero images differs by {d:.3g}, bound {bound:.3g}", flush=True)
    assert d <= bound
