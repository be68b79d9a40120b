"""The fine-DM plane on every route its kernel can take: channels in one slice or many
(uneven ones among them), windows of narrow and wide pulses and ones too wide for the LDS,
rows that reach past both ends of the block, and planes that are not word-aligned.  Bit for
bit against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2606_27262_amd import synth
from paper_2606_27262_amd import workloads as W
from plan_tables import oracle_plan

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("nch,copies", [(64, 1), (192, 1), (448, 1), (192, 400)])
def test_fine_plane_routes(nch, copies, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_27262_amd import spotlight as spl
    pd = W.make_plan(nch, 300.0, 500.0, 1.31072e-3, 900, 0.0, 60.0, 40, (1, 2, 4, 8))
    plan = spl.Plan.from_dict(pd)
    n_in, ndm, n_out = plan.info["n_in"], plan.info["ndm"], plan.info["n_out"]
    x = synth.make_block(W.block_spec(pd, n_in, [synth.Pulse(t0=300.0, dm=30.0, fwhm=3.0, snr=30.0)]), 5, 0,
                         pd["widths"])[:, :n_in]
    batch = spl.Batch([plan], hit_capacity=1 << 16)
    block = spl.upload_block(x)
    batch.run([block], spl.new_candidates(1 << 14))
    # the last of the seven names no pulse: zero planes; then windows of all alignments
    rng = np.random.default_rng(nch)
    recs = np.zeros(7 + 40, oracle.CAND_DTYPE)
    recs["dm_index"] = [20, 0, ndm - 1, 20, 20, 7, 20, *rng.integers(10, ndm, 40)]
    recs["t_sample"] = [300, 0, n_out - 1, 300, 500, 150, 300, *rng.integers(100, n_out - 100, 40)]
    recs["width"] = [1, 4, 8, 40, 400, 30000, 0, *rng.integers(1, 60, 40)]
    if copies > 1:
        recs = recs[:7]
    many = np.concatenate([recs] * copies)[: max(recs.size, copies)]
    dev = torch.from_numpy(many.view(np.int32).reshape(-1, 8).copy()).cuda()
    n = many.size
    flat = torch.full((n * 2 * 64 * 256 + 1,), 77, dtype=torch.int16, device="cuda")
    out = flat[offset:offset + n * 2 * 64 * 256].view(n, 2, 64, 256)
    spl.snippets(batch, dev, out=out, fine_keep=0.1)
    got = out.cpu().numpy().view(np.uint16)
    o = oracle_plan(plan)
    X0 = np.broadcast_to(np.int64(0), (o["D"].shape[0], o["n_dd"]))
    for i, r in enumerate(recs):
        if r["width"] < 1:
            want = np.zeros((2, 64, 256), np.uint16)
        else:
            want = np.stack([
                oracle.fine_dm_snippet(x, o["n_in"], pd["fch1"], pd["foff"], pd["tsamp"],
                                       float(o["dms"][int(r["dm_index"])]), int(r["width"]), int(r["t_sample"]), 0.1),
                oracle.snippets(x, o["D"], X0, o["n_out"], o["L"], int(r["dm_index"]), int(r["t_sample"]))[1]])
        for j in range(i, n, recs.size):
            assert np.array_equal(got[j], want), (i, j, r)
