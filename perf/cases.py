"""The work a user of this framework has it do, as cases that can be timed.

`listed()` names the cases, `draw(rng)` gives one more of the same ranges, `prepare`
makes what a program holds before the call (blocks on the GPU, plans, batches, ranker
weights), `run` makes one pass through the public entry points, `work` states the bytes
and operations of one pass and `exact` the float64 values of the ranker's outputs.

Seven kinds of work, all of them steps of the real-time search:
  search     one block of every beam: dedispersion, normaliser, boxcars, peak filters
  turn       a block that arrives time-major, turned to channel-major rows
  assemble   the next block of a continuous stream from the last one and the new samples
  snippets   the classifier's two feature planes of the candidates of a search
  score      logits of candidates
  train      one training step of the ranker
  inject     bursts added to a block that is already quantised
"""
import math
import os

import numpy as np
import torch
import torch.nn.functional as F

import paper_2606_27262_amd as _pkg
from paper_2606_27262_amd import spotlight as spl
from paper_2606_27262_amd import synth
from paper_2606_27262_amd import workloads as W

DEVICE = "cuda"
BANDS = {3: (300.0, 500.0), 4: (550.0, 750.0)}   # MHz
WIDTHS = (1, 2, 4, 8, 16, 32, 64, 128, 256)
ALT = {"band": 3, "nch": 2048, "n_out": 32768, "tsamp": 0.65536e-3, "dm_step": 1000.0 / 1024, "trials": 1024}


def listed():
    c2 = {"kind": "search", "band": 4, "nch": 4096, "n_out": 16384, "tsamp": 1.31072e-3, "dm_step": 2000.0 / 2048,
          "trials": 2048, "w_max": 256, "segments": 1, "pulses": 10, "rfi": True, "zero_dm": 0.0, "mixed": False,
          "hit_cap": 0, "cand_cap": 1 << 16}
    return [
        # the smallest search: one coarse beam, where launches and latency count
        {**c2, "name": "search-1x256ch", "band": 3, "nch": 256, "n_out": 8192, "dm_step": 500.0 / 128, "trials": 128,
         "w_max": 64, "pulses": 1, "rfi": False, "beams": 1, "graph": False},
        # one beam at full resolution, searched by itself as its block arrives
        {**c2, "name": "search-1x4096ch", "beams": 1, "graph": False, "pulses": 20},
        # one GPU's share of the beams of the telescope, one graph launch per block
        {**c2, "name": "search-24x4096ch", "beams": 24, "graph": True, "cand_cap": 1 << 20},
        # beams of both bands in one batch, with broad-band interference: dense hit lists
        {**c2, "name": "search-4-uneven", "dm_step": 3000.0 / 3072, "trials": 3072, "beams": 4, "graph": True,
         "mixed": True, "zero_dm": 0.2, "hit_cap": 1 << 26, "cand_cap": 1 << 19},
        # a block from a recorder that writes spectra one after another
        {"name": "turn-4096x26305", "kind": "turn", "nch": 4096, "n_t": 26305},
        # a block of a continuous stream: 9921 samples of overlap and 16384 new ones
        {"name": "assemble-4096x26305", "kind": "assemble", "nch": 4096, "n_out": 16384, "carry": 9921},
        # the candidates of a few beams made into the classifier's input
        {**c2, "name": "snippets-256", "kind": "snippets", "beams": 1, "graph": False, "n": 256, "fine": False},
        # the same with the DM-time plane on a narrow DM range around each candidate
        {**c2, "name": "snippets-fine-256", "kind": "snippets", "beams": 1, "graph": False, "n": 256, "fine": True},
        # a quiet block's candidates scored, and those of 24 beams (a ragged last pass)
        {"name": "score-24", "kind": "score", "n": 24, "max_batch": 32},
        {"name": "score-1677", "kind": "score", "n": 1677, "max_batch": 256},
        # one step of training the ranker
        {"name": "train-256", "kind": "train", "n": 256, "max_batch": 256},
        # ten test bursts injected into a beam's block while it is searched
        {"name": "inject-10x4096ch", "kind": "inject", "band": 4, "nch": 4096, "n_out": 16384, "tsamp": 1.31072e-3,
         "bursts": 10, "argmax": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("search", "search", "search", "search", "turn", "assemble", "snippets", "snippets", "score",
                       "train", "inject"))
    if kind == "turn":
        return {"kind": kind, "nch": 16 * _log(rng, 8, 256), "n_t": _log(rng, 1024, 48000)}
    if kind == "assemble":
        return {"kind": kind, "nch": _log(rng, 100, 4096), "n_out": 16 * _log(rng, 128, 2048),
                "carry": _log(rng, 500, 12000)}
    if kind == "score":
        return {"kind": kind, "n": _log(rng, 1, 2000), "max_batch": rng.choice((32, 96, 256, 512))}
    if kind == "train":
        m = rng.choice((64, 128, 256))
        return {"kind": kind, "n": rng.choice((m, m, rng.randint(m // 2, m))), "max_batch": m}
    band = rng.choice((3, 4, 4))
    if kind == "inject":
        return {"kind": kind, "band": band, "nch": _log(rng, 200, 4096), "n_out": _log(rng, 2048, 20000),
                "tsamp": rng.choice((0.65536e-3, 1.31072e-3)), "bursts": rng.randint(1, 12),
                "argmax": rng.random() < 0.3}
    c = {"kind": kind, "band": band, "w_max": rng.choice((16, 64, 256)), "segments": rng.choice((1, 1, 1, 3)),
         "pulses": rng.randint(1, 12), "rfi": rng.random() < 0.7, "zero_dm": 0.0, "mixed": False, "hit_cap": 0,
         "cand_cap": 1 << 17, "tsamp": rng.choice((0.65536e-3, 1.31072e-3))}
    c["dm_step"] = rng.choice((0.25, 0.5, 250.0 / 256, 1.0)) * (2.0 if band == 4 and rng.random() < 0.3 else 1.0)
    if kind == "snippets":
        c.update(nch=64 * _log(rng, 8, 64), n_out=_log(rng, 4096, 16384), trials=_log(rng, 300, 1200), beams=1,
                 graph=False, n=_log(rng, 8, 300), fine=rng.random() < 0.5)
        return c
    c.update(nch=_log(rng, 64, 4096), n_out=_log(rng, 2048, 32768), trials=_log(rng, 64, 3072),
             beams=rng.choice((1, 1, 2, 5, 12)))
    while c["beams"] * c["nch"] * c["n_out"] * c["trials"] > 8e11:
        c["trials"] = max(64, c["trials"] // 2 + 1)
        c["beams"] = max(1, c["beams"] // 2)
    c["graph"] = c["beams"] > 1 or rng.random() < 0.5
    return c


def _plan_dict(c, alt=False):
    q = ALT if alt else c
    fch1, foff = synth.band_edges(q["nch"], *BANDS[q["band"]])
    return dict(nchans=q["nch"], fch1=fch1, foff=foff, tsamp=q["tsamp"], n_out=q["n_out"],
                norm_window=-(-q["n_out"] // c["segments"]), dm_ranges=[(0.0, q["dm_step"], q["trials"])],
                widths=tuple(w for w in WIDTHS if w <= c["w_max"]), threshold=6.0)


def _plan_dicts(c):
    """One plan per beam; beams of the same band share the dict."""
    a = _plan_dict(c)
    b = _plan_dict(c, True) if c["mixed"] else a
    return [a if k % 2 == 0 else b for k in range(c["beams"])]


def _search_state(c, seed):
    pds = _plan_dicts(c)
    made = {id(pd): spl.Plan.from_dict(pd) for pd in pds}
    plans = [made[id(pd)] for pd in pds]
    blocks = []
    for k, (pd, p) in enumerate(zip(pds, plans)):
        blocks.append(W.c2_like_block_torch(pd, p.info["n_in"], seed, k, c["pulses"],
                                            dm_max_pulse=max(60.0, 0.9 * W.dm_max(pd)),
                                            rfi_frac=0.02 if c["rfi"] else 0.0, zero_dm_rate=c["zero_dm"],
                                            device=DEVICE)[1])
    batch = spl.Batch(plans, mode=spl.MODE_PERSISTENT_GRAPH if c["graph"] else spl.MODE_PLAIN_PER_BEAM,
                      hit_capacity=c["hit_cap"])
    batch.attach()
    cands = torch.zeros((c["cand_cap"], 8), dtype=torch.int32, device=DEVICE)
    stats = torch.zeros(spl.STATS_WORDS, dtype=torch.int64, device=DEVICE)
    return {"batch": batch, "blocks": blocks, "cands": cands, "stats": stats}


def _images(n, g):
    """BF16 bit patterns of n snippets: standardised noise, every other one with a pulse
    that falls off across DM (plane 0) and spans the band (plane 1)."""
    v = torch.randn((n, 2, 64, 256), generator=g, device=DEVICE)
    row = torch.arange(64, device=DEVICE)[:, None] - 32.0
    col = torch.arange(256, device=DEVICE)[None, :] - 128.0
    width = torch.exp(torch.rand((n, 1, 1), generator=g, device=DEVICE) * 3.0)
    amp = (4.0 + 16.0 * torch.rand((n, 1, 1), generator=g, device=DEVICE)) * (torch.arange(n, device=DEVICE) % 2 == 0
                                                                            ).view(n, 1, 1)
    spread = torch.sqrt(width ** 2 + (0.5 * row) ** 2)
    v[:, 0] += amp * width / spread * torch.exp(-0.5 * (col / spread) ** 2)
    v[:, 1] += 0.3 * amp * torch.exp(-0.5 * (col / width) ** 2)
    return v.to(torch.bfloat16).view(torch.int16)


def _generator(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed) * 2654435761 % (1 << 62))
    return g


def _weights():
    return np.load(os.path.join(os.path.dirname(_pkg.__file__), "data", "ranker_weights.npy"), allow_pickle=False)


def _ranker_inputs(c, seed):
    g = _generator(seed)
    snip = _images(c["n"], g)
    return snip, (torch.arange(c["n"], device=DEVICE) % 2 == 0).to(torch.float32)


def prepare(case, seed):
    c = case
    k = c["kind"]
    if k == "search":
        return {"kind": k, **_search_state(c, seed)}
    if k == "snippets":
        s = _search_state(c, seed)
        s["batch"].run(s["blocks"], s["cands"], s["stats"])
        found = min(int(s["stats"][1].item()), c["cand_cap"])
        at = torch.arange(c["n"], device=DEVICE) * max(1, found) // c["n"]
        s.update(kind=k, picked=s["cands"][at].contiguous(), fine=0.1 if c["fine"] else None,
                 planes=torch.empty((c["n"], 2, 64, 256), dtype=torch.int16, device=DEVICE))
        return s
    if k in ("score", "train"):
        snip, labels = _ranker_inputs(c, seed)
        r = spl.Ranker(max_batch=c["max_batch"], device=DEVICE)
        r.set_weights(_weights())
        return {"kind": k, "ranker": r, "snip": snip, "labels": labels}
    g = _generator(seed)
    if k == "turn":
        return {"kind": k, "out": None,
                "x": torch.randint(0, 256, (c["n_t"], c["nch"]), generator=g, device=DEVICE, dtype=torch.uint8)}
    if k == "assemble":
        n_in = c["n_out"] + c["carry"]
        pitch = -(-n_in // 256) * 256
        prev = torch.randint(0, 256, (c["nch"], pitch), generator=g, device=DEVICE, dtype=torch.uint8)
        stage = spl.new_stage(c["nch"], c["n_out"], device=DEVICE)
        stage.copy_(torch.randint(0, 256, stage.shape, generator=g, device=DEVICE, dtype=torch.uint8))
        return {"kind": k, "prev": prev, "stage": stage, "next": torch.zeros_like(prev), "n_out": c["n_out"],
                "n_in": n_in}
    fch1, foff = synth.band_edges(c["nch"], *BANDS[c["band"]])
    pd = dict(nchans=c["nch"], fch1=fch1, foff=foff, tsamp=c["tsamp"])
    spec = W.block_spec(pd, c["n_out"])
    rng = np.random.default_rng([int(seed), 77])
    # later bursts have larger DMs and none is wider than its slot: no two meet in a channel
    widest = max(2.0, min(32.0, c["n_out"] / (c["bursts"] + 1) / 12.0))
    bursts = synth.pulses_evenly(rng, c["bursts"], c["n_out"], 50.0, 500.0, 1.0, widest, 8.0, 50.0)
    bursts = [synth.Pulse(t0=b.t0, dm=dm, fwhm=b.fwhm, snr=b.snr)
              for b, dm in zip(bursts, sorted(b.dm for b in bursts))]
    t_start, signal = synth.burst_windows(spec, bursts)
    clean = synth.make_block_torch(spec, seed, 0, device=DEVICE)
    words = torch.randint(-(1 << 31), 1 << 31, signal.shape, generator=g, device=DEVICE, dtype=torch.int64)
    return {"kind": k, "clean": clean, "block": torch.zeros_like(clean), "n_t": c["n_out"],
            "t_start": torch.from_numpy(t_start).to(DEVICE), "signal": torch.from_numpy(signal).to(DEVICE),
            "words": words.to(torch.int32), "mode": spl.INJECT_ARGMAX if c["argmax"] else spl.INJECT_SAMPLE}


def run(s):
    k = s["kind"]
    if k == "search":
        cands, stats = s["batch"].run(s["blocks"], s["cands"], s["stats"])
        # the DM transforms stay readable for the candidates' snippets
        return {"cands": cands, "stats": stats, "transforms": [
            s["batch"].dm_transform(b)[:, :p.info["n_dd"]] for b, p in enumerate(s["batch"].plans)]}
    if k == "snippets":
        return spl.snippets(s["batch"], s["picked"], out=s["planes"], fine_keep=s["fine"])
    if k == "score":
        return s["ranker"].score(s["snip"])
    if k == "train":
        loss = s["ranker"].train_step(s["snip"], s["labels"], 1e-3)
        return {"loss": loss, "grads": s["ranker"].grads()}
    if k == "turn":
        out = spl.corner_turn(s["x"], out=s["out"])
        s["out"] = out
        return out[:, :s["x"].shape[0]]
    if k == "assemble":
        spl.stream_assemble(s["next"], s["prev"], s["stage"], s["n_out"], s["n_in"])
        return s["next"]
    s["block"].copy_(s["clean"])   # the block as it arrives: every pass injects into a fresh one
    return spl.inject_quantised(s["block"], s["t_start"], s["signal"], s["words"], mode=s["mode"], n_t=s["n_t"])


def _max_delay(pd):
    f_ref, f_low = pd["fch1"], pd["fch1"] + (pd["nchans"] - 1) * pd["foff"]
    start, step, n = pd["dm_ranges"][-1]
    return int(round(4148.8064239 * (start + step * (n - 1)) * (1.0 / f_low ** 2 - 1.0 / f_ref ** 2) / pd["tsamp"]))


# floating-point operations of one candidate's forward pass (four convolutions and the head)
_FORWARD = 2.0 * (64 * 256 * 32 * 18 + (32 * 128 + 16 * 64 + 8 * 32) * 32 * 288 + 2048 * 64 + 64)
_PLANES = 2 * 64 * 256 * 2


def work(case):
    """Bytes that have to be read and written once, and operations: the additions of the
    definition for sums over channels, multiplications and additions for the ranker."""
    c = case
    k = c["kind"]
    if k == "search":
        nbytes = adds = 0.0
        for pd in _plan_dicts(c):
            trials = pd["dm_ranges"][0][2]
            n_dd = pd["n_out"] + max(pd["widths"]) - 1
            nbytes += pd["nchans"] * (n_dd + _max_delay(pd)) + 4.0 * trials * n_dd   # the block; the DM transform
            adds += float(trials) * pd["nchans"] * pd["n_out"]
        return {"bytes": nbytes, "flops": adds}
    if k == "snippets":
        rows = 64.0 if c["fine"] else 1.0   # rows of sums over all channels
        return {"bytes": c["n"] * (c["nch"] * 256.0 + 64 * 256 * 4 + _PLANES),
                "flops": c["n"] * rows * c["nch"] * 256.0}
    if k == "score":
        return {"bytes": c["n"] * (_PLANES + 4.0) + 4.0 * 159553, "flops": c["n"] * _FORWARD}
    if k == "train":
        return {"bytes": c["n"] * float(_PLANES) + 4.0 * 159553 * 7, "flops": 3.0 * c["n"] * _FORWARD}
    if k == "turn":
        return {"bytes": 2.0 * c["nch"] * c["n_t"], "flops": 0.0}
    if k == "assemble":
        return {"bytes": 2.0 * c["nch"] * (c["n_out"] + c["carry"]), "flops": 0.0}
    # a block copied and the bursts' samples: signal, word, one byte in and out
    values = 100.0 * c["bursts"] * c["nch"]
    return {"bytes": 2.0 * c["nch"] * c["n_out"] + 10.0 * values, "flops": 100.0 * values}


def _parameters():
    v = torch.from_numpy(_weights().astype(np.float64).ravel()).to(DEVICE).requires_grad_(True)
    shapes = [(32, 2, 3, 3), (32,)] + [(32, 32, 3, 3), (32,)] * 3 + [(64, 2048), (64,), (1, 64), (1,)]
    parts, at = [], 0
    for s in shapes:
        n = int(np.prod(s))
        parts.append(v[at:at + n].view(s))
        at += n
    return v, parts


def _logits64(x, p):
    """The network in float64: convolutions as sums of nine shifted products."""
    for k in range(4):
        w, b = p[2 * k], p[2 * k + 1]
        n, ci, h, wd = x.shape
        cols = F.unfold(x, 3, padding=1)                                   # [n][ci*9][h*w]
        x = (torch.matmul(w.reshape(32, ci * 9), cols) + b[:, None]).view(n, 32, h, wd)
        x = F.max_pool2d(F.relu(x), 2)
    x = x.reshape(x.shape[0], 2048)
    x = F.relu(torch.matmul(x, p[8].t()) + p[9])
    return (torch.matmul(x, p[10].t()) + p[11])[:, 0]


def exact(case, seed):
    """Float64 logits, or loss and gradients, of the ranker's cases; every other kind
    returns whole numbers only."""
    if case["kind"] not in ("score", "train"):
        return None
    snip, labels = _ranker_inputs(case, seed)
    x = snip.view(torch.bfloat16).to(torch.float64)
    v, p = _parameters()
    if case["kind"] == "score":
        with torch.no_grad():
            return torch.cat([_logits64(x[i:i + 128], p) for i in range(0, x.shape[0], 128)])
    total = torch.zeros((), dtype=torch.float64, device=DEVICE)
    for i in range(0, x.shape[0], 64):
        z, y = _logits64(x[i:i + 64], p), labels[i:i + 64].to(torch.float64)
        part = F.binary_cross_entropy_with_logits(z, y, reduction="sum") / x.shape[0]
        part.backward(retain_graph=True)   # v's views are shared by the parts
        total += part.detach()
    return {"loss": total.reshape(1), "grads": v.grad}
