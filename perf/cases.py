"""The work that is timed: decoding steps as a serving program calls them.

Four kinds of pass, each through the public entry points of
``paper_2606_02955_amd``:

* ``step``: one ``fdllm_decode_step`` on given logits.  A request batch of B
  sequences spans L positions; every sequence has one active block of ``blk``
  positions, of which ``lo`` to ``hi`` are still masked (a step early in a
  block has all of them, a late one a few).  The batch's mask and tokens are
  set at the start of the pass (one device copy, as a program does when it
  takes up a batch), because the step updates them in place.
* ``confidence``: ``fdllm_confidence`` followed by ``fdllm_select_profile``,
  for a program that keeps the confidences and decides apart.
* ``lmhead``: one ``fdllm_lmhead_decode_step`` from hidden states and the
  output embedding.
* ``generation``: a whole generation on the device (``Generation.run``), with
  the library's synthetic logits producer in the model's place.

Vocabulary 126464 is LLaDA's; blocks of 32 and 64, spans of 256 to 1024 and
f = 1.0 / 0.75, tau = 0.9 are the decoding settings of the workloads in
``workloads/``; the other sizes are generic.
"""
from __future__ import annotations

import math

import torch

import paper_2606_02955_amd as fd

MASK_ID = -1          # token id in x where a position is still masked
MAX_LOGITS_BYTES = 8.4e9
MAX_LM_FLOPS = 4.3e12


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def _step(name, B, L, blk, V, dtype="bf16", lo=None, hi=None, selector="profile", param=1.0):
    return {"name": name, "kind": "step", "B": B, "L": L, "blk": blk, "V": V, "dtype": dtype,
            "lo": blk if lo is None else lo, "hi": blk if hi is None else hi,
            "selector": selector, "param": param}


def _lmhead(name, B, L, blk, d, V, lo=None, hi=None, selector="profile", param=1.0):
    return {"name": name, "kind": "lmhead", "B": B, "L": L, "blk": blk, "d": d, "V": V,
            "lo": blk if lo is None else lo, "hi": blk if hi is None else hi,
            "selector": selector, "param": param}


def listed():
    return [
        # one request, the first step of a block, float32 logits: the smallest call
        _step("step_b1_f32", 1, 32, 32, 126464, "f32"),
        # a small server's batch in mid-generation, logits of the whole span at
        # hand (no cache), each block somewhere on its way from 32 to 1 masked
        _step("step_b64_span512", 64, 512, 32, 126464, lo=1, hi=32),
        # the largest batch, first step of a block: every position masked
        _step("step_b1024_full", 1024, 32, 32, 126464),
        # the same batch near the end of its blocks: one to three masked each
        _step("step_b1024_late", 1024, 32, 32, 126464, lo=1, hi=3, selector="factor", param=0.75),
        # a batch that is no multiple of the chip, blocks wider than a wavefront
        _step("step_b300_blk128", 300, 256, 128, 32000, lo=32, hi=128, selector="threshold", param=0.9),
        # a vocabulary of odd length, ragged blocks
        _step("step_b48_odd_vocab", 48, 200, 40, 50257, lo=5, hi=40),
        # float32 logits, confidences and decision apart
        {"name": "confidence_b100_f32", "kind": "confidence", "B": 100, "L": 48, "blk": 48, "V": 126464,
         "dtype": "f32", "lo": 8, "hi": 48, "param": 0.75},
        # the LM head for one request's block: latency of batch 1
        _lmhead("lmhead_b1", 1, 32, 32, 4096, 126464),
        # the LM head for four requests' blocks
        _lmhead("lmhead_b4", 4, 32, 32, 4096, 126464),
        # hidden states of whole spans, a partly masked block active in each
        _lmhead("lmhead_b8_span256", 8, 256, 32, 3072, 126464, lo=1, hi=32),
        # a large batch's blocks through the LM head: the matrix-core end
        _lmhead("lmhead_b128", 128, 32, 32, 4096, 126464),
        # whole generations on the device: every step of eight sequences
        {"name": "generation_b8", "kind": "generation", "B": 8, "G": 256, "blk": 32, "V": 126464,
         "selector": "profile", "param": 1.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _masked_range(rng, blk):
    stage = rng.random()
    if stage < 0.35:
        return blk, blk                               # first step of the blocks
    if stage < 0.75:
        return 1, blk                                 # anywhere
    return 1, max(1, blk // 8)                        # near the end


def draw(rng):
    """One more case of the ranges above."""
    kind = rng.choice(["step", "step", "step", "confidence", "lmhead", "lmhead", "lmhead", "generation"])
    selector, param = rng.choice([("profile", 1.0), ("profile", 0.75), ("factor", 1.0), ("factor", 0.75),
                                  ("threshold", 0.9)])
    if kind == "generation":
        return {"kind": kind, "B": _log_int(rng, 1, 8), "G": 32 * rng.randint(2, 8), "blk": rng.choice([16, 32]),
                "V": _log_int(rng, 4000, 126464), "selector": selector, "param": param}
    if kind == "lmhead":
        blk = rng.choice([16, 32, 32, 32, 48, 64])
        span = blk * rng.choice([1, 1, 1, 2, 8])
        B = max(1, _log_int(rng, 1, 128) * 32 // blk)
        d = 512 * rng.randint(2, 8) if rng.random() < 0.75 else 64 * rng.randint(16, 64)
        V = _log_int(rng, 16000, 152000)
        lo, hi = _masked_range(rng, blk)
        while 2.0 * B * blk * d * V > MAX_LM_FLOPS:
            B = max(1, B // 2)
        return _lmhead_unnamed(B, span, blk, d, V, lo, hi, selector, param)
    dtype = "f32" if kind == "confidence" or rng.random() < 0.2 else "bf16"
    blk = rng.choice([8, 16, 32, 32, 32, 40, 48, 64, 100, 128])
    span = blk * rng.choice([1, 1, 2, 4, 8])
    B = _log_int(rng, 1, 1024)
    V = _log_int(rng, 4000, 152000)
    if rng.random() < 0.7:
        V = max(8, V // 8 * 8)
    esize = 4 if dtype == "f32" else 2
    while B * span * V * esize > MAX_LOGITS_BYTES:
        if span > blk:
            span = max(blk, span // 2 // blk * blk)
        else:
            B = max(1, B // 2)
    lo, hi = _masked_range(rng, blk)
    case = {"kind": kind, "B": B, "L": span, "blk": blk, "V": V, "dtype": dtype, "lo": lo, "hi": hi, "param": param}
    if kind == "confidence":
        case["param"] = rng.choice([1.0, 0.75])
    else:
        case["selector"] = selector
    return case


def _lmhead_unnamed(*args):
    case = _lmhead("", *args)
    del case["name"]
    return case


def _masked_counts(case):
    """Masked positions of each sequence's active block: lo..hi, spread evenly."""
    n = case["hi"] - case["lo"] + 1
    return [case["lo"] + (7 * b + 3) % n for b in range(case["B"])]


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class State:
    pass


def _gen(seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed((int(seed) * 0x9E3779B97F4A7C15 + 0x2606) & ((1 << 63) - 1))
    return g


def _windows(case, g, dev):
    """Active blocks, mask (the positions after the block are masked too) and
    the flat indices of the candidates, the block's masked positions."""
    B, L, blk = case["B"], case["L"], case["blk"]
    k = torch.randint(0, L // blk, (B,), generator=g, device=dev)
    counts = torch.tensor(_masked_counts(case), device=dev)
    order = torch.rand((B, blk), generator=g, device=dev).argsort(dim=1)
    in_block = order < counts.view(B, 1)
    mask = torch.zeros((B, L), dtype=torch.uint8, device=dev)
    pos = (k * blk).view(B, 1) + torch.arange(blk, device=dev)
    mask.scatter_(1, pos, in_block.to(torch.uint8))
    rows = mask.view(-1).nonzero().view(-1)
    mask |= (torch.arange(L, device=dev) >= ((k + 1) * blk).view(B, 1)).to(torch.uint8)
    return (k * blk).to(torch.int32), ((k + 1) * blk).to(torch.int32), mask, rows


def _sequence_state(s, case, mask, g, dev):
    """mask and x in one buffer, so a batch is taken up with one copy."""
    B, L, V = case["B"], case["L"], case["V"]
    n = B * L
    s.fresh = torch.empty((5 * n,), dtype=torch.uint8, device=dev)
    x = torch.randint(0, V, (B, L), generator=g, device=dev).to(torch.int32)
    x[mask.bool()] = MASK_ID
    s.fresh[:4 * n].view(torch.int32).copy_(x.view(-1))
    s.fresh[4 * n:].copy_(mask.view(-1))
    s.batch = s.fresh.clone()
    s.x = s.batch[:4 * n].view(torch.int32).view(B, L)
    s.mask = s.batch[4 * n:].view(B, L)


def _outputs(s, B, L, dev):
    s.tokens = torch.empty((B, L), dtype=torch.int32, device=dev)
    s.conf = torch.empty((B, L), dtype=torch.float32, device=dev)
    s.eps = torch.empty((B, L), dtype=torch.float32, device=dev)
    s.lse = torch.empty((B, L), dtype=torch.float32, device=dev)
    s.commit = torch.empty((B, L), dtype=torch.uint8, device=dev)
    s.n_commit = torch.empty((B,), dtype=torch.int32, device=dev)


def _spikes(n, g, dev):
    """Heights of the model's choice over its background: 60% confident."""
    sure = torch.rand((n,), generator=g, device=dev) < 0.6
    u = torch.rand((n,), generator=g, device=dev)
    return torch.where(sure, 8.0 + 6.0 * u, 6.0 * u)


def _fill_logits(logits, rows, g, dev):
    """N(0, 1) plus a spike per row; one row in twenty has its top value twice.
    Only the candidates' rows hold logits (no other row is read)."""
    V = logits.shape[-1]
    flat = logits.view(-1, V)
    chunk = max(1, int(6e7) // V)
    for first in range(0, rows.numel(), chunk):
        idx = rows[first:first + chunk]
        n = idx.numel()
        r = torch.empty((n, V), dtype=torch.float32, device=dev).normal_(generator=g)
        t = torch.randint(0, V, (n, 2), generator=g, device=dev)
        r.scatter_add_(1, t[:, :1], _spikes(n, g, dev).view(n, 1))
        top = r.amax(dim=1, keepdim=True)
        second = torch.where(torch.rand((n, 1), generator=g, device=dev) < 0.05, top, r.gather(1, t[:, 1:]))
        r.scatter_(1, t[:, 1:], second)
        flat[idx] = r.to(logits.dtype)


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    s = State()
    s.kind = case["kind"]
    if s.kind == "generation":
        s.gen = fd.Generation(case["B"], case["G"], case["blk"], case["V"], seed=int(seed) + 1,
                              selector=case["selector"], param=case["param"])
        return s
    g = _gen(seed, dev)
    B, L, V = case["B"], case["L"], case["V"]
    s.start, s.end, mask, s.rows = _windows(case, g, dev)
    _sequence_state(s, case, mask, g, dev)
    _outputs(s, B, L, dev)
    s.selector, s.param = case.get("selector"), case["param"]
    if s.kind == "lmhead":
        d = case["d"]
        s.weight = torch.empty((V, d), dtype=torch.bfloat16, device=dev).normal_(generator=g).mul_(d ** -0.5)
        # hidden states that point at a token each, over a background
        n = B * L
        s.hidden = torch.empty((B, L, d), dtype=torch.bfloat16, device=dev)
        flat = s.hidden.view(n, d)
        for first in range(0, n, 8192):
            k = min(8192, n - first)
            w = s.weight[torch.randint(0, V, (k,), generator=g, device=dev)].float()
            h = torch.empty((k, d), dtype=torch.float32, device=dev).normal_(generator=g)
            h += w * (_spikes(k, g, dev) / w.square().sum(dim=1)).view(k, 1)
            flat[first:first + k] = h.to(torch.bfloat16)
        need = fd.fdllm_lmhead_workspace_size(B, L, d, V)
    else:
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        s.logits = torch.empty((B, L, V), dtype=dt, device=dev)
        _fill_logits(s.logits, s.rows, g, dev)
        need = fd.fdllm_workspace_size(B, L, V, dt)
    s.workspace = torch.empty((max(need, 256),), dtype=torch.uint8, device=dev)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    if s.kind == "generation":
        steps = s.gen.run()
        return {"steps": steps, "x": s.gen.x, "mask": s.gen.mask, "hist": s.gen.hist, "logits": s.gen.logits}
    if s.kind == "confidence":
        fd.fdllm_confidence(s.logits, s.mask, s.start, s.end, s.tokens, s.conf, s.eps, s.lse)
        fd.fdllm_select_profile(s.conf, s.eps, s.mask, s.start, s.end, s.param, s.commit, s.n_commit)
        return {"tokens": s.tokens, "conf": s.conf, "eps": s.eps, "lse": s.lse, "commit": s.commit,
                "n_commit": s.n_commit}
    s.batch.copy_(s.fresh)
    if s.kind == "lmhead":
        fd.fdllm_lmhead_decode_step(s.hidden, s.weight, s.mask, s.start, s.end, s.x, s.selector, s.param,
                                    tokens=s.tokens, conf=s.conf, eps=s.eps, lse=s.lse, commit=s.commit,
                                    n_commit=s.n_commit, workspace=s.workspace)
    else:
        fd.fdllm_decode_step(s.logits, s.mask, s.start, s.end, s.x, s.selector, s.param, tokens=s.tokens,
                             conf=s.conf, eps=s.eps, lse=s.lse, commit=s.commit, n_commit=s.n_commit,
                             workspace=s.workspace)
    return {"tokens": s.tokens, "conf": s.conf, "eps": s.eps, "lse": s.lse, "commit": s.commit,
            "n_commit": s.n_commit, "x": s.x, "mask": s.mask}


def work(case):
    if case["kind"] == "generation":
        # every step writes the active blocks' logits and reads the masked rows
        # (half a block on average); a sequence takes about 0.55 steps a
        # position at these settings
        B, G, blk, V = case["B"], case["G"], case["blk"], case["V"]
        return {"bytes": 0.55 * G * B * 1.5 * blk * V * 2.0, "flops": 0.0}
    n = sum(_masked_counts(case))
    slots = case["B"] * case["L"]
    small = 18.0 * slots + 12.0 * case["B"]
    if case["kind"] == "lmhead":
        d, V = case["d"], case["V"]
        return {"bytes": 2.0 * V * d + 2.0 * n * d + small, "flops": 2.0 * n * V * d}
    return {"bytes": n * float(case["V"]) * (4 if case["dtype"] == "f32" else 2) + small, "flops": 0.0}


def tolerance(case):
    if case["kind"] == "generation":
        # the producer's bits are fixed; a step's decision moves only where a
        # confidence sits within its rounding of a boundary
        return {"rel": 1e-6, "differ": 0.005}
    if case["kind"] == "lmhead":
        # float32 accumulation over the hidden dimension, in any order
        return {"rel": 1e-5, "differ": 0.005}
    # float32 outputs of sums carried in 64 bits
    return {"rel": 1e-6, "differ": 0.002}


# ---------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ---------------------------------------------------------------------------
def _exact_rows(l64):
    top, tok = l64.max(dim=1)
    tok = (l64 == top.view(-1, 1)).to(torch.uint8).argmax(dim=1)      # the lowest index
    e = (l64 - top.view(-1, 1)).exp_()
    e.scatter_(1, tok.view(-1, 1), 0.0)
    rest = e.sum(dim=1)
    return tok, 1.0 / (1.0 + rest), rest / (1.0 + rest), top + torch.log1p(rest)


def exact(case, seed):
    if case["kind"] == "generation":
        return None
    s = prepare(case, seed)
    B, L = case["B"], case["L"]
    dev = s.mask.device
    tokens = torch.full((B * L,), -1, dtype=torch.int32, device=dev)
    conf = torch.zeros((B * L,), dtype=torch.float64, device=dev)
    eps = torch.ones((B * L,), dtype=torch.float64, device=dev)
    lse = torch.zeros((B * L,), dtype=torch.float64, device=dev)
    rows = s.rows
    if case["kind"] == "lmhead":
        w = s.weight.double()
        flat = s.hidden.view(B * L, -1)
        chunk = 128
    else:
        flat = s.logits.view(B * L, -1)
        chunk = max(1, int(3e7) // case["V"])
    for first in range(0, rows.numel(), chunk):
        idx = rows[first:first + chunk]
        l64 = flat[idx].double()
        if case["kind"] == "lmhead":
            l64 = l64 @ w.t()
        t, c, e, z = _exact_rows(l64)
        tokens[idx], conf[idx], eps[idx], lse[idx] = t.to(torch.int32), c, e, z
    out = {"tokens": tokens.view(B, L), "conf": conf.view(B, L), "eps": eps.view(B, L), "lse": lse.view(B, L),
           "commit": None, "n_commit": None}
    if case["kind"] != "confidence":
        out.update(x=None, mask=None)
    return out
