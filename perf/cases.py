"""Performance cases: the calls that a program using this package makes, over
the range of sizes, nests and data types it makes them with.

listed() gives the named cases, draw() one more of the same ranges.
prepare() makes what a program holds before the call (activations, packed
weights, routing and workspace buffers, in one case a captured graph), run()
is one pass through the public entry points, work() the bytes and operations
the pass cannot do without, tolerance() how far another correct
implementation may be off, and exact() the same outputs in binary64 with
plain torch.

Inputs are drawn on the GPU from the seed alone: Gaussian activations, gate
and expert weights (std 1, 0.02, 0.02), per-(request, expert) bit-widths from
the case's choices.  They are the recipes of workloads.py, drawn with torch's
generator so that a full-size layer takes a fraction of a second.

Kinds of case:
  layer     route (bit-width table, or learned bit-width routers) + forward
  block     a decode step of a stacked decoder, replayed from a HIP graph:
            residual + RMS norm, route, forward
  streamed  route, HEBF order, forward with the experts copied from pinned
            host memory
  pack      MWQ quantize + bit-plane pack of expert weights
  calibrate calibration-aware MWQ of one expert matrix: factor + pack
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2504_15299_amd import api

DEV = "cuda:0"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


# ---- cases -------------------------------------------------------------------

def _layer(name, **kw):
    c = dict(name=name, kind="layer", d=4096, f=14336, E=8, k=2, T=16, group=128, dtype="bf16",
             b_min=2, b_max=8, bits="2,3,4,8", probs="0.2,0.3,0.3,0.2", per="request_expert",
             requests=16, zipf=0.0, learned=False, shared_f=0, shared_bits=8)
    c.update(kw)
    return c


def listed():
    return [
        # one user, one token: the latency of a single decode step
        _layer("decode_1", T=1, requests=1),
        # the serving batch the package's benchmark quotes
        _layer("decode_16"),
        # a decoder block of the 64-sequence stack, one bit-width tier per
        # sequence, launched as a captured graph like a serving loop does
        _layer("decode_64_block_graph", kind="block", T=64, requests=64, bits="2,4,8", probs="",
               per="request"),
        # a dense SwiGLU FFN as the one-expert layer, nest 2..4
        _layer("dense_decode_16", d=5120, f=13824, E=1, k=1, b_max=4, bits="2,3,4",
               probs="0.3,0.4,0.3", per="request"),
        # prompts of four requests, expert load ~ Zipf(1.1)
        _layer("prefill_2048", T=2048, requests=4, bits="2,4,8", probs="", zipf=1.1),
        # a short ragged prompt batch, nest 5..8, learned bit-width routers
        _layer("prefill_301_learned", T=301, requests=1, b_min=5, bits="5,6,7,8", probs="",
               learned=True),
        # fine-grained layer with a shared expert, hottest experts widest
        _layer("fine_512_shared", d=2048, f=1408, E=64, k=6, T=512, group=64, requests=1,
               bits="8,4,3,2", probs="", per="hottest", shared_f=5632),
        # the same layer decoding a small batch
        _layer("fine_24_shared", d=2048, f=1408, E=64, k=6, T=24, group=64, requests=1,
               bits="8,4,3,2", probs="", per="hottest", shared_f=5632),
        # small fp32 layer: launches and latency
        _layer("tiny_64_f32", d=256, f=512, T=64, group=64, dtype="f32", requests=1,
               bits="2,4,8", probs=""),
        # experts from pinned host memory, nothing resident at the start
        _layer("streamed_16", kind="streamed", d=2048, f=5632),
        # packing one expert's W1/W3 when a model is prepared
        dict(name="pack_expert", kind="pack", E=1, rows=28672, cols=4096, group=128, b_min=2,
             b_max=8),
        # calibration-aware packing of a fine-grained expert's W1/W3
        dict(name="calibrate_expert", kind="calibrate", rows=2816, cols=2048, group=64, gamma=128,
             b_min=2, b_max=8, tokens=2048),
    ]


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


_NESTS = (  # b_min, b_max, widths, probabilities
    (2, 8, "2,3,4,8", "0.2,0.3,0.3,0.2"),
    (2, 8, "2,4,8", ""),
    (2, 4, "2,3,4", "0.3,0.4,0.3"),
    (5, 8, "5,6,7,8", ""),
)


def draw(rng: random.Random):
    fam = rng.choice(["decode", "decode", "block", "dense", "prefill", "prefill", "fine", "fine",
                      "tiny", "streamed", "pack", "calibrate"])
    b_min, b_max, bits, probs = rng.choice(_NESTS)
    nest = dict(b_min=b_min, b_max=b_max, bits=bits, probs=probs)
    d, f = 128 * rng.randint(8, 32), 128 * rng.randint(8, 112)
    if fam == "pack":
        # row counts are multiples of 32 and need not fill a tile
        rows, cols = 32 * _logint(rng, 16, 880), 128 * _logint(rng, 4, 112)
        E = 2 if rows * cols < 1 << 25 else 1
        while rows * cols > 28672 * 4096:
            rows = rows // 64 * 32
        return dict(kind="pack", E=E, rows=rows, cols=cols, group=rng.choice([64, 128]),
                    b_min=b_min, b_max=b_max)
    if fam == "calibrate":
        gamma = rng.choice([64, 128])
        return dict(kind="calibrate", rows=32 * _logint(rng, 8, 88), cols=128 * rng.randint(2, 16),
                    group=rng.choice([64, gamma]), gamma=gamma, b_min=b_min, b_max=b_max,
                    tokens=_logint(rng, 128, 2048))
    if fam in ("decode", "block"):
        T = _logint(rng, 1, 64)
        E = rng.choice([4, 8, 8, 16])
        c = _layer("", d=d, f=f if E < 16 else min(f, 7168), E=E, k=rng.choice([1, 2, 2]), T=T,
                   requests=T, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                   learned=fam == "decode" and rng.random() < 0.25,
                   kind="block" if fam == "block" else "layer",
                   per="request" if fam == "block" else "request_expert", **nest)
        if fam == "block":
            c["dtype"] = "bf16"
    elif fam == "dense":
        T = _logint(rng, 1, 64)
        c = _layer("", d=128 * rng.randint(16, 40), f=128 * rng.randint(32, 108), E=1, k=1, T=T,
                   requests=T, per="request", **nest)
    elif fam == "prefill":
        c = _layer("", d=d, f=f, T=_logint(rng, 65, 2048), requests=rng.randint(1, 4),
                   group=rng.choice([128, 128, 64]), zipf=rng.choice([0.0, 1.1]),
                   learned=rng.random() < 0.25, **nest)
    elif fam == "fine":
        E = rng.choice([16, 32, 64])
        c = _layer("", d=64 * rng.randint(8, 32), f=64 * rng.randint(4, 22), E=E,
                   k=rng.randint(2, 6), T=_logint(rng, 1, 512), group=64, requests=1,
                   per="hottest" if b_max == 8 and b_min == 2 else "request_expert",
                   shared_f=rng.choice([0, 1, 1]) * 64 * rng.randint(8, 88),
                   shared_bits=b_max, **nest)
        if c["per"] == "hottest":
            c.update(bits="8,4,3,2", probs="")
    elif fam == "tiny":
        g = rng.choice([64, 128])
        c = _layer("", d=g * rng.randint(2, 6), f=g * rng.randint(2, 8), T=_logint(rng, 1, 128),
                   group=g, dtype="f32", requests=1, **nest)
    else:
        c = _layer("", kind="streamed", d=128 * rng.randint(4, 16), f=128 * rng.randint(8, 44),
                   T=_logint(rng, 1, 128), requests=1, **nest)
    del c["name"]
    return c


# ---- inputs --------------------------------------------------------------------

_X, _WG, _WR, _W13, _W2, _S13, _S2, _Y, _BITS = range(9)


def _gen(seed, purpose, i=0):
    # a seed of its own for every tensor, so that exact() can draw each again
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1_000_003 + purpose * 8191 + i) & ((1 << 62) - 1))
    return g


def _randn(shape, seed, purpose, i=0, std=1.0):
    return torch.randn(shape, generator=_gen(seed, purpose, i), device=DEV).mul_(std)


def _weights(c, seed, purpose, rows, cols, E):
    """Packed weights of E matrices, each expert drawn and packed by itself."""
    w = api.MWQ.empty(E, rows, cols, c["group"], c["b_min"], c["b_max"], device=DEV)
    for e in range(E):
        api.pack_mwq(_randn((1, rows, cols), seed, purpose, e, 0.02), w.expert(e))
    return w


def _choices(c):
    ch = np.array([int(b) for b in c["bits"].split(",")], np.uint8)
    p = [float(v) for v in c["probs"].split(",")] if c["probs"] else None
    return ch, p


def _gate(c, seed):
    Wg = _randn((c["E"], c["d"]), seed, _WG, 0, 0.02)
    bias = None
    if c["zipf"] > 0:
        p = (np.arange(c["E"]) + 1.0) ** -c["zipf"]
        bias = torch.from_numpy(np.log(p / p.sum()).astype(np.float32)).to(DEV)
    return Wg, bias


def _top(c, x, Wg, bias):
    """Gate logits, top-k experts and softmax weights in binary64."""
    logits = x.double() @ Wg.double().t()
    if bias is not None:
        logits = logits + bias.double()
    v, i = torch.sort(logits, dim=1, descending=True, stable=True)
    return logits, i[:, :c["k"]], torch.softmax(v[:, :c["k"]], dim=1)


def _requests(c):
    per = max(c["T"] // c["requests"], 1)
    return np.minimum(np.arange(c["T"]) // per, c["requests"] - 1).astype(np.int32)


def _bit_table(c, seed, x, Wg, bias):
    """[requests][E] bit-widths."""
    ch, p = _choices(c)
    R, E = c["requests"], c["E"]
    rng = np.random.default_rng([seed, _BITS])
    if c["per"] == "hottest":  # a quarter of the experts per width, hottest widest
        idx = _top(c, x, Wg, bias)[1]
        counts = torch.bincount(idx.reshape(-1), minlength=E).cpu().numpy()
        order = np.argsort(-counts, kind="stable")
        t = np.empty(E, np.uint8)
        t[order] = ch[np.minimum(np.arange(E) * len(ch) // E, len(ch) - 1)]
        t = np.repeat(t[None], R, axis=0)
    elif c["per"] == "request":
        t = np.repeat(rng.choice(ch, size=(R, 1), p=p), E, axis=1)
    else:
        t = rng.choice(ch, size=(R, E), p=p)
    return t.astype(np.uint8)


def _layer_inputs(c, seed):
    """Everything of a layer but the expert weights."""
    s = dict(x=_randn((c["T"], c["d"]), seed, _X).to(DTYPES[c["dtype"]]))
    s["Wg"], s["bias"] = _gate(c, seed)
    L = c["b_max"] - c["b_min"] + 1
    if c["learned"]:
        s["Wr"] = _randn((c["E"], L, c["d"]), seed, _WR, 0, 0.05)
        s["br"] = _randn((c["E"], L), seed, _WR, 1, 0.05)
    else:
        s["req"] = torch.from_numpy(_requests(c)).to(DEV)
        s["table"] = torch.from_numpy(_bit_table(c, seed, s["x"], s["Wg"], s["bias"])).to(DEV)
    if c["kind"] == "block":
        # the residual stream before the block and the previous layer's
        # output; the block routes their normalised sum
        s["res"] = s.pop("x").float()
        s["y"] = _randn((c["T"], c["d"]), seed, _Y, 0, 0.5).to(torch.bfloat16)
    return s


def prepare(case, seed):
    c = case
    if c["kind"] == "pack":
        W = _randn((c["E"], c["rows"], c["cols"]), seed, _W13, 0, 0.02)
        return dict(c=c, W=W, out=api.MWQ.empty(c["E"], c["rows"], c["cols"], c["group"],
                                                c["b_min"], c["b_max"], device=DEV))
    if c["kind"] == "calibrate":
        X, lam = _calib_x(c, seed)
        W = _randn((1, c["rows"], c["cols"]), seed, _W13, 0, 0.02)
        return dict(c=c, W=W, X=X, lam=lam,
                    out=api.MWQ.empty(1, c["rows"], c["cols"], c["group"], c["b_min"], c["b_max"],
                                      device=DEV))
    T, d, f, E, k = c["T"], c["d"], c["f"], c["E"], c["k"]
    s = _layer_inputs(c, seed)
    s["c"] = c
    s["w13"] = _weights(c, seed, _W13, 2 * f, d, E)
    s["w2"] = _weights(c, seed, _W2, d, f, E)
    s["shared"] = None
    if c["shared_f"]:
        s["shared"] = (_weights(c, seed, _S13, 2 * c["shared_f"], d, 1),
                       _weights(c, seed, _S2, d, c["shared_f"], 1), c["shared_bits"])
    # buffers that a serving program keeps
    s["r"] = api.Routing.empty(T, E, k, c["b_min"], c["b_max"], device=DEV)
    s["ws"] = torch.empty(api.moe_forward_workspace(T, d, f, E, k, c["shared_f"]),
                          dtype=torch.uint8, device=DEV)
    s["out"] = torch.empty((T, d), dtype=DTYPES[c["dtype"]], device=DEV)
    if c["learned"]:
        s["bit_logits"] = torch.empty((T, E, c["b_max"] - c["b_min"] + 1), device=DEV)
    if c["kind"] == "streamed":
        s["h13"], s["h2"] = _to_host(s["w13"]), _to_host(s["w2"])
        for w in (s["w13"], s["w2"]):  # the device copy starts empty
            for t in (w.planes, w.scales, w.zeros):
                t.zero_()
        s["io"] = torch.cuda.Stream()
        s["events"] = [torch.cuda.Event() for _ in range(E * (c["b_max"] - c["b_min"] + 1))]
    if c["kind"] == "block":
        s["stream"] = torch.empty_like(s["res"])
        s["h"] = torch.empty((T, d), dtype=torch.bfloat16, device=DEV)
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _block_step(s)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _block_step(s)
    return s


def _to_host(w):
    return api.MWQ(w.n_experts, w.rows, w.cols, w.group, w.b_min, w.b_max,
                   *[torch.empty(t.shape, dtype=t.dtype, pin_memory=True).copy_(t)
                     for t in (w.planes, w.scales, w.zeros)])


def _calib_x(c, seed):
    """Calibration activations with correlated features (AR(1), 0.9) and the
    damping, 1 % of the Hessian's mean diagonal."""
    n = c["cols"]
    z = _randn((c["tokens"], n), seed, _X)
    a = torch.arange(n, device=DEV, dtype=torch.float64)
    lag = a[:, None] - a[None, :]
    mix = torch.where(lag >= 0, torch.pow(0.9, lag.clamp(min=0)), torch.zeros_like(lag))
    mix = mix * math.sqrt(1 - 0.81)
    mix[:, 0] /= math.sqrt(1 - 0.81)
    X = (z.double() @ mix.t()).float().contiguous()
    lam = 0.01 * float((2.0 * X.double().square().sum(0)).mean())
    return X, lam


# ---- one pass ------------------------------------------------------------------

def _route(s):
    c = s["c"]
    if c["learned"]:
        api.route_learned(s["x"], s["Wg"], s["bias"], c["k"], s["Wr"], s["br"], c["b_min"],
                          c["b_max"], out=s["r"], bit_logits=s["bit_logits"])
    else:
        api.route(s["x"], s["Wg"], s["bias"], c["k"], s["req"], s["table"], c["b_min"],
                  c["b_max"], out=s["r"])


def _block_step(s):
    s["stream"].copy_(s["res"])
    s["x"] = api.residual_rmsnorm(s["stream"], s["y"], h=s["h"])
    _route(s)
    api.moe_forward(s["x"], s["w13"], s["w2"], s["r"], s["c"]["k"], out=s["out"],
                    workspace=s["ws"])


def _layer_outputs(s):
    r = s["r"]
    o = dict(out=s["out"], logits=r.logits, topk_idx=r.topk_idx, topk_w=r.topk_w,
             topk_bits=r.topk_bits, hist=r.hist)
    if s["c"]["learned"]:
        o["bit_logits"] = s["bit_logits"]
    return o


def run(s):
    c = s["c"]
    if c["kind"] == "pack":
        w = api.pack_mwq(s["W"], s["out"])
        return dict(planes=w.planes, scales=w.scales, zeros=w.zeros)
    if c["kind"] == "calibrate":
        U, info = api.mwq_calib_factor(s["X"], s["lam"])
        w = api.pack_mwq_calibrated(s["W"], U, c["gamma"], s["out"])
        return dict(U=U, info=info, planes=w.planes, scales=w.scales, zeros=w.zeros)
    if c["kind"] == "block":
        s["graph"].replay()
        return dict(_layer_outputs(s), stream=s["stream"], h=s["h"])
    _route(s)
    if c["kind"] == "streamed":
        hist = s["r"].hist.cpu().numpy()  # the unit order is made on the host
        units = api.hebf_order(hist, c["b_min"], c["b_max"])
        resident = np.zeros(c["E"], np.uint8)
        api.moe_forward_streamed(s["x"], s["h13"], s["h2"], s["w13"], s["w2"], resident, s["r"],
                                 c["k"], hist, units, s["events"][:len(units)], s["io"],
                                 out=s["out"], workspace=s["ws"])
        return dict(_layer_outputs(s), resident=resident)
    api.moe_forward(s["x"], s["w13"], s["w2"], s["r"], c["k"], shared=s["shared"], out=s["out"],
                    workspace=s["ws"])
    return _layer_outputs(s)


# ---- bytes and operations ------------------------------------------------------

def _mwq_bytes(rows, cols, group, b_min, bits):
    return rows * cols * bits / 8 + rows * (cols // group) * (2 * (bits - b_min + 1) + 1)


def work(case):
    c = case
    if c["kind"] == "pack":
        n = c["E"] * c["rows"] * c["cols"]
        return dict(bytes=4 * n + c["E"] * _mwq_bytes(c["rows"], c["cols"], c["group"],
                                                      c["b_min"], c["b_max"]),
                    # min/max, round, residual; two passes per residual level
                    flops=n * (8 + 4 * (c["b_max"] - c["b_min"])))
    if c["kind"] == "calibrate":
        n, h, T = c["rows"], c["cols"], c["tokens"]
        lv = c["b_max"] - c["b_min"] + 1
        return dict(bytes=4 * T * h + 4 * h * h + 4 * n * h
                    + _mwq_bytes(n, h, c["group"], c["b_min"], c["b_max"]),
                    # symmetric Hessian, Cholesky, triangular inverse, and one
                    # compensation pass per level
                    flops=T * h * h + 2 * h ** 3 / 3 + lv * n * h * h)
    # the routing of a sample with uniform (or Zipf) expert choice
    rng = np.random.default_rng(1)
    T, d, f, E, k = c["T"], c["d"], c["f"], c["E"], c["k"]
    p = (np.arange(E) + 1.0) ** -c["zipf"]
    score = rng.gumbel(size=(T, E)) + np.log(p)
    top = np.argsort(-score, axis=1)[:, :k]
    ch, pr = _choices(c)
    if c["learned"]:
        wid = rng.choice(ch, size=(T, E))
    elif c["per"] == "hottest":
        order = np.argsort(-np.bincount(top.reshape(-1), minlength=E), kind="stable")
        t = np.empty(E, int)
        t[order] = ch[np.minimum(np.arange(E) * len(ch) // E, len(ch) - 1)]
        wid = np.repeat(t[None], T, axis=0)
    else:
        t = rng.choice(ch, size=(c["requests"], 1 if c["per"] == "request" else E), p=pr)
        wid = np.broadcast_to(t, (c["requests"], E))[_requests(c)]
    maxbit = np.zeros(E, int)
    for t in range(T):
        for e in top[t]:
            maxbit[e] = max(maxbit[e], int(wid[t, e]))
    g, es = c["group"], 2 if c["dtype"] == "bf16" else 4
    nbytes = sum(_mwq_bytes(2 * f, d, g, c["b_min"], int(b)) + _mwq_bytes(d, f, g, c["b_min"], int(b))
                 for b in maxbit if b)
    flops = 6.0 * d * f * T * k + 2.0 * T * E * d
    nbytes += 2 * T * d * es + 4 * E * d
    if c["learned"]:
        lv = c["b_max"] - c["b_min"] + 1
        nbytes += 4 * E * lv * d
        flops += 2.0 * T * E * lv * d
    if c["shared_f"]:
        sf = c["shared_f"]
        nbytes += (_mwq_bytes(2 * sf, d, g, c["b_min"], c["shared_bits"])
                   + _mwq_bytes(d, sf, g, c["b_min"], c["shared_bits"]))
        flops += 6.0 * d * sf * T
    if c["kind"] == "block":
        nbytes += 10 * T * d
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    if case["kind"] == "calibrate":
        # the factor is rounded once from binary64 and the codes are decided by
        # one binary32 operation sequence: an entry of the factor that rounds
        # the other way may move the later codes of a row
        return dict(rel=1e-6, max=1e-4, differ=2e-3)
    # bf16 operands and results with fp32 sums; near-tied logits may pick
    # another expert for a few of the selections
    return dict(rel=1e-2, max=0.1, differ=0.005)


# ---- the same outputs in binary64 ------------------------------------------------

def _mwq_levels(W, group, b_min, b_max):
    """The MWQ codes' values of W [rows][cols] float: yields (bits, W^_bits) for
    bits = b_min .. b_max, W^ in binary64.  The codes follow the documented
    binary32 steps (each group's base range with zero included, then one sign
    and the mean magnitude of the residual per level, summed in ascending
    column order)."""
    rows, cols = W.shape
    r = W.reshape(rows * (cols // group), group).t().contiguous()  # [group][n]
    qmax = float((1 << b_min) - 1)
    mn, mx = r.amin(0).clamp(max=0), r.amax(0).clamp(min=0)
    s = ((mx - mn) / qmax).half().float()
    s = torch.where((s > 0) & torch.isfinite(s), s, torch.ones_like(s))
    z = torch.round(-mn / s).clamp(0, qmax)
    q = torch.round(r / s + z).clamp(0, qmax)
    what = (q - z) * s
    r = r - what
    acc = what.double()
    del what, q

    def value():
        return acc.t().contiguous().reshape(rows, cols)

    yield b_min, value()
    for b in range(b_min + 1, b_max + 1):
        a = torch.zeros_like(s)
        for i in range(group):
            a = a + r[i].abs()
        sb = (a / float(group)).half().float()
        step = torch.where(r >= 0, sb, -sb)
        r = r - step
        acc = acc + step.double()
        yield b, value()


def _ffn(c, seed, p13, p2, e, f, x, bits):
    """SwiGLU of expert e at the rows' bit-widths: x [n][d] and bits [n] -> [n][d]."""
    d = x.shape[1]
    y = torch.zeros((x.shape[0], d), dtype=torch.float64, device=DEV)
    W13 = _randn((1, 2 * f, d), seed, p13, e, 0.02)[0]
    W2 = _randn((1, d, f), seed, p2, e, 0.02)[0]
    top = int(bits.max())
    l13 = _mwq_levels(W13, c["group"], c["b_min"], top)
    l2 = _mwq_levels(W2, c["group"], c["b_min"], top)
    for (b, V13), (_, V2) in zip(l13, l2):
        at = torch.nonzero(bits == b).reshape(-1)
        if at.numel():
            ac = x[at] @ V13.t()
            h = torch.nn.functional.silu(ac[:, :f]) * ac[:, f:]
            y[at] = h @ V2.t()
    return y


def exact(case, seed):
    c = case
    if c["kind"] == "pack":
        return None  # whole numbers, decided in binary32
    if c["kind"] == "calibrate":
        X, lam = _calib_x(c, seed)
        X = X.double()
        H = 2.0 * X.t() @ X + lam * torch.eye(c["cols"], dtype=torch.float64, device=DEV)
        # H^-1 = U^T U with U upper triangular
        J = torch.linalg.cholesky(H.flip(0, 1))
        eye = torch.eye(c["cols"], dtype=torch.float64, device=DEV)
        U = torch.linalg.solve_triangular(J, eye, upper=False).flip(0, 1)
        return dict(U=U, info=None, planes=None, scales=None, zeros=None)
    s = _layer_inputs(c, seed)
    o = {}
    if c["kind"] == "block":
        res = s["res"].double() + s["y"].double()
        h = res / torch.sqrt(res.square().mean(1, keepdim=True) + 1e-5)
        o.update(stream=res, h=h)
        x = h.to(torch.bfloat16)  # h is handed on in bf16
    else:
        x = s["x"]
    logits, idx, w = _top(c, x, s["Wg"], s["bias"])
    xd = x.double()
    if c["learned"]:
        bl = torch.einsum("td,eld->tel", xd, s["Wr"].double()) + s["br"].double()
        wid = c["b_min"] + bl.argmax(2)
        o["bit_logits"] = bl
    else:
        wid = s["table"].long()[s["req"].long()]
    bits = torch.gather(wid, 1, idx)
    out = torch.zeros_like(xd)
    for e in range(c["E"]):
        t, i = torch.nonzero(idx == e, as_tuple=True)
        if t.numel():
            y = _ffn(c, seed, _W13, _W2, e, c["f"], xd[t], bits[t, i])
            out.index_add_(0, t, w[t, i][:, None] * y)
    if c["shared_f"]:
        every = torch.full((c["T"],), c["shared_bits"], dtype=torch.int64, device=DEV)
        out += _ffn(c, seed, _S13, _S2, 0, c["shared_f"], xd, every)
    L = c["b_max"] - c["b_min"] + 1
    hist = torch.bincount((idx * L + bits - c["b_min"]).reshape(-1), minlength=c["E"] * L)
    o.update(out=out, logits=logits, topk_idx=idx, topk_w=w, topk_bits=bits,
             hist=hist.reshape(c["E"], L))
    if c["kind"] == "streamed":
        o["resident"] = None
    return o
