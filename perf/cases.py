"""The decoder's workloads, as a user's program calls them: what is prepared, one pass, its least work, and its exact result.

A case is one of five kinds:
  stream      one stream through `decode` (FP32, int8 or hard-decision input, blocked or full-frame, one or many traces per block)
  quantised   FP32 LLRs through `quantize`, then the int8 decode
  punctured   int8 values of a punctured stream through `depuncture`, then the decode
  batch       frames of mixed codes through `Batch.decode`
  serve       requests in pinned host memory through `Server`, from submission until all have completed
Codes are the three of the benchmark (K=7 rate 1/2 and 1/3, K=9 rate 1/2) and smaller ones of the tests.
"""
import math

import numpy as np
import torch

import paper_2011_09337_amd as vit

CODES = {
    "k7r12": (7, (0o171, 0o133)),
    "k7r13": (7, (0o133, 0o171, 0o165)),
    "k9r12": (9, (0o561, 0o753)),
    "k8r12": (8, (0o247, 0o371)),
    "k6r12": (6, (0o53, 0o75)),
    "k5r12": (5, (0o23, 0o35)),
    "k4r14": (4, (0o13, 0o15, 0o17, 0o11)),
    "k3r12": (3, (0o7, 0o5)),
}
MIX = ("k7r12", "k7r13", "k9r12")           # the codes of batches and of serving
RATE34 = ((1, 1), (1, 0), (0, 1))           # rate 3/4 from a rate-1/2 code
LLR_TYPE = {"f32": vit.VIT_LLR_F32, "i8": vit.VIT_LLR_I8}


def _overlap(k):
    return 5 * k if k <= 7 else 8 * (k - 1)


def _stream(name, code, n, dtype, L, v, **kw):
    case = {"name": name, "kind": "stream", "code": code, "n": n, "dtype": dtype, "L": L, "v": v, "terminated": True,
            "metric_bits": 0, "f0": 0, "w": 0, "ebn0": 3.0}
    case.update(kw)
    return case


def listed():
    return [
        # one short terminated frame decoded whole: a control-channel message, where the call's latency counts
        _stream("frame_i8_full", "k7r12", 1000, "i8", 0, 0),
        # a 4096-bit frame of soft values in blocks: the smallest blocked call
        _stream("frame_f32", "k7r12", 4096, "f32", 256, 42),
        # the continuous FP32 stream of the benchmark, at its block length
        _stream("stream_f32", "k7r12", 1 << 24, "f32", 512, 35),
        # the same length from int8 LLRs: a receiver that quantises its soft values
        _stream("stream_i8", "k7r12", 1 << 24, "i8", 512, 35),
        # the long code, int8, at the overlap it needs
        _stream("stream_i8_k9", "k9r12", 1 << 22, "i8", 256, 64, ebn0=2.0),
        # hard decisions of an open stream of odd length with a short code: a capture cut anywhere
        _stream("stream_hard_k5", "k5r12", 1000003, "hard", 256, 25, terminated=False, ebn0=5.0),
        # many traces per block, started from the stored best states
        _stream("subframes_f32", "k7r12", 1 << 22, "f32", 512, 35, f0=56, w=45),
        # soft values that arrive as FP32 and are quantised before the decode
        {"name": "quantised_k7r13", "kind": "quantised", "code": "k7r13", "n": 3000001, "L": 512, "v": 35, "ebn0": 2.0},
        # a rate-3/4 link: zeros put back in the punctured slots, then the rate-1/2 decode
        {"name": "punctured_i8", "kind": "punctured", "code": "k7r12", "n": 1 << 20, "L": 512, "v": 70, "ebn0": 5.0},
        # thousands of int8 frames of three codes, lengths uniform in [40, 6144], in shapes as the autotuner picks them
        {"name": "batch_i8", "kind": "batch", "frames": 8192, "dtype": "i8", "low": 40, "high": 6144, "tuned": True},
        # a small FP32 batch in the default shapes
        {"name": "batch_f32_small", "kind": "batch", "frames": 48, "dtype": "f32", "low": 40, "high": 6144, "tuned": False},
        # a burst of requests through the serving loop, lengths lognormal around 1024 bits
        {"name": "serve_i8", "kind": "serve", "frames": 2048, "median": 1024.0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("stream", "stream", "stream", "stream", "quantised", "punctured", "batch", "batch", "serve"))
    if kind == "serve":
        return {"kind": kind, "frames": _log(rng, 16, 2048), "median": rng.uniform(200.0, 1024.0)}
    if kind == "batch":
        return {"kind": kind, "frames": _log(rng, 4, 6000), "dtype": rng.choice(("i8", "i8", "f32")), "low": 40,
                "high": rng.randint(200, 6144), "tuned": rng.random() < 0.5}
    if kind == "quantised":
        return {"kind": kind, "code": rng.choice(("k7r12", "k7r13", "k9r12", "k6r12")), "n": _log(rng, 500, 3000000),
                "L": 64 * rng.randint(2, 12), "v": 8 * rng.randint(5, 9), "ebn0": rng.uniform(1.0, 4.0)}
    if kind == "punctured":
        return {"kind": kind, "code": "k7r12", "n": _log(rng, 500, 1 << 20), "L": 64 * rng.randint(2, 12),
                "v": rng.randint(60, 90), "ebn0": rng.uniform(4.0, 6.0)}
    code = rng.choice(("k7r12", "k7r12", "k7r13", "k9r12", "k9r12", "k8r12", "k6r12", "k5r12", "k4r14", "k3r12"))
    k = CODES[code][0]
    dtype = rng.choice(("f32", "f32", "i8", "i8", "hard"))
    n = _log(rng, 100, 1 << (21 if k > 7 else 23))
    L = 8 * rng.randint(8, 128 if k < 8 else 48)
    v = rng.randint(4 * k, 8 * k)
    sub = dtype == "f32" and rng.random() < 0.15
    if n <= 2000 and rng.random() < 0.5 and not sub:
        L, v = 0, 0
    case = _stream("", code, n, dtype, L, v, terminated=rng.random() < 0.7, ebn0=rng.uniform(1.0, 6.0),
                   metric_bits=16 if dtype == "i8" and L <= 512 and rng.random() < 0.2 else 0,
                   f0=max(24, L // 16) if sub else 0, w=5 * k if sub else 0)
    del case["name"]
    return case


# ---------------------------------------------------------------- inputs
def _coded(k, gens, bits, terminated):
    """Coded bits of eq. (1), time-major: tap m of a generator multiplies in_{t-m}."""
    n = bits.numel()
    N = n + (k - 1 if terminated else 0)
    x = torch.zeros(N + k - 1, dtype=torch.uint8, device=bits.device)
    x[k - 1:k - 1 + n] = bits
    out = torch.zeros((N, len(gens)), dtype=torch.uint8, device=bits.device)
    for b, g in enumerate(gens):
        for m in range(k):
            if (g >> (k - 1 - m)) & 1:
                out[:, b] ^= x[k - 1 - m:k - 1 - m + N]
    return out


def _sigma(ebn0, rate):
    return math.sqrt(1.0 / (2.0 * rate * 10.0 ** (ebn0 / 10.0)))


def _llrs(code, n, terminated, ebn0, gen, rate=None, mask=None):
    """LLRs 2y/sigma^2 of a random message over BPSK and AWGN (FP32), and the int8 scale that maps a noiseless one to 8."""
    k, gens = CODES[code]
    sigma = _sigma(ebn0, rate or 1.0 / len(gens))
    bits = torch.randint(0, 2, (n,), dtype=torch.uint8, device="cuda", generator=gen)
    coded = _coded(k, gens, bits, terminated)
    if mask is not None:
        keep = torch.tensor(mask, dtype=torch.bool, device="cuda").repeat(coded.shape[0] // len(mask) + 1, 1)
        coded = coded[keep[:coded.shape[0]]]
    y = 1.0 - 2.0 * coded.reshape(-1).float()
    y += sigma * torch.randn(y.shape, device="cuda", generator=gen)
    return y * (2.0 / sigma ** 2), 4.0 * sigma ** 2


def _int8(llr, scale):
    return (llr * scale).round().clamp_(-127, 127).to(torch.int8)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _lengths(case):
    """Length, code and Eb/N0 of each frame: the traffic is the case's, the messages and the noise are the seed's."""
    r = np.random.default_rng(case["frames"])
    if case["kind"] == "serve":
        n = np.clip(np.round(r.lognormal(math.log(case["median"]), 1.0, case["frames"])), 40, 16384).astype(np.int64)
    else:
        n = r.integers(case["low"], case["high"] + 1, size=case["frames"])
    return n, r.integers(0, len(MIX), size=case["frames"]), r.uniform(1.0, 5.0, size=case["frames"])


def _frames(case, seed, dtype):
    """Terminated frames of mixed codes, one behind the other: their list, and the LLRs of all of them."""
    n, cid, ebn0 = _lengths(case)
    stages = n + np.array([CODES[MIX[c]][0] - 1 for c in cid])
    size = stages * np.array([len(CODES[MIX[c]][1]) for c in cid])
    off = np.cumsum(size) - size
    llr = torch.empty(int(size.sum()), dtype=torch.float32 if dtype == "f32" else torch.int8, device="cuda")
    g = _gen(seed)
    for c, code in enumerate(MIX):  # all frames of a code in one stream, cut apart: each is a message between known tails
        k, gens = CODES[code]
        mine = np.nonzero(cid == c)[0]
        if mine.size == 0:
            continue
        ends = np.cumsum(stages[mine])
        total = int(ends[-1])
        bits = torch.randint(0, 2, (total,), dtype=torch.uint8, device="cuda", generator=g)
        tail = (ends[:, None] - 1 - np.arange(k - 1)[None]).reshape(-1)
        bits[torch.from_numpy(tail).cuda()] = 0
        y = 1.0 - 2.0 * _coded(k, gens, bits, False).reshape(-1).float()
        sigma = torch.from_numpy(np.array([_sigma(e, 1.0 / len(gens)) for e in ebn0[mine]])).float().cuda()
        sigma = sigma.repeat_interleave(torch.from_numpy(size[mine]).cuda())
        y += sigma * torch.randn(y.shape, device="cuda", generator=g)
        y *= 2.0 / sigma ** 2
        y = y if dtype == "f32" else _int8(y, 4.0 * sigma ** 2)
        at = np.repeat(off[mine] - (np.cumsum(size[mine]) - size[mine]), size[mine]) + np.arange(int(size[mine].sum()))
        llr[torch.from_numpy(at).cuda()] = y
    return n, cid, off, llr


def _shapes(case):
    """(L, v, v1, waves) per code of a batch: as the autotuner picks them, or the library's defaults."""
    if case["kind"] == "serve" or case["tuned"]:
        return [(512, 35, -1, 1), (512, 35, -1, 1), (256, 64, -1, 1)]
    return None


def _serve_layout(n, off, llr_bytes):
    out_off = (llr_bytes + 63) // 64 * 64 + np.cumsum((n + 15) // 16 * 2) - (n + 15) // 16 * 2
    return out_off, int(out_off[-1] + (n[-1] + 15) // 16 * 2)


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind in ("batch", "serve"):
        n, cid, off, llr = _frames(case, seed, case.get("dtype", "i8"))
        state["codes"] = [vit.make_code(*CODES[c]) for c in MIX]
        state["tune"] = _shapes(case)
        if kind == "batch":
            bytes_ = (n + 7) // 8
            out_off = np.cumsum(bytes_) - bytes_
            fr = np.zeros(n.size, dtype=vit.FRAME_DTYPE)
            fr["code_id"], fr["terminated"], fr["n"], fr["llr_off"], fr["out_off"] = cid, 1, n, off, out_off
            state.update(frames=fr, llr=llr, out=torch.zeros(int(bytes_.sum()), dtype=torch.uint8, device="cuda"),
                         batch=vit.Batch())
            return state
        out_off, total = _serve_layout(n, off, llr.numel())
        host = torch.zeros(total, dtype=torch.uint8, pin_memory=True)
        host[:llr.numel()] = llr.view(torch.uint8).cpu()
        server = vit.Server(state["codes"], host, tune=state["tune"], llr_type=vit.VIT_LLR_I8, arena_bytes=32 << 20,
                            max_frames=4096, max_items=65536)
        req = server.requests(n.size)
        req["code_id"], req["terminated"], req["n"] = cid, 1, n
        req["llr"], req["out"], req["tag"] = host.data_ptr() + off, host.data_ptr() + out_off, np.arange(n.size)
        state.update(server=server, host=host, requests=req, results=host[int(out_off[0]):])
        return state
    k, gens = CODES[case["code"]]
    state["code"] = vit.make_code(k, gens)
    g = _gen(seed)
    if kind == "punctured":
        llr, scale = _llrs(case["code"], case["n"], True, case["ebn0"], g, rate=0.75, mask=RATE34)
        state["received"] = _int8(llr, scale)
    elif kind == "quantised":
        state["llr"], state["scale"] = _llrs(case["code"], case["n"], True, case["ebn0"], g)
    else:
        llr, scale = _llrs(case["code"], case["n"], case["terminated"], case["ebn0"], g)
        state["llr"] = llr if case["dtype"] == "f32" else _int8(llr, scale) if case["dtype"] == "i8" else (llr < 0).to(torch.uint8)
    return state


# ---------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "stream":
        return vit.decode(state["code"], state["llr"], case["n"], case["L"], case["v"], terminated=case["terminated"],
                          subframe_bits=case["f0"], subframe_overlap=case["w"], metric_bits=case["metric_bits"])
    if kind == "quantised":
        q = vit.quantize(state["llr"], state["scale"])
        return q, vit.decode(state["code"], q, case["n"], case["L"], case["v"])
    if kind == "punctured":
        full = vit.depuncture(state["received"], RATE34, case["n"] + state["code"].k - 1)
        return full, vit.decode(state["code"], full, case["n"], case["L"], case["v"])
    if kind == "batch":
        return state["batch"].decode(state["codes"], state["frames"], state["llr"], state["out"], tune=state["tune"])
    server, req = state["server"], state["requests"]
    sent = 0
    while sent < len(req):
        sent += server.submit(req[sent:])[1]
    server.drain()
    done = server.poll()
    if len(done) != len(req) or (done["status"] != vit.VIT_OK).any():
        raise RuntimeError("a request did not complete")
    return state["results"]


# ---------------------------------------------------------------- least work
def work(case):
    """LLRs read once and bits written once; two additions, a comparison and a selection per state and trellis stage."""
    kind = case["kind"]
    if kind in ("batch", "serve"):
        mean = {"batch": (case.get("low", 0) + case.get("high", 0)) / 2.0, "serve": 1.6 * case.get("median", 0.0)}[kind]
        width = 4 if case.get("dtype") == "f32" else 1
        per = [(len(CODES[c][1]) * width + 0.125, 4.0 * (1 << (CODES[c][0] - 1))) for c in MIX]
        return {"bytes": case["frames"] * mean * sum(p[0] for p in per) / 3, "flops": case["frames"] * mean * sum(p[1] for p in per) / 3}
    k, gens = CODES[case["code"]]
    n, beta = case["n"], len(gens)
    flops = 4.0 * (1 << (k - 1)) * n
    if kind == "quantised":
        return {"bytes": n * (5.0 * beta + 0.125), "flops": flops}
    if kind == "punctured":
        return {"bytes": n * (4.0 / 3.0 + beta + 0.125), "flops": flops}
    return {"bytes": n * (beta * (4 if case["dtype"] == "f32" else 1) + 0.125), "flops": flops}


# ---------------------------------------------------------------- exact results
def _viterbi(code, llr, base, s, e, cs, ce, known, zero):
    """Maximum-likelihood paths of windows [s, e) of one code's frames, metrics in 64 bits: their core bits, one row a window.
    llr: flat values; base: each window's frame; known / zero: windows that start / end in state 0."""
    k, gens = CODES[code]
    S, beta, dev = 1 << (k - 1), len(gens), llr.device
    idx = torch.arange(S, device=dev)
    pred = [((idx << 1) & (S - 1)) | j for j in (0, 1)]
    reg = [((idx >> (k - 2)) << (k - 1)) | p for p in pred]
    sign = []
    for r in reg:
        taps = torch.tensor([[bin(int(x) & g).count("1") & 1 for x in r.tolist()] for g in gens], device=dev)
        sign.append(1 - 2 * taps)  # beta x S
    M = e - s
    most = int(M.max())
    val = llr.to(torch.float64 if llr.is_floating_point() else torch.int64)
    metric = torch.zeros((M.numel(), S), dtype=val.dtype, device=dev)
    metric[known, 1:] = -(1 << 40)
    won = torch.empty((most, M.numel(), S), dtype=torch.bool, device=dev)
    for t in range(most):
        at = (base + (s + t).clamp(max=e - 1) * beta)
        x = [val[at + b][:, None] for b in range(beta)]
        c = []
        for j in (0, 1):
            d = x[0] * sign[j][0]
            for b in range(1, beta):
                d = d + x[b] * sign[j][b]
            c.append(metric[:, pred[j]] + d)
        won[t] = c[1] > c[0]
        metric = torch.where((t < M)[:, None], torch.maximum(c[0], c[1]), metric)
    state = torch.where(zero, torch.zeros_like(M), torch.max(metric, 1).indices)
    top = metric.max(1, keepdim=True).values
    state = torch.where(zero, state, torch.where(metric == top, idx[None], S).min(1).values)
    bits = torch.zeros((M.numel(), int((ce - cs).max())), dtype=torch.uint8, device=dev)
    rows = torch.arange(M.numel(), device=dev)
    for t in range(most - 1, -1, -1):
        live = t < M
        core = live & (s + t >= cs) & (s + t < ce)
        bits[rows[core], (s + t - cs)[core]] = (state >> (k - 2))[core].to(torch.uint8)
        odd = won[t][rows, state].long()
        state = torch.where(live, ((state << 1) & (S - 1)) | odd, state)
    return bits


def _exact(code, llr, bases, ns, terminated, L, v):
    """Blocked decode of frames of one code: a list of each frame's packed bytes."""
    k = CODES[code][0]
    w = []
    for f, (base, n) in enumerate(zip(bases, ns)):
        N = n + (k - 1 if terminated else 0)
        size, v1, v2 = (L, v // 2, v - v // 2) if L else (n, 0, N - n)
        cs = np.arange(0, n, size, dtype=np.int64)
        ce = np.minimum(cs + size, n)
        w.append(np.stack([np.full(cs.size, base), np.maximum(cs - v1, 0), np.minimum(ce + v2, N), cs, ce, np.full(cs.size, N)]))
    cols = torch.from_numpy(np.concatenate(w, 1)).to(llr.device)
    per = max(1, int(1.5e9 / ((1 << (k - 1)) * max(1, int((cols[2] - cols[1]).max())))))
    rows = []
    for a in range(0, cols.shape[1], per):
        base, s, e, cs, ce, N = cols[:, a:a + per]
        b = _viterbi(code, llr, base, s, e, cs, ce, s == 0, (e == N) if terminated else torch.zeros_like(e, dtype=torch.bool))
        keep = torch.arange(b.shape[1], device=llr.device)[None] < (ce - cs)[:, None]
        rows.append(b[keep])
    bits = torch.cat(rows)
    out, at = [], 0
    for n in ns:
        full = torch.zeros((n + 7) // 8 * 8, dtype=torch.uint8, device=llr.device)
        full[:n] = bits[at:at + n]
        out.append((full.view(-1, 8) << torch.arange(8, device=llr.device, dtype=torch.uint8)).sum(1, dtype=torch.uint8))
        at += n
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        if case["frames"] > 4096 or kind == "serve":
            return None
        n, cid, off, llr = _frames(case, seed, case["dtype"])
        shapes = _shapes(case) or [(256, _overlap(CODES[c][0]), -1, 1) for c in MIX]
        got = [None] * n.size
        for c, code in enumerate(MIX):
            mine = np.nonzero(cid == c)[0]
            if mine.size:
                for i, b in zip(mine, _exact(code, llr, off[mine], n[mine], True, shapes[c][0], shapes[c][1])):
                    got[i] = b
        return torch.cat(got)
    if case.get("f0"):
        return None
    g = _gen(seed)
    if kind == "punctured":
        llr, scale = _llrs(case["code"], case["n"], True, case["ebn0"], g, rate=0.75, mask=RATE34)
        N, beta = case["n"] + CODES[case["code"]][0] - 1, len(RATE34[0])
        keep = torch.tensor(RATE34, dtype=torch.bool, device="cuda").repeat(N // len(RATE34) + 1, 1)[:N]
        full = torch.zeros((N, beta), dtype=torch.int8, device="cuda")
        full[keep] = _int8(llr, scale)
        full = full.reshape(-1)
        return full, _exact(case["code"], full, [0], [case["n"]], True, case["L"], case["v"])[0]
    if kind == "quantised":
        llr, scale = _llrs(case["code"], case["n"], True, case["ebn0"], g)
        q = (llr * torch.tensor(scale, dtype=torch.float32, device="cuda")).round().clamp(-127, 127).to(torch.int8)
        return q, _exact(case["code"], q, [0], [case["n"]], True, case["L"], case["v"])[0]
    x = prepare(case, seed)["llr"]
    if case["dtype"] == "hard":
        x = (1 - 2 * (x != 0).to(torch.int8)).to(torch.int8)
    return _exact(case["code"], x, [0], [case["n"]], case["terminated"], case["L"], case["v"])[0]
