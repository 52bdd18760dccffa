"""Workloads of the decoder, as a program that uses it would run them.

Each case is one call (or one training step) through the public entry points
of paper_2011_13579_amd: one-call decodes of equal-length frames, plans over
batches of one or several codes, one long stream cut into windows, a stream
pushed in pieces, the quantiser, and the best-metric gradient.  Inputs are
BPSK soft values over AWGN (LLR = 2y/sigma^2; int8 values hold 32y rounded,
as the quantiser writes them), made on the GPU from a seed alone.

    listed()             the fixed cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs, plan and output buffers
    run(state)           one pass
    work(case)           bytes and operations one pass cannot do without
    exact(case, seed)    path metrics and gradients in 64 bits, without the
                         library
"""
import math

import numpy as np
import torch

import paper_2011_13579_amd as mv

CODES = {
    "k5": (5, ("23", "35")),
    "k7": (7, ("133", "171")),
    "k8": (8, ("247", "371")),
    "k9": (9, ("557", "663", "711")),
}
MIX = ("k5", "k7", "k9")  # the codes of a mixed batch
DEV = "cuda:0"


def code_of(name):
    K, gens = CODES[name]
    return mv.Code.from_octal(K, list(gens))


def taps_of(name):
    K, gens = CODES[name]
    return K, [int(g, 8) for g in gens]


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------
def listed():
    return [
        # one short frame: a control channel decoded as it arrives
        {"name": "frame_k7_f32", "kind": "uniform", "code": "k7", "dtype": "f32", "frames": 1,
         "n": 1024, "terminated": True, "db": 3.0},
        # a handful of odd-sized frames: one radio slot
        {"name": "slot_k7_i8", "kind": "uniform", "code": "k7", "dtype": "i8", "frames": 16,
         "n": 1001, "terminated": True, "db": 3.0},
        # the large batch of the repository's benchmark, int8 and float32
        {"name": "batch_k7_i8", "kind": "plan", "code": "k7", "dtype": "i8", "radix": 4,
         "frames": 4096, "n": 8192, "terminated": True, "db": 3.0},
        {"name": "batch_k7_f32", "kind": "plan", "code": "k7", "dtype": "f32", "radix": 2,
         "frames": 4096, "n": 8192, "terminated": True, "db": 3.0},
        # half-precision soft values, ragged sizes, free-ending frames
        {"name": "batch_k7_f16", "kind": "uniform", "code": "k7", "dtype": "f16", "frames": 999,
         "n": 3001, "terminated": False, "db": 4.0},
        # the code with the most states, medium batches
        {"name": "batch_k9_i8", "kind": "uniform", "code": "k9", "dtype": "i8", "frames": 512,
         "n": 4000, "terminated": True, "db": 2.0},
        # a recorded stream, decoded in one call with default options
        {"name": "stream_k7_i8", "kind": "stream", "code": "k7", "dtype": "i8", "n": 1 << 26,
         "chunk": 2048, "overlap": 64, "db": 4.0},
        # a live stream arriving in pieces
        {"name": "push_k7_i8", "kind": "push", "code": "k7", "dtype": "i8", "n": 1 << 18,
         "chunk": 2048, "overlap": 64, "radix": 4, "db": 4.0},
        # 10000 frames of three codes and lengths 64 to 16384, a tuned and
        # recorded plan; and an ordinary plan over a smaller float batch
        {"name": "mixed_i8", "kind": "mixed", "dtype": "i8", "frames": 10000, "n_min": 64,
         "n_max": 16384, "tuned": True},
        {"name": "mixed_f32", "kind": "mixed", "dtype": "f32", "frames": 1500, "n_min": 64,
         "n_max": 4096, "tuned": False},
        # one training step through the decoder: best metric and its gradient
        {"name": "backward_k7_f32", "kind": "backward", "code": "k7", "frames": 2048, "n": 1024,
         "db": 2.0},
        # float soft values of the large batch to int8
        {"name": "quantize", "kind": "quantize", "values": 4096 * 8198 * 2},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["uniform"] * 5 + ["plan"] * 2 + ["stream", "push", "mixed", "backward",
                                                        "quantize"])
    db = round(rng.uniform(1.5, 5.0), 2)
    if kind in ("uniform", "plan"):
        code = rng.choice(["k5", "k7", "k7", "k7", "k8", "k9"])
        states = 1 << (CODES[code][0] - 1)
        n = _log(rng, 64, 16384)
        # states x stages no more than the large batch's
        most = max(1, min(8192, (4096 * 8192 * 64) // (2 * states * (n + 8))))
        c = {"kind": kind, "code": code, "dtype": rng.choice(["f32", "i8", "i8", "f16"]),
             "frames": _log(rng, 1, most), "n": n, "terminated": rng.random() < 0.6, "db": db}
        if kind == "plan":
            packed = c["dtype"] == "i8" and code in ("k5", "k7")
            c["radix"] = rng.choice([0, 4]) if packed else rng.choice([0, 2])
        return c
    if kind == "stream":
        return {"kind": kind, "code": rng.choice(["k5", "k7", "k7"]),
                "dtype": rng.choice(["i8", "i8", "f32"]), "n": _log(rng, 1 << 14, 1 << 25) | 1,
                "chunk": rng.choice([1024, 2048, 4096]), "overlap": rng.choice([48, 64, 96]),
                "db": db}
    if kind == "push":
        return {"kind": kind, "code": "k7", "dtype": rng.choice(["i8", "f32"]),
                "n": _log(rng, 1 << 13, 1 << 20), "chunk": rng.choice([1024, 2048]),
                "overlap": 64, "radix": 0, "db": db}
    if kind == "mixed":
        return {"kind": kind, "dtype": rng.choice(["i8", "f32"]), "frames": _log(rng, 50, 4000),
                "n_min": 64, "n_max": _log(rng, 1024, 8192), "tuned": False}
    if kind == "backward":
        return {"kind": kind, "code": rng.choice(["k5", "k7", "k9"]), "frames": _log(rng, 4, 2048),
                "n": _log(rng, 64, 1024), "db": db}
    return {"kind": "quantize", "values": _log(rng, 1 << 10, 1 << 26) | 1}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1 + 7919 * int(seed))
    return g


def _encode(x, K, taps):
    """x: uint8 [..., S] inputs from state 0 -> coded uint8 [..., S, beta]."""
    S = x.shape[-1]
    xp = torch.nn.functional.pad(x, (K - 1, 0))
    out = torch.zeros(x.shape + (len(taps),), dtype=torch.uint8, device=x.device)
    for b, g in enumerate(taps):
        for k in range(K):  # tap k takes the input K-1-k stages back
            if (g >> k) & 1:
                out[..., b] ^= xp[..., k:k + S]
    return out


def _channel(coded, db, beta, gen, dtype):
    """Soft values of the coded bits; db: a number or a tensor like coded."""
    db = torch.as_tensor(db, dtype=torch.float32, device=coded.device)
    sigma2 = (beta / 2.0) * torch.pow(10.0, -db / 10.0)
    y = torch.randn(coded.shape, generator=gen, device=coded.device)
    y.mul_(torch.sqrt(sigma2)).add_(1.0).sub_(coded, alpha=2.0)
    if dtype == "i8":
        return torch.clamp(torch.round(32.0 * y), -127, 127).to(torch.int8)
    llr = y.mul_(2.0 / sigma2)
    return llr.half() if dtype == "f16" else llr


def _uniform_llr(case, seed, dtype):
    K, taps = taps_of(case["code"])
    gen = _gen(seed)
    F, n = case["frames"], case["n"]
    term = case.get("terminated", True)
    S = n + (K - 1 if term else 0)
    x = torch.zeros((F, S), dtype=torch.uint8, device=DEV)
    x[:, :n] = torch.randint(0, 2, (F, n), generator=gen, device=DEV, dtype=torch.uint8)
    return _channel(_encode(x, K, taps), case["db"], len(taps), gen, dtype).reshape(F, -1)


def _stream_llr(case, seed):
    K, taps = taps_of(case["code"])
    gen = _gen(seed)
    x = torch.randint(0, 2, (case["n"],), generator=gen, device=DEV, dtype=torch.uint8)
    return _channel(_encode(x, K, taps), case["db"], len(taps), gen, case["dtype"]).reshape(-1)


def _mixed_frames(case):
    """Frames of the mixed batch (host): per frame code index, length, dB, and
    the frame table; soft values are laid out code by code.  The frames belong
    to the case (a plan describes them), the soft values to the seed."""
    rng = np.random.default_rng(1000003 * case["frames"] + case["n_max"])
    F = case["frames"]
    n = np.rint(np.exp(rng.uniform(math.log(case["n_min"]), math.log(case["n_max"]), F)))
    n = n.astype(np.int64)
    ci = rng.integers(0, len(MIX), F)
    db = rng.uniform(1.0, 5.0, F)
    fr = np.zeros(F, mv.FRAME_DTYPE)
    pos = 0
    for c, name in enumerate(MIX):
        K, taps = taps_of(name)
        idx = np.flatnonzero(ci == c)
        S = n[idx] + K - 1
        fr["llr_offset"][idx] = pos + np.concatenate([[0], np.cumsum(S)[:-1]]) * len(taps) \
            if len(idx) else 0
        fr["n_stages"][idx] = S
        pos += int(S.sum()) * len(taps)
    words = (n + 31) // 32
    fr["bit_offset"] = np.concatenate([[0], np.cumsum(words)[:-1]]) * 32
    fr["n_out"] = n
    fr["code"] = ci
    fr["flags"] = 3  # known start, zero end
    return ci, n, db, fr


def _mixed_llr(case, seed, ci, n, db, dtype):
    gen = _gen(seed)
    parts = []
    for c, name in enumerate(MIX):
        K, taps = taps_of(name)
        idx = np.flatnonzero(ci == c)
        S = torch.as_tensor(n[idx] + K - 1, device=DEV)
        total = int((n[idx] + K - 1).sum())
        # the frames back to back: their zero tails bring the encoder to state 0
        x = torch.randint(0, 2, (total,), generator=gen, device=DEV, dtype=torch.uint8)
        ends = torch.cumsum(S, 0)
        for k in range(1, K):
            x[ends - k] = 0
        d = torch.repeat_interleave(torch.as_tensor(db[idx], dtype=torch.float32, device=DEV), S)
        parts.append(_channel(_encode(x, K, taps), d[:, None], len(taps), gen, dtype).reshape(-1))
    return torch.cat(parts)


# --------------------------------------------------------------------------
# the calls
# --------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case}
    if kind == "uniform":
        st["code"] = code_of(case["code"])
        st["llr"] = _uniform_llr(case, seed, case["dtype"])
    elif kind == "plan":
        code = code_of(case["code"])
        st["llr"] = _uniform_llr(case, seed, case["dtype"])
        st["plan"] = mv.Plan([code], mv.uniform_frames(code, case["frames"], case["n"],
                                                       case["terminated"]),
                             case["dtype"], case["radix"])
        st["out"] = st["plan"].empty_outputs(DEV)
    elif kind == "stream":
        st["code"] = code_of(case["code"])
        st["llr"] = _stream_llr(case, seed)
    elif kind == "push":
        st["llr"] = _stream_llr(case, seed)
        st["dec"] = mv.StreamDecoder(code_of(case["code"]), case["dtype"], case["chunk"],
                                     case["overlap"], max_push_stages=case["n"],
                                     radix=case["radix"])
    elif kind == "mixed":
        ci, n, db, fr = _mixed_frames(case)
        st["llr"] = _mixed_llr(case, seed, ci, n, db, case["dtype"])
        st["plan"] = mv.Plan([code_of(c) for c in MIX], fr, case["dtype"],
                             autotune=case["tuned"], graph=case["tuned"])
        st["out"] = st["plan"].empty_outputs(DEV)
    elif kind == "backward":
        st["code"] = code_of(case["code"])
        st["llr"] = _uniform_llr(case, seed, "f32").requires_grad_(True)
        st["g"] = torch.randn(case["frames"], generator=_gen(seed + 500009), device=DEV)
    else:
        st["x"] = torch.randn(case["values"], generator=_gen(seed), device=DEV).mul_(8.0)
        st["q"] = torch.empty(case["values"], dtype=torch.int8, device=DEV)
    return st


def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "uniform":
        bits, metric = mv.decode(st["llr"], st["code"], case["n"], case["terminated"])
        return {"bits": bits, "metric": metric}
    if kind in ("plan", "mixed"):
        bits, metric, end = st["plan"].decode(st["llr"], *st["out"])
        return {"bits": bits, "metric": metric, "end": end}
    if kind == "stream":
        return {"bits": mv.decode_stream(st["llr"], st["code"], case["n"], case["chunk"],
                                         case["overlap"])}
    if kind == "push":
        words, nb = st["dec"].push(st["llr"])
        return {"bits": words, "count": nb}
    if kind == "backward":
        bits, metric = mv.ViterbiDecode.apply(st["llr"], st["code"], case["n"])
        (grad,) = torch.autograd.grad(metric, st["llr"], st["g"])
        return {"bits": bits, "metric": metric.detach(), "grad": grad}
    return {"q": mv.quantize_i8(st["x"], 4.0, out=st["q"])}


def work(case):
    """Soft values read once, bits (and gradients) written once; two additions
    and one selection per state and stage."""
    kind = case["kind"]
    if kind == "quantize":
        return {"bytes": 5 * case["values"], "flops": 2 * case["values"]}
    size = {"f32": 4, "f16": 2, "i8": 1}[case.get("dtype", "f32")]
    if kind == "mixed":
        # expected stages of log-uniform lengths
        mean = (case["n_max"] - case["n_min"]) / math.log(case["n_max"] / case["n_min"])
        nb = fl = 0.0
        for name in MIX:
            K, gens = CODES[name]
            stages = case["frames"] / len(MIX) * (mean + K - 1)
            nb += stages * (size * len(gens) + 1 / 8)
            fl += stages * 3 * (1 << (K - 1))
        return {"bytes": nb, "flops": fl}
    K, gens = CODES[case["code"]]
    stages = case["n"] * case.get("frames", 1)
    if case.get("terminated", kind == "backward"):
        stages += case["frames"] * (K - 1)
    nb = stages * (size * len(gens) + 1 / 8)
    if kind == "backward":
        nb += stages * 4 * len(gens)
    return {"bytes": nb, "flops": stages * 3 * (1 << (K - 1))}


# --------------------------------------------------------------------------
# the same values in 64 bits, by plain torch
# --------------------------------------------------------------------------
def _trellis(name):
    """Even predecessor of each state and the +-1 outputs of both branches."""
    K, taps = taps_of(name)
    ns = 1 << (K - 1)
    sign = torch.zeros((2, ns, len(taps)), dtype=torch.float64)
    for d in range(2):
        for j in range(ns):
            i = ((j << 1) & (ns - 1)) | d
            reg = ((j >> (K - 2)) << (K - 1)) | i
            for b, g in enumerate(taps):
                sign[d, j, b] = -1.0 if bin(g & reg).count("1") & 1 else 1.0
    even = torch.tensor([(j << 1) & (ns - 1) for j in range(ns)])
    return K, ns, even.to(DEV), sign.to(DEV)


def _best(name, llr, keep=False):
    """Path metrics [F, states] after llr [F, S, beta] from state 0, and the
    decisions of every stage when keep is set."""
    K, ns, even, sign = _trellis(name)
    F, S, _ = llr.shape
    pm = torch.full((F, ns), -math.inf, dtype=torch.float64, device=DEV)
    pm[:, 0] = 0.0
    dec = torch.zeros((S, F, ns), dtype=torch.bool, device=DEV) if keep else None
    s0, odd = sign[0].t().contiguous(), even + 1
    for t in range(S):
        m = llr[:, t].double() @ s0  # the odd predecessor's branch is its negative
        a, b = pm[:, even] + m, pm[:, odd] - m
        if keep:
            dec[t] = b > a
        pm = torch.maximum(a, b)
    return pm, dec


def exact(case, seed):
    kind = case["kind"]
    if kind in ("uniform", "plan"):
        if case["n"] > 9000:
            return None
        K, taps = taps_of(case["code"])
        llr = _uniform_llr(case, seed, case["dtype"])
        pm, _ = _best(case["code"], llr.view(case["frames"], -1, len(taps)))
        m = pm[:, 0] if case["terminated"] else pm.max(1).values
        m = m.round().to(torch.int64) if case["dtype"] == "i8" else m
        out = {"bits": None, "metric": m}
        if kind == "plan":
            out["end"] = None
        return out
    if kind == "mixed" and case["n_max"] <= 4096:
        ci, n, db, fr = _mixed_frames(case)
        llr = _mixed_llr(case, seed, ci, n, db, case["dtype"])
        metric = torch.zeros(case["frames"], dtype=torch.float64, device=DEV)
        for c, name in enumerate(MIX):
            K, ns, even, sign = _trellis(name)
            beta, s0 = sign.shape[2], sign[0].t().contiguous()
            idx = np.flatnonzero(ci == c)
            idx = idx[np.argsort(-fr["n_stages"][idx].astype(np.int64), kind="stable")]
            S = fr["n_stages"][idx].astype(np.int64)
            off = torch.as_tensor(fr["llr_offset"][idx], device=DEV)
            col = torch.arange(beta, device=DEV)
            where = torch.as_tensor(idx, device=DEV)
            pm = torch.full((len(idx), ns), -math.inf, dtype=torch.float64, device=DEV)
            pm[:, 0] = 0.0
            for t in range(int(S.max()) if len(S) else 0):
                live = int(np.searchsorted(-S, -t, side="left"))  # frames with S > t
                m = llr[(off[:live] + t * beta)[:, None] + col].double() @ s0
                p = torch.maximum(pm[:live, even] + m, pm[:live, even + 1] - m)
                done = int(np.searchsorted(-S, -(t + 1), side="left"))
                if done < live:
                    metric[where[done:live]] = p[done:, 0]
                pm = p[:done] if done else p
        m = metric.round().to(torch.int64) if case["dtype"] == "i8" else metric
        return {"bits": None, "metric": m, "end": None}
    if kind == "backward":
        K, taps = taps_of(case["code"])
        F, n = case["frames"], case["n"]
        llr = _uniform_llr(case, seed, "f32").view(F, -1, len(taps))
        if F * llr.shape[1] << (K - 1) > 1 << 30:
            return None
        g = torch.randn(F, generator=_gen(seed + 500009), device=DEV).double()
        pm, dec = _best(case["code"], llr, keep=True)
        _, ns, even, sign = _trellis(case["code"])
        grad = torch.zeros(llr.shape, dtype=torch.float64, device=DEV)
        j = torch.zeros(F, dtype=torch.int64, device=DEV)
        for t in range(llr.shape[1] - 1, -1, -1):
            d = dec[t].gather(1, j[:, None])[:, 0].long()
            grad[:, t] = sign[d, j] * g[:, None]
            j = even[j] + d
        return {"bits": None, "metric": pm[:, 0], "grad": grad.view(F, -1)}
    return None
