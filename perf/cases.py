"""The codec's work as user programs call it, one case per call pattern.

A case names a direction (encode or decode), a codec (the Huffman codec or
PivCo-Golomb), how the data is cut (streams, bytes, block size), where the
symbols come from, the stream options (v1 or v2 trees, raw bitmaps, rANS or
tANS nodes) and the entry point: ``plan`` (a batch plan replayed per step),
``batch`` (``pivco_decode_batch`` on streams that are new to the library),
``single`` (``pivco_decode`` / ``pivco_encode``, the synchronous calls) or
``async`` (``pivco_encode_async``, one call per stream on one HIP stream).

Sizes and the distributions' parameters belong to the case; a seed draws the
symbols (and which ids the Zipf ranks map to).
"""
import math

import numpy as np
import torch

from paper_2606_05765_amd import pivco as P

KiB, MiB = 1 << 10, 1 << 20

_DEFAULTS = {"codec": "huffman", "streams": 1, "lo": 0, "source": "geometric", "param": 0.8,
             "ans": 0, "flat": False}


def _case(name, op, api, n, block, **kw):
    c = dict(_DEFAULTS, op=op, api=api, n=n, block=block)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one page of text-like bytes, the caller waits for it
        _case("decode_4k", "decode", "single", 4 * KiB + 1, 64 * KiB, source="zipf", param=1.1),
        # one 1 MiB block replayed from a plan: the latency of a single block
        _case("decode_block_1m", "decode", "plan", MiB, MiB),
        # one admission round of a decode server: 16 requests of 16 KiB - 64 MiB
        # in blocks of 1 MiB, new to the library, skewed nodes as tANS
        _case("decode_requests_tans", "decode", "batch", 64 * MiB, MiB, streams=16, lo=16 * KiB,
              source="mixed", param=0, ans=3),
        # the benchmark's default: 4096 independent blocks of 4 KiB - 4 MiB
        _case("decode_mix4096", "decode", "plan", 4 * MiB, 0, streams=4096, lo=4 * KiB,
              source="mixed", param=0, ans=1),
        # a large text-like buffer in 64 KiB blocks, flat-subtree trees
        _case("decode_zipf256m_v2", "decode", "plan", 256 * MiB, 64 * KiB, source="zipf", param=1.1,
              flat=True),
        # a large, very skewed buffer in 128 KiB blocks, skewed nodes as rANS
        _case("decode_skew256m_rans", "decode", "plan", 256 * MiB, 128 * KiB, source="skew", param=0.9,
              ans=1),
        # the smallest encode of use: one ragged block, the caller waits for the length
        _case("encode_64k", "encode", "single", 64 * KiB - 37, 64 * KiB, source="zipf", param=1.1),
        # a large buffer in one call
        _case("encode_zipf256m", "encode", "async", 256 * MiB, 64 * KiB, source="zipf", param=1.1),
        # many independent blocks of all sizes, one call each on one stream
        _case("encode_mix256_rans", "encode", "async", 4 * MiB, 0, streams=256, lo=4 * KiB,
              source="mixed", param=0, ans=1),
        # a skewed buffer with a ragged tail, flat-subtree trees, skewed nodes as tANS
        _case("encode_skew64m_tans_v2", "encode", "async", 64 * MiB + 12345, 128 * KiB, source="skew",
              param=0.9, ans=3, flat=True),
        # unary-coded small values (mean code length 2), both directions
        _case("golomb_decode_64m", "decode", "single", 64 * MiB, 64 * KiB, codec="golomb", param=0.5),
        _case("golomb_encode_64m", "encode", "single", 64 * MiB, 64 * KiB, codec="golomb", param=0.5),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["decode", "encode"])
    if rng.random() < 0.15:
        return _case(None, op, "single", _log_uniform(rng, 4 * KiB, 64 * MiB),
                     _log_uniform(rng, 4 * KiB, MiB), codec="golomb", param=round(rng.uniform(0.2, 0.8), 3))
    ans = rng.choice([0, 1, 3])
    flat = rng.random() < 0.4
    if rng.random() < 0.35:     # independent streams of mixed distributions
        hi = _log_uniform(rng, 64 * KiB, 4 * MiB)
        return _case(None, op, "async" if op == "encode" else rng.choice(["plan", "batch"]), hi,
                     rng.choice([0, _log_uniform(rng, 16 * KiB, MiB)]), streams=_log_uniform(rng, 4, 256),
                     lo=4 * KiB, source="mixed", param=0, ans=ans, flat=flat)
    source = rng.choice(["geometric", "zipf", "uniform", "skew"])
    param = {"geometric": round(rng.uniform(0.5, 0.95), 3), "zipf": round(rng.uniform(0.8, 1.5), 3),
             "uniform": rng.randint(2, 256), "skew": round(rng.uniform(0.75, 0.97), 3)}[source]
    return _case(None, op, rng.choice(["single", "async"] if op == "encode" else ["single", "plan", "batch"]),
                 _log_uniform(rng, 4 * KiB, 256 * MiB), _log_uniform(rng, 4 * KiB, 4 * MiB),
                 source=source, param=param, ans=ans, flat=flat)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _shapes(case):
    """(bytes, block size, source, parameter) of every stream; the same for
    every seed."""
    if case["streams"] == 1:
        return [(case["n"], case["block"] or case["n"], case["source"], case["param"])]
    rs = np.random.RandomState(4096 + case["streams"])
    out = []
    for _ in range(case["streams"]):
        n = int(round(math.exp(rs.uniform(math.log(case["lo"]), math.log(case["n"])))))
        source = ("geometric", "zipf", "uniform")[rs.randint(3)]
        param = {"geometric": rs.uniform(0.5, 0.95), "zipf": rs.uniform(0.8, 1.5),
                 "uniform": rs.randint(2, 257)}[source]
        out.append((n, case["block"] or n, source, param))
    return out


def _probabilities(source, param, rs=None):
    p = np.zeros(256)
    if source == "geometric":
        p[:] = float(param) ** np.arange(256)
    elif source == "zipf":
        q = np.arange(1, 257, dtype=np.float64) ** -float(param)
        p[rs.permutation(256) if rs is not None else np.arange(256)] = q
    elif source == "uniform":
        p[:int(param)] = 1.0
    else:                       # skew: one symbol holds most of the mass
        t = 0.7 ** np.arange(1, 256)
        p[0] = float(param)
        p[1:] = (1.0 - float(param)) * t / t.sum()
    return p / p.sum()


def _inputs(case, seed):
    """Every stream's symbols (uint8, on the GPU), by inverse CDF."""
    rs = np.random.RandomState(seed % (1 << 32))
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    shapes = _shapes(case)
    cdf = np.stack([np.cumsum(_probabilities(s, v, rs))[:255] for _, _, s, v in shapes])
    cdf = torch.from_numpy(cdf.astype(np.float32)).cuda()
    out = []
    for i, (n, _, _, _) in enumerate(shapes):
        x = torch.empty(n, dtype=torch.uint8, device="cuda")
        for a in range(0, n, 32 * MiB):
            u = torch.rand(min(32 * MiB, n - a), generator=g, device="cuda")
            x[a:a + u.numel()] = torch.searchsorted(cdf[i], u, right=True, out_int32=True)
        out.append(x)
    return out


def _rows(sizes):
    """Rows of one buffer, each at a multiple of 256 bytes: (offsets, total)."""
    offs, at = [], 0
    for n in sizes:
        offs.append(at)
        at += -(-n // 256) * 256
    return offs, max(at, 256)


def _buffer(sizes):
    offs, total = _rows(sizes)
    buf = torch.zeros(total, dtype=torch.uint8, device="cuda")
    return buf, [buf[o:o + n] for o, n in zip(offs, sizes)]


def _options(case):
    return {"ans_mode": case["ans"], "flat": case["flat"]}


def _encoder(case, xs):
    """What a program that encodes keeps: streams' buffers, lengths, statuses
    and one workspace."""
    o = _options(case)
    blocks = [b for _, b, _, _ in _shapes(case)]
    buf, outs = _buffer([P.pivco_encode_bound(x.numel(), b, **o) for x, b in zip(xs, blocks)])
    ws = max(P.pivco_encode_workspace(x.numel(), b, **o) for x, b in zip(xs, blocks))
    return {"xs": xs, "blocks": blocks, "options": o, "buf": buf, "outs": outs,
            "lens": torch.zeros(len(xs), dtype=torch.int64, device="cuda"),
            "status": torch.zeros(len(xs), dtype=torch.int32, device="cuda"),
            "ws": torch.empty(max(ws, 256), dtype=torch.uint8, device="cuda")}


def _encode_all(e):
    for i, x in enumerate(e["xs"]):
        P.pivco_encode_async(x, e["outs"][i], e["lens"][i:i + 1], e["status"][i:i + 1], e["ws"],
                             e["blocks"][i], **e["options"])


def prepare(case, seed):
    case = dict(_DEFAULTS, **case)
    xs = _inputs(case, seed)
    state = {"case": case}
    if case["codec"] == "golomb":
        if case["op"] == "encode":
            state["x"] = xs[0]
            state["buf"], _ = _buffer([int(P.lib().pivco_golomb_encode_bound(xs[0].numel(), case["block"]))])
        else:
            state["streams"] = [P.pivco_golomb_encode(xs[0], case["block"])]
            state["out"] = torch.empty_like(xs[0])
        return state
    if case["ans"] == 3:        # the library copies its tANS tables on their first use
        P.pivco_encode(xs[0][:256], 256, ans_mode=3)
    if case["op"] == "encode":
        state.update(_encoder(case, xs))
        return state
    e = _encoder(case, xs)
    _encode_all(e)
    state["streams"] = [o[:n].clone() for o, n in zip(e["outs"], e["lens"].cpu().tolist())]
    state["buf"], state["outs"] = _buffer([x.numel() for x in xs])
    del e, xs
    state["ws"] = P.Workspace(P.pivco_decode_workspace(state["streams"], state["outs"]))
    if case["api"] == "plan":
        state["plan"] = P.BatchPlan(state["streams"], state["outs"], ws=state["ws"])
    return state


def _collect(state, stream):
    """A caller that gathers streams in a buffer of its own."""
    state["buf"][:stream.numel()].copy_(stream)
    return {"out": state["buf"], "len": stream.numel()}


def run(state):
    case = state["case"]
    if case["codec"] == "golomb":
        if case["op"] == "encode":
            return _collect(state, P.pivco_golomb_encode(state["x"], case["block"]))
        outs, status = P.pivco_golomb_decode(state["streams"], [state["out"]])
        return {"out": outs[0], "status": status}
    if case["op"] == "encode":
        if case["api"] == "single":
            return _collect(state, P.pivco_encode(state["xs"][0], state["blocks"][0], **state["options"]))
        _encode_all(state)
        return {"out": state["buf"], "lens": state["lens"], "status": state["status"]}
    if case["api"] == "plan":
        state["plan"].launch()
        return {"out": state["buf"], "status": state["plan"].status}
    if case["api"] == "single":
        _, status = P.pivco_decode(state["streams"][0], state["outs"][0], ws=state["ws"])
    else:
        _, status = P.pivco_decode_batch(state["streams"], state["outs"], ws=state["ws"])
    return {"out": state["buf"], "status": status}


def work(case):
    """Symbols once and coded bytes once.  The coded bytes are the symbols'
    entropy (for Golomb the mean unary length) and, per block, the header's
    128 bytes of code lengths and 2 bytes of count per internal node."""
    case = dict(_DEFAULTS, **case)
    total = 0.0
    for n, block, source, param in _shapes(case):
        p = _probabilities(source, param)
        if case["codec"] == "golomb":
            total += n * (1.0 + float((p * np.arange(1, 257)).sum()) / 8)
        else:
            q = p[p > 0]
            present = int((q * min(n, block) >= 1).sum())
            total += n * (1.0 - float((q * np.log2(q)).sum()) / 8)
            total += -(-n // block) * (136 + 2 * max(present - 1, 0))
    return {"bytes": total, "flops": 0}


def exact(case, seed):
    """A decode returns the symbols that were encoded."""
    case = dict(_DEFAULTS, **case)
    if case["op"] == "encode":
        return None
    xs = _inputs(case, seed)
    if case["codec"] == "golomb":
        return {"out": xs[0], "status": np.zeros(1, np.int32)}
    buf, rows = _buffer([x.numel() for x in xs])
    for row, x in zip(rows, xs):
        row.copy_(x)
    if case["api"] == "plan":
        return {"out": buf, "status": torch.zeros(len(xs), dtype=torch.int32)}
    return {"out": buf, "status": np.zeros(len(xs), np.int32)}
