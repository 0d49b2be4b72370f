"""The work a user of the trace-monitoring library has it do, as measured cases.

One pass is one call of a public entry point on a device-resident trace:
Context.eval_into (one trace), Context.eval_batch_into (many traces in one
call), or StreamGroup.push_chunks followed by StreamGroup.read (online
monitoring).  The traces are those of the workloads module (the paper's three
case studies, the two-level user/request trace, the long single trace, the
batch and the log streams), drawn on the device from the seed alone; the
layouts and properties are that module's own.

Every output is a whole number (verdict codes, counts, sizes, packed keys,
positions), so outputs are compared for equality.
"""
import math

import numpy as np
import torch

from paper_1411_2239_amd import lib, workloads

DEV = "cuda:0"


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def listed():
    return [
        # Case study 1 (sockets of a web server, 12-byte records, two
        # properties, truth values only).  16,384 events is the paper's
        # smallest trace: launches and host time count, not bandwidth.
        {"name": "sockets_16k", "kind": "sockets", "n": 16_384, "keys": 1000, "outputs": "root"},
        # the same at the size the latency of one call is quoted on
        {"name": "sockets_100k", "kind": "sockets", "n": 100_000, "keys": 1000, "outputs": "root"},
        # the paper's largest trace
        {"name": "sockets_8m", "kind": "sockets", "n": 8_388_608, "keys": 1000, "outputs": "root"},
        # Two nested quantifiers, an odd ordinary size, everything asked for:
        # which requests and which users fail, with their keys and counts
        {"name": "users_1m_all", "kind": "users", "n": 1_000_003, "users": 1000, "outputs": "all"},
        # the same shape at the headline size, truth values only
        {"name": "users_10m", "kind": "users", "n": 10_000_000, "users": 10_000, "outputs": "root"},
        # Case study 2 (cloud storage): propositions computed from record data
        {"name": "chunks_10m", "kind": "chunks", "n": 10_000_000, "users": 10_000, "preds": 2, "outputs": "instances"},
        # online verdicts of a recorded trace: the first conclusive prefix of
        # every instance and the verdict after every event
        {"name": "timeline_10m", "kind": "timeline", "n": 10_000_000, "keys": 100_000, "events": True},
        # Case study 3 (proxy cache): cache events of a video join all its
        # requests; the failing videos and requests are asked for
        {"name": "proxy_10m", "kind": "proxy", "n": 10_000_000, "videos": 4096, "wide": False, "outputs": "all"},
        # the same with raw 32-bit ids (ranked before they are packed), an
        # odd size, the values of every video's and request's ids
        {"name": "proxy_wide_1m", "kind": "proxy", "n": 1_500_007, "videos": 4096, "wide": True, "outputs": "all"},
        # one long trace, a million 32-bit keys, monitors of 3, 8 and 16 states,
        # the verdict of every instance
        {"name": "large_500m", "kind": "large", "n": 500_000_000, "keys": 1_000_000, "outputs": "instances"},
        # 4,096 independent traces of 1 k to 1 M events in one call, 16 properties
        {"name": "batch_4096", "kind": "batch", "traces": 4096, "min_len": 1000, "max_len": 1_000_000, "props": 16},
        # online monitoring: one push of 16 log chunks (4 k to 256 k events) of
        # 64 streams, and the truth value of every stream after it
        {"name": "serving_16", "kind": "serving", "streams": 64, "chunks": 16, "bindings": 100_000},
    ]


def _log_int(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi], odd half of the time."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        v |= 1
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["sockets", "users", "chunks", "timeline", "proxy", "large", "batch", "serving"])
    if kind == "sockets":
        return {"kind": kind, "n": _log_int(rng, 1000, 8_388_608), "keys": _log_int(rng, 8, 4000),
                "outputs": rng.choice(["root", "instances"])}
    if kind == "users":
        n = _log_int(rng, 20_000, 20_000_000)
        return {"kind": kind, "n": n, "users": _log_int(rng, 10, max(20, n // 1000)),
                "outputs": rng.choice(["root", "instances", "all"])}
    if kind == "chunks":
        return {"kind": kind, "n": _log_int(rng, 10_000, 20_000_000), "users": _log_int(rng, 50, 16_000),
                "preds": rng.choice([1, 2]), "outputs": rng.choice(["root", "instances"])}
    if kind == "timeline":
        return {"kind": kind, "n": _log_int(rng, 10_000, 16_000_000), "keys": _log_int(rng, 100, 200_000),
                "events": rng.choice([True, False])}
    if kind == "proxy":
        return {"kind": kind, "n": _log_int(rng, 50_000, 10_000_000), "videos": _log_int(rng, 16, 4096),
                "wide": rng.choice([True, False]), "outputs": rng.choice(["root", "all"])}
    if kind == "large":
        return {"kind": kind, "n": _log_int(rng, 30_000_000, 300_000_000), "keys": _log_int(rng, 10_000, 1_000_000),
                "outputs": rng.choice(["root", "instances"])}
    if kind == "batch":
        return {"kind": kind, "traces": _log_int(rng, 8, 2048), "min_len": 1000,
                "max_len": _log_int(rng, 4000, 500_000), "props": rng.choice([1, 4, 16])}
    return {"kind": kind, "streams": rng.choice([8, 64]), "chunks": _log_int(rng, 1, 128), "bindings": 100_000}


# --------------------------------------------------------------------------
# traces, drawn on the device
# --------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, n, dtype=torch.float64):
    return torch.rand(n, generator=g, device=DEV, dtype=dtype)


def _zipf(g, n, ranks, s):
    """n ranks in [0, ranks), P(r) proportional to (r + 1)^-s."""
    w = np.arange(1, ranks + 1, dtype=np.float64) ** (-s)
    cdf = torch.from_numpy(np.cumsum(w) / w.sum()).to(DEV)
    return torch.clamp(torch.searchsorted(cdf, _rand(g, n), right=True), max=ranks - 1)


def _perm(g, n):
    return torch.randperm(n, generator=g, device=DEV)


def _distinct32(ranks, seed):
    """Distinct, random-looking 32-bit values of ranks (an odd multiplier is a bijection)."""
    return (ranks * 0x9E3779B1 + (int(seed) * 40_503 + 12_345)) & 0xFFFFFFFF


def _records16(typ, k0, k1=None):
    n = typ.numel()
    rec = torch.zeros((n, 4), dtype=torch.int32, device=DEV)
    rec[:, 0] = torch.arange(n, device=DEV, dtype=torch.int32)
    rec[:, 1] = typ.to(torch.int32)
    rec[:, 2] = k0.to(torch.int64).to(torch.int32)
    if k1 is not None:
        rec[:, 3] = k1.to(torch.int64).to(torch.int32)
    return rec.view(torch.uint8).reshape(-1)


def _bits(n):
    return max(1, int(n - 1).bit_length())


def _choice(g, n, p):
    cdf = torch.from_numpy(np.cumsum(np.asarray(p, dtype=np.float64))[:-1].copy()).to(DEV)
    return torch.searchsorted(cdf, _rand(g, n), right=True)


def _sockets(c, seed):
    """12-byte records {ts, type u16, pad u16, socket}; 0.1 / 0.5 / 0.35 / 0.05
    open / receive / respond / close, sockets uniform."""
    g, n = _gen(seed), c["n"]
    rec = torch.zeros((n, 3), dtype=torch.int32, device=DEV)
    rec[:, 0] = torch.arange(n, device=DEV, dtype=torch.int32)
    rec[:, 1] = _choice(g, n, [0.1, 0.5, 0.35, 0.05]).to(torch.int32)
    rec[:, 2] = torch.randint(0, c["keys"], (n,), generator=g, device=DEV, dtype=torch.int32)
    lay = workloads.socket_layout()
    lay.key_bits = [_bits(c["keys"])]
    return lay, workloads.socket_properties(), rec.view(torch.uint8).reshape(-1)


def _users(c, seed):
    """Requests of users with Zipf(1.2) shares: issue, a geometric number of
    progress events, done with probability 0.95; in time order, topped up with
    other events on existing requests."""
    g, n, users = _gen(seed), c["n"], c["users"]
    want = max(users, int(n / 2.95))
    w = np.arange(1, users + 1, dtype=np.float64) ** -1.2
    per_user = np.maximum(1, np.round(want * w / w.sum())).astype(np.int64)
    total_req = int(per_user.sum())
    req_user = torch.repeat_interleave(_perm(g, users), torch.from_numpy(per_user).to(DEV))
    req_id = _perm(g, total_req)
    # requests in random order, so that those that no longer fit belong to any user
    order = _perm(g, total_req)
    req_user, req_id = req_user[order], req_id[order]
    prog = torch.floor(torch.log2(1.0 / torch.clamp(_rand(g, total_req), min=1e-9))).to(torch.int64)
    done = _rand(g, total_req) < 0.95
    per_req = 1 + prog + done.to(torch.int64)
    keep = int((torch.cumsum(per_req, 0) <= n).sum().item())
    req_user, req_id, done, per_req = req_user[:keep], req_id[:keep], done[:keep], per_req[:keep]
    first = torch.cumsum(per_req, 0) - per_req
    ev = torch.repeat_interleave(torch.arange(keep, device=DEV), per_req)
    total = ev.numel()
    pos = torch.arange(total, device=DEV) - first[ev]
    typ = (pos > 0).to(torch.int64)
    typ[(first + per_req - 1)[done]] = 2
    t = (_rand(g, keep) * 1e6)[ev] + pos + _rand(g, total)
    if n > total:
        ev = torch.cat([ev, torch.randint(0, keep, (n - total,), generator=g, device=DEV)])
        typ = torch.cat([typ, torch.full((n - total,), 3, dtype=torch.int64, device=DEV)])
        t = torch.cat([t, _rand(g, n - total) * 1e6])
    o = torch.argsort(t, stable=True)
    lay = workloads.user_request_layout(_bits(users), _bits(total_req))
    return lay, workloads.user_request_properties(), _records16(typ[o], req_user[ev[o]], req_id[ev[o]])


def _chunks(c, seed):
    """Uploads of users with Zipf(1.1) activity; every event carries the
    user's average chunk size; 2 % of the users only upload maximum chunks."""
    g, n, users = _gen(seed), c["n"], c["users"]
    user = _perm(g, users)[_zipf(g, n, users, 1.1)]
    heavy = _rand(g, users) < 0.02
    typ = (_rand(g, n) < 0.4).to(torch.int64)
    top = workloads.CHUNK_MAX
    avg = torch.randint(1, top, (n,), generator=g, device=DEV)
    u = _rand(g, n)
    avg[u < 0.05] = top
    avg[(u >= 0.05) & (u < 0.08)] = 0
    avg[heavy[user]] = top
    lay = workloads.chunk_upload_layout(c["preds"], _bits(users))
    return lay, workloads.chunk_upload_properties(c["preds"]), _records16(typ, user, avg)


def _prop_bits(g, n, p):
    typ = torch.zeros(n, dtype=torch.int32, device=DEV)
    for i, x in enumerate(p):
        typ |= (_rand(g, n, torch.float32) < x).to(torch.int32) << i
    return typ


def _timeline(c, seed):
    """One level, 32-bit keys, three properties that become conclusive."""
    g, n = _gen(seed), c["n"]
    key = _distinct32(_zipf(g, n, c["keys"], 1.1), seed)
    return workloads.prop_layout(3, 1, [32]), workloads.timeline_properties(), _records16(
        _prop_bits(g, n, (0.02, 0.9, 0.5)), key)


def _proxy(c, seed):
    """Requests for videos with Zipf(1) popularity; a video's cache state
    alternates at Poisson(4) random times (parent events naming only it)."""
    g, n, videos = _gen(seed), c["n"], c["videos"]
    n_req = int(n / 3.45 * 1.05) + 64
    vid = _zipf(g, n_req, videos, 1.0)
    t_req = _rand(g, n_req)
    n_chg = torch.poisson(torch.full((videos,), 4.0, device=DEV), generator=g).to(torch.int64)
    chg_vid = torch.repeat_interleave(torch.arange(videos, device=DEV), n_chg)
    at = torch.sort(chg_vid.to(torch.float64) + _rand(g, chg_vid.numel())).values
    chg_first = torch.cumsum(n_chg, 0) - n_chg
    chg_k = torch.arange(chg_vid.numel(), device=DEV) - chg_first[chg_vid]
    cached = ((torch.searchsorted(at, vid.to(torch.float64) + t_req) - chg_first[vid]) & 1) == 1
    fault = _rand(g, n_req) < 0.002
    req_type = torch.where(cached, torch.where(fault, 4, 2), 3)
    prog = torch.floor(torch.log(torch.clamp(_rand(g, n_req), min=1e-12)) / math.log(0.6)).to(torch.int64)
    done = torch.nonzero(_rand(g, n_req) < 0.95).reshape(-1)
    prog_req = torch.repeat_interleave(torch.arange(n_req, device=DEV), prog)
    prog_k = torch.arange(prog_req.numel(), device=DEV) - (torch.cumsum(prog, 0) - prog)[prog_req]
    gap = 1e-6
    t = torch.cat([t_req, t_req[prog_req] + gap * (1 + prog_k) * _rand(g, prog_req.numel()),
                   t_req[done] + gap * (2 + prog[done]), at - chg_vid])
    typ = torch.cat([req_type, torch.full_like(prog_req, 5), torch.full_like(done, 6), chg_k & 1])
    v = torch.cat([vid, vid[prog_req], vid[done], chg_vid])
    r = torch.cat([torch.arange(n_req, device=DEV), prog_req, done, torch.zeros_like(chg_vid)])
    o = torch.argsort(t, stable=True)[:n]
    typ, v, r = typ[o], v[o], r[o]
    if c["wide"]:
        kv, kr, vb, rb = _distinct32(v, seed), _distinct32(r, seed + 1), 32, 32
    else:
        kv, kr, vb, rb = _perm(g, videos)[v], _perm(g, n_req)[r], _bits(videos), _bits(n_req)
    rec = _records16(typ, kv, torch.where(typ < 2, torch.zeros_like(kr), kr))
    if rec.numel() != 16 * n:
        raise ValueError("too few events drawn")
    return workloads.proxy_cache_layout(True, vb, rb), workloads.proxy_cache_properties(), rec


def _large(c, seed):
    g, n, block = _gen(seed), c["n"], 1 << 26
    w = np.arange(1, c["keys"] + 1, dtype=np.float64) ** -1.1
    cdf = torch.from_numpy(np.cumsum(w) / w.sum()).to(DEV)
    rec = torch.zeros((n, 4), dtype=torch.int32, device=DEV)
    for a in range(0, n, block):
        b = min(n, a + block)
        r = torch.clamp(torch.searchsorted(cdf, _rand(g, b - a), right=True), max=c["keys"] - 1)
        rec[a:b, 0] = torch.arange(a, b, device=DEV, dtype=torch.int32)
        rec[a:b, 1] = _prop_bits(g, b - a, (0.02, 0.9, 0.5))
        rec[a:b, 2] = _distinct32(r, seed).to(torch.int32)
    lay = workloads.prop_layout(3, 1, [32])
    lay.type_bytes = 1
    return lay, list(workloads.LARGE_PROPERTIES), rec.view(torch.uint8).reshape(-1)


def _spread(lo, hi, k):
    """k sizes spread evenly over the logarithm of [lo, hi]."""
    return [int(math.exp(math.log(lo) + (i + 0.5) / k * math.log(hi / lo))) for i in range(k)]


def _batch(c, seed):
    """Traces whose lengths are spread over the logarithm of the range, in an
    order drawn from the seed; keys Zipf(1.1) over max(16, length / 256) values
    of each trace (inverse of the continuous distribution function)."""
    g = _gen(seed)
    lens = np.random.RandomState(int(seed) % (1 << 31)).permutation(_spread(c["min_len"], c["max_len"], c["traces"]))
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(offsets[-1])
    lens_d = torch.from_numpy(lens.astype(np.int64)).to(DEV)
    ks = torch.clamp(lens_d // 256, min=16)
    typ = _prop_bits(g, n, (0.3, 0.3, 0.3))
    rec = torch.zeros((n, 4), dtype=torch.int32, device=DEV)
    rec[:, 1] = typ
    del typ
    for a in range(0, n, 1 << 26):
        b = min(n, a + (1 << 26))
        at = torch.arange(a, b, device=DEV)
        t = torch.searchsorted(torch.from_numpy(offsets[1:]).to(DEV), at, right=True)
        k = ks[t]
        top = (k + 1).to(torch.float64) ** -0.1
        r = ((1.0 + _rand(g, b - a) * (top - 1.0)) ** -10.0 - 1.0).to(torch.int64)
        r = torch.minimum(torch.clamp(r, min=0), k - 1)
        rec[a:b, 0] = (at - torch.from_numpy(offsets).to(DEV)[t]).to(torch.int32)
        rec[a:b, 2] = ((r + t) % k).to(torch.int32)
    lay = workloads.prop_layout(3, 1, [_bits(max(16, int(lens.max()) // 256))])
    lay.type_bytes = 1
    return lay, workloads.batch_properties(c["props"]), rec.view(torch.uint8).reshape(-1), [int(x) for x in offsets]


_PUSHES = 8          # pushes a serving state goes round


def _serving(c, seed):
    """Chunks of `streams` log streams: every event picks one of the stream's
    `bindings` (user, request) pairs; 0.3 / 0.3 / 0.35 / 0.05 issue / progress /
    done / other.  Returns the records of all pushes and, per push, the chunks'
    sizes and streams (a chunk's records lie one after another)."""
    g, rs = _gen(seed), np.random.RandomState(int(seed) % (1 << 31))
    S, B = c["streams"], c["bindings"]
    user_of = _zipf(g, S * B, 1000, 1.2).reshape(S, B)
    pushes = []
    for _ in range(_PUSHES):
        sizes = rs.permutation(_spread(4096, 262_144, c["chunks"]))
        pushes.append(([int(x) for x in sizes], [int(x) for x in rs.randint(0, S, c["chunks"])]))
    size = torch.tensor([x for p in pushes for x in p[0]], device=DEV)
    stream = torch.repeat_interleave(torch.tensor([x for p in pushes for x in p[1]], device=DEV), size)
    n = stream.numel()
    b = torch.randint(0, B, (n,), generator=g, device=DEV)
    rec = _records16(_choice(g, n, [0.3, 0.3, 0.35, 0.05]), user_of[stream, b], (b * 7919 + 13) % B)
    return workloads.serving_layout(S, 1000, B), workloads.user_request_properties(), rec, pushes


_TRACES = {"sockets": _sockets, "users": _users, "chunks": _chunks, "timeline": _timeline, "proxy": _proxy,
           "large": _large}


# --------------------------------------------------------------------------
# one state, one pass
# --------------------------------------------------------------------------
def _context(lay, props):
    ctx = lib.Context(0)
    ctx.set_layout(lay)
    return ctx, [ctx.add_spec(p) for p in props]


def _capacity(c):
    """Instances (and nodes) the case's trace can have, at most."""
    if c["kind"] == "users":
        return c["n"] // 2 + 2 * c["users"] + 16
    if c["kind"] == "proxy":
        return int(c["n"] / 3.45 * 1.05) + 64
    return c.get("keys") or c["users"]


def prepare(case, seed):
    c = case
    if c["kind"] == "batch":
        lay, props, rec, offsets = _batch(c, seed)
        ctx, ids = _context(lay, props)
        T, P = c["traces"], len(ids)
        return {"kind": "batch", "ctx": ctx, "ids": ids, "rec": rec, "offsets": offsets,
                "verdict": torch.zeros(T * P, dtype=torch.uint8, device=DEV),
                "counts": torch.zeros(T * P * 6, dtype=torch.int64, device=DEV),
                "ws": ctx.batch_workspace(offsets[-1], T, ids)}
    if c["kind"] == "serving":
        lay, props, rec, pushes = _serving(c, seed)
        ctx, ids = _context(lay, props)
        grp = lib.StreamGroup(ctx, ids, c["streams"], c["bindings"], sum(pushes[0][0]))
        at, todo = rec.data_ptr(), []
        for sizes, streams in pushes:
            ptrs = []
            for s in sizes:
                ptrs.append(at)
                at += 16 * s
            todo.append((ptrs, sizes, streams))
        return {"kind": "serving", "ctx": ctx, "grp": grp, "rec": rec, "todo": todo, "i": 0}
    lay, props, rec = _TRACES[c["kind"]](c, seed)
    ctx, ids = _context(lay, props)
    n, out = c["n"], c.get("outputs", "root")
    timeline = c["kind"] == "timeline"
    res = ctx.alloc_result(len(ids), _capacity(c), instances=timeline or out in ("instances", "all"),
                           nodes=out == "all", timeline=timeline, n_events=n if c.get("events") else 0,
                           key_values=out == "all" and c.get("wide", False))
    outputs = {}
    for k, v in vars(res).items():
        for m, x in enumerate(v if isinstance(v, list) else [v]):
            if isinstance(x, torch.Tensor):
                outputs["%s%d" % (k, m)] = x.zero_()      # entries beyond the instances stay zero
    return {"kind": "eval", "ctx": ctx, "ids": ids, "rec": rec, "n": n, "res": res, "ws": ctx.workspace(n, ids),
            "outputs": outputs}


def run(state):
    s = state
    if s["kind"] == "eval":
        s["ctx"].eval_into(s["rec"], s["n"], s["ids"], s["res"], s["ws"])
        return s["outputs"]
    if s["kind"] == "batch":
        s["ctx"].eval_batch_into(s["rec"], s["offsets"], s["ids"], s["verdict"], s["counts"], s["ws"])
        return {"verdict": s["verdict"], "counts": s["counts"]}
    ptrs, sizes, streams = s["todo"][s["i"] % len(s["todo"])]
    s["i"] += 1
    s["grp"].push_chunks(ptrs, sizes, streams)
    verdict, counts, bindings = s["grp"].read()     # the verdicts on the host: a monitor acts on them
    return {"verdict": verdict, "counts": counts, "bindings": bindings}


def work(case):
    """Bytes: every record read once, every output written once.  Operations:
    one state step per event and property."""
    c = case
    if c["kind"] == "batch":
        n = sum(_spread(c["min_len"], c["max_len"], c["traces"]))
        return {"bytes": 16 * n + c["traces"] * c["props"] * 49, "flops": n * c["props"]}
    if c["kind"] == "serving":
        n = sum(_spread(4096, 262_144, c["chunks"]))
        return {"bytes": 16 * n + c["streams"] * 57, "flops": n}
    n, P = c["n"], {"sockets": 2, "users": 1, "chunks": 1 + c.get("preds", 0), "timeline": 3, "proxy": 2, "large": 3}[c["kind"]]
    out = c.get("outputs", "root")
    inst = {"users": n // 3, "proxy": int(n / 3.45)}.get(c["kind"], c.get("keys") or c.get("users"))
    nodes = c.get("users") if c["kind"] == "users" else c.get("videos", 0)
    b = (12 if c["kind"] == "sockets" else 16) * n + 57 * P
    if out in ("instances", "all") or c["kind"] == "timeline":
        b += inst * (8 + P)
    if out == "all":
        b += nodes * (8 + 25 * P) + (inst * 8 + nodes * 4 if c.get("wide") else 0)
    if c["kind"] == "timeline":
        b += inst * 4 * P + (n * P if c["events"] else 0)
    return {"bytes": b, "flops": n * P}


# --------------------------------------------------------------------------
# closed forms
# --------------------------------------------------------------------------
def _percent(top, n, num, den, when):
    """Def. 7 for A >= num/den when no child is conclusively false: `when` if
    the share of the `top` children reaches num/den, else presumably false."""
    return torch.where(top * den >= num * n, when, 2)


def exact(case, seed):
    """The socket and the user/request traces from the definition, by their
    properties' closed forms on finite traces: G(a -> F b) is presumably true
    (3) when no a follows the last b and presumably false (2) otherwise;
    (G a) -> (F b) is true (5) once an event is not a, else presumably false.
    The other traces' properties have no such form."""
    c = case
    if c["kind"] not in ("sockets", "users") or c["n"] > 20_000_000:
        return None
    sockets = c["kind"] == "sockets"
    lay, props, rec = _TRACES[c["kind"]](c, seed)
    r = rec.view(torch.int32).reshape(c["n"], -1).to(torch.int64)
    typ, at = r[:, 1], torch.arange(c["n"], device=DEV)
    a, b = (1, 2) if sockets else (0, 2)
    key = r[:, 2] if sockets else (r[:, 2] << lay.key_bits[1]) | r[:, 3]
    keys, inst = torch.unique(key, return_inverse=True)
    k = keys.numel()

    def last(t):
        return torch.full((k,), -1, dtype=torch.int64, device=DEV).scatter_reduce(
            0, inst[typ == t], at[typ == t], "amax")

    verdicts = [torch.where(last(a) > last(b), 2, 3)]
    if sockets:
        other = torch.zeros(k, dtype=torch.int64, device=DEV).scatter_add(0, inst, (typ != a).to(torch.int64))
        verdicts.append(torch.where(other > 0, 5, 2))
    cap, P = _capacity(c), len(verdicts)
    out = {}
    if sockets:
        root = [torch.bincount(v, minlength=6) for v in verdicts]
        total = torch.tensor(k, device=DEV)
        # property 0: no child above presumably true; property 1: T children reach Tc
        tops = [_percent(root[0][3], total, 19, 20, 3), _percent(root[1][5], total, 19, 20, 4)]
        sizes = [k, 0]
    else:
        user = keys >> lay.key_bits[1]
        users, of = torch.unique(user, return_inverse=True)
        m = users.numel()
        cnt = torch.zeros((m, 6), dtype=torch.int64, device=DEV)
        cnt.view(-1).scatter_add_(0, of * 6 + verdicts[0], torch.ones_like(of))
        node = _percent(cnt[:, 3], cnt.sum(1), 9, 10, 3)
        root = [torch.bincount(node, minlength=6)]
        tops = [torch.where(root[0][3] >= 500, 3, torch.where(root[0][3] + root[0][2] >= 500, 2, 1))]
        sizes = [k, m, 0]
    out["root_verdict0"] = torch.stack(tops).to(torch.uint8)
    out["root_counts0"] = torch.cat(root)
    out["sizes0"] = torch.tensor(sizes, device=DEV)

    def padded(x, n, dtype):
        y = torch.zeros(n, dtype=dtype, device=DEV)
        y[:x.numel()] = x
        return y

    if c["outputs"] in ("instances", "all"):
        out["inst_keys0"] = padded(keys, cap, torch.int64)
        out["inst_verdict0"] = torch.cat([padded(v, cap, torch.uint8) for v in verdicts])
    if c["outputs"] == "all":
        out["node_keys1"] = padded(users, cap, torch.int64)
        out["node_counts1"] = padded(cnt.view(-1), P * cap * 6, torch.int32)
        out["node_verdict1"] = padded(node, cap, torch.uint8)
    return out
