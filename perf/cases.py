"""The work this framework is measured on: frames of interaction sessions over
the windowed KV pool, through its public entry points.

A case is a pool shape, a set of sessions at a point of their calls, and one
frame (or part of one) that a serving loop asks for: a chunk per session and
then single-token decode rounds.  ``api`` says how it is asked for: "frame" is
one frame_step call, "layers" the per-layer calls that a model's own layer
loop makes (append + chunk prefill, or the decode with the append fused),
"reprefill" opens a session, prefills one long chunk and closes it again.

Positions advance from pass to pass as in a call, so the ring keeps turning;
the number of keys a query sees stays the same once the window is full.
"""
import math

import torch

import paper_2607_02640_amd as mtn

DEV = "cuda"
THETA = 1.0e6


def _case(name, api, dtype, heads, d, sinks, window, sessions, layers, chunk, decodes,
          filled=1.0, scale=1.0):
    c = {"api": api, "dtype": dtype, "hq": heads[0], "hkv": heads[1], "d": d, "sinks": sinks,
         "window": window, "sessions": sessions, "layers": layers, "chunk_lo": chunk[0],
         "chunk_hi": chunk[1], "dec_lo": decodes[0], "dec_hi": decodes[1],
         "filled": filled, "scale": scale}
    if name:
        c = {"name": name, **c}
    return c


def listed():
    return [
        # the smallest work: the tiny parity shape (4 sessions, one fp32 layer,
        # a 128-token window); launches and host latency
        _case("tiny-f32", "frame", "f32", (8, 2), 64, 4, 128, 4, 1, (8, 8), (4, 4)),
        # one caller alone on the GPU, a whole frame of every layer: the
        # response latency of an idle server (Qwen3-Omni-shaped attention)
        _case("one-session", "frame", "bf16", (32, 4), 128, 4, 4096, 1, 48, (25, 25), (16, 16)),
        # the headline batch: 128 sessions at the Qwen3-Omni shape (4 of the 48
        # equal layers), 25-token chunk and 16 decodes
        _case("batch-128", "frame", "bf16", (32, 4), 128, 4, 4096, 128, 4, (25, 25), (16, 16)),
        # one staggered group of 32 of those sessions with the FP8 cache
        _case("group-32-fp8", "frame", "fp8", (32, 4), 128, 4, 4096, 32, 8, (25, 25), (16, 16)),
        # a model's layer loop over a decode token for all 128 sessions, FP8
        _case("decode-128-fp8", "layers", "fp8", (32, 4), 128, 4, 4096, 128, 8, (1, 1), (0, 0)),
        # a model's layer loop over a chunk for all 128 sessions, FP8
        _case("chunk-128-fp8", "layers", "fp8", (32, 4), 128, 4, 4096, 128, 4, (25, 25), (0, 0)),
        # the layer loop over a chunk for one GPU's share of 16 sessions, bf16
        _case("chunk-16", "layers", "bf16", (32, 4), 128, 4, 4096, 16, 8, (25, 25), (0, 0)),
        # speech frames of one token and one decode, multi-head attention
        # (Moshi-shaped, 64 sessions, 8 of 32 layers)
        _case("speech-64", "frame", "bf16", (32, 32), 128, 4, 2048, 64, 8, (1, 1), (1, 1),
              scale=1.0 / math.sqrt(128.0)),
        # ragged chunks and decodes over many sessions, a third of them still
        # filling their window (MiniCPM-o-shaped, 4 of 36 layers)
        _case("ragged-256", "frame", "bf16", (32, 8), 128, 4, 2048, 256, 4, (10, 40), (8, 24),
              filled=0.7),
        # application-level recycling: a session's sinks and last window
        # re-encoded as one chunk of a fresh, unbounded session
        _case("reprefill", "reprefill", "bf16", (32, 4), 128, 4, 0, 1, 2, (4100, 4100), (0, 0)),
        # head dimension 64, an odd batch of ragged frames
        _case("d64-bf16", "frame", "bf16", (16, 2), 64, 4, 1500, 21, 4, (9, 33), (3, 7),
              filled=0.8),
        # fp32 cache and activations, odd sizes
        _case("f32-frames", "frame", "f32", (16, 4), 128, 5, 900, 13, 2, (5, 21), (2, 5),
              filled=0.8),
    ]


def draw(rng):
    """A case of the listed ones' ranges: cache type and head shape as the
    framework supports them, sessions and windows over their whole range."""
    def logint(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))
    while True:
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp8", "fp8", "f32"])
        d = 128 if dtype == "fp8" else rng.choice([128, 128, 64])
        hkv = rng.choice([2, 4, 8]) if dtype != "bf16" or rng.random() < 0.8 else 32
        g = 1 if hkv == 32 else rng.choice([1, 2, 4, 8, 8])
        window = logint(96, 4300 if dtype != "f32" else 1500)
        sessions = logint(1, 256 if dtype != "f32" else 24)
        layers = rng.choice([1, 2, 4, 8]) if dtype != "f32" else rng.choice([1, 2])
        lo = rng.choice([1, 4, 10, 25])
        chunk = (lo, lo + rng.choice([0, 0, 3, 15]))
        api = rng.choice(["frame", "frame", "frame", "layers", "layers", "reprefill"])
        filled = rng.choice([1.0, 1.0, 0.7])
        dec = (rng.choice([1, 2, 8]), 0)
        dec = (dec[0], dec[0] + rng.choice([0, 4]))
        if api == "layers":
            chunk, dec = (chunk[0], chunk[0]), rng.choice([(0, 0), (1, 1), (3, 3)])
        if api == "reprefill":
            n = logint(300, 4300 if dtype != "f32" else 900)
            window, sessions, layers, chunk, dec, filled = 0, 1, rng.choice([1, 2]), (n, n), (0, 0), 1.0
        c = _case(None, api, dtype, (g * hkv, hkv), d, rng.choice([0, 4, 4, 17]), window,
                  sessions, layers, chunk, dec, filled)
        w, top = work(c), work(listed()[2])
        if w["bytes"] <= top["bytes"] / 4 and w["flops"] <= top["flops"] / 4:
            return c


# ---------------------------------------------------------------------------
# the state of a case: everything follows from the case and the seed
# ---------------------------------------------------------------------------
def _lengths(c):
    """(tokens before the frame, chunk tokens, decodes) per session."""
    n = c["sessions"]

    def spread(lo, hi, i, k):  # an even, unordered spread of [lo, hi] over the sessions
        return lo + (i * k + k // 2) % (hi - lo + 1)
    if c["api"] == "reprefill":
        have = [0] * n
    else:
        full = c["sinks"] + c["window"]
        n_full = int(round(c["filled"] * n))
        have = [full + spread(0, max(1, c["window"] // 8), i, 37) if i < n_full
                else spread(full // 10, full - 1, i, 331) for i in range(n)]
    chunk = [spread(c["chunk_lo"], c["chunk_hi"], i, 13) for i in range(n)]
    dec = [spread(c["dec_lo"], c["dec_hi"], i, 7) for i in range(n)]
    return have, chunk, dec


def _io(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


class _Inputs:
    """The rows a case's tokens bring, drawn in one order from the seed."""

    def __init__(self, c, seed):
        self.c, self.gen = c, torch.Generator(device=DEV)
        self.gen.manual_seed(int(seed) * 2654435761 % (1 << 31) + 17)

    def rows(self, *shape):
        t = torch.randn(shape, generator=self.gen, device=DEV, dtype=torch.float32)
        return t.mul_(self.c["scale"]).to(_io(self.c))

    def history(self):
        """Plans that bring every session to its length: (session indices,
        tokens each, k, v) with k and v [layers][tokens][kv heads][d]."""
        c = self.c
        have, chunk, _ = _lengths(c)
        cmax, done = max(chunk), [0] * c["sessions"]
        while True:
            idx = [i for i in range(c["sessions"]) if done[i] < have[i]]
            if not idx:
                return
            nt = [min(cmax, have[i] - done[i]) for i in idx]
            for i, m in zip(idx, nt):
                done[i] += m
            shape = (c["layers"], sum(nt), c["hkv"], c["d"])
            yield idx, nt, self.rows(*shape), self.rows(*shape)

    def frame(self):
        """The frame's own rows, chunk and decode: dict of q, k, v tensors."""
        c = self.c
        _, chunk, dec = _lengths(c)
        tc, md = sum(chunk), max(dec)
        f = {"q_chunk": self.rows(c["layers"], tc, c["hq"], c["d"]),
             "k_chunk": self.rows(c["layers"], tc, c["hkv"], c["d"]),
             "v_chunk": self.rows(c["layers"], tc, c["hkv"], c["d"])}
        if md:
            lead = (md, c["layers"], c["sessions"])
            f["q_dec"] = self.rows(*lead, c["hq"], c["d"])
            f["k_dec"] = self.rows(*lead, c["hkv"], c["d"])
            f["v_dec"] = self.rows(*lead, c["hkv"], c["d"])
        return f


def prepare(case, seed):
    c = case
    have, chunk, dec = _lengths(c)
    n, cmax = c["sessions"], max(chunk)
    kw = dict(n_layers=c["layers"], n_q_heads=c["hq"], n_kv_heads=c["hkv"], head_dim=c["d"],
              max_chunk=cmax, max_sessions=n, dtype=c["dtype"], rope_theta=THETA)
    if c["api"] == "reprefill":
        kw.update(n_sink=0, window=None, max_len=cmax, n_blocks=-(-cmax // 16))
    else:
        ring = -(-(c["window"] + cmax - 1) // 16) + -(-c["sinks"] // 16)
        kw.update(n_sink=c["sinks"], window=c["window"], n_blocks=n * ring)
    kv = torch.empty(mtn.Pool.required(**kw), dtype=torch.uint8, device=DEV)
    pool = mtn.Pool(**kw, kv=kv)
    inputs = _Inputs(c, seed)
    s = {"case": c, "pool": pool, "chunk": chunk, "dec": dec}
    if c["api"] != "reprefill":
        s["sids"] = [pool.session_open() for _ in range(n)]
        for idx, nt, k, v in inputs.history():
            pool.plan_begin([s["sids"][i] for i in idx], nt)
            for l in range(c["layers"]):
                pool.frame_append_kv(l, k[l], v[l])
            pool.plan_commit()
    s.update(inputs.frame())
    # output rows that a ragged batch's later rounds do not write stay zero
    s["out_chunk"] = torch.zeros_like(s["q_chunk"])
    s["lse_chunk"] = torch.zeros(s["q_chunk"].shape[:3], dtype=torch.float32, device=DEV)
    if max(dec):
        s["out_dec"] = torch.zeros_like(s["q_dec"])
        s["lse_dec"] = torch.zeros(s["q_dec"].shape[:4], dtype=torch.float32, device=DEV)
    torch.cuda.synchronize()
    return s


def run(state):
    s, c, pool = state, state["case"], state["pool"]
    if c["api"] == "frame":
        pool.frame_step(s["sids"], s["chunk"], s["dec"], s["q_chunk"], s["k_chunk"], s["v_chunk"],
                        s["out_chunk"], s.get("q_dec"), s.get("k_dec"), s.get("v_dec"),
                        s.get("out_dec"), lse_chunk=s["lse_chunk"], lse_dec=s.get("lse_dec"))
    else:
        fresh = c["api"] == "reprefill"
        sids = [pool.session_open()] if fresh else s["sids"]
        pool.plan_begin(sids, s["chunk"])
        for l in range(c["layers"]):
            if max(s["chunk"]) == 1:
                pool.attend_decode_append(l, s["k_chunk"][l], s["v_chunk"][l], s["q_chunk"][l],
                                          s["out_chunk"][l], s["lse_chunk"][l])
            else:
                pool.frame_append_kv(l, s["k_chunk"][l], s["v_chunk"][l])
                pool.attend_chunk_prefill(l, s["q_chunk"][l], s["out_chunk"][l],
                                          s["lse_chunk"][l])
        pool.plan_commit()
        for j in range(max(s["dec"])):
            pool.plan_begin(sids, [1] * len(sids))
            for l in range(c["layers"]):
                pool.attend_decode_append(l, s["k_dec"][j, l], s["v_dec"][j, l], s["q_dec"][j, l],
                                          s["out_dec"][j, l], s["lse_dec"][j, l])
            pool.plan_commit()
        if fresh:
            pool.session_close(sids[0])
    out = {"out_chunk": s["out_chunk"], "lse_chunk": s["lse_chunk"]}
    if max(s["dec"]):
        out.update(out_dec=s["out_dec"], lse_dec=s["lse_dec"])
    return out


def work(case):
    """Each round (the chunk, then every decode) reads the keys and values its
    queries see once per KV head, its q, k and v rows, and writes its outputs
    and the appended rows; 4 D flops per (query head, visible key)."""
    c = case
    have, chunk, dec = _lengths(c)
    eb = {"f32": 4, "bf16": 2, "fp8": 1}[c["dtype"]]
    io = 4 if c["dtype"] == "f32" else 2
    token = c["hkv"] * (2 * c["d"] * eb + (2 if c["dtype"] == "fp8" else 0))
    rows = 2 * c["hq"] * c["d"] * io + 2 * c["hkv"] * c["d"] * io + token + 4 * c["hq"]
    unbounded = c["api"] == "reprefill"

    def seen(t):  # keys the query at position t sees
        return t + 1 if unbounded else min(t + 1, c["sinks"] + c["window"])
    byts = flops = 0
    for p, m, k in zip(have, chunk, dec):
        for start, cnt in [(p, m)] + [(p + m + j, 1) for j in range(k)]:
            old = start if unbounded else min(start, c["sinks"] + c["window"] - 1)
            byts += old * token + cnt * rows
            flops += sum(seen(t) for t in range(start, start + cnt)) * 4 * c["hq"] * c["d"]
    return {"bytes": byts * c["layers"], "flops": flops * c["layers"]}


def tolerance(case):
    # fp32: sums in another order (measured up to 4.8e-7 against 64 bits, so
    # about 1e-6 between two such paths).  bf16 and FP8 caches: queries,
    # probabilities and outputs rounded to bf16 (measured up to 3.4e-3).
    return {"rel": 4e-6} if case["dtype"] == "f32" else {"rel": 1.3e-2, "max": 0.2}


# ---------------------------------------------------------------------------
# the same frame in 64 bits with plain torch
# ---------------------------------------------------------------------------
def _rotate(x, pos):
    """Rotate-half RoPE of x [T][H][D] at positions pos [T]."""
    half = x.shape[-1] // 2
    inv = THETA ** (-2.0 * torch.arange(half, device=DEV, dtype=torch.float64) / x.shape[-1])
    ang = (pos.to(torch.float64)[:, None] * inv)[:, None]
    cos, sin, a, b = ang.cos(), ang.sin(), x[..., :half].double(), x[..., half:].double()
    return torch.cat([a * cos - b * sin, b * cos + a * sin], dim=-1)


def _e4m3(x):
    """What an FP8 cache holds of each row: E4M3 codes times the smallest
    power of two that keeps the row's largest magnitude within 448."""
    x = x.float()
    top = x.abs().amax(dim=-1, keepdim=True).double()
    e = torch.where(top > 0, torch.ceil(torch.log2(top / 448.0)), torch.zeros_like(top))
    e = torch.where(top * torch.exp2(-e) > 448.0, e + 1, e)
    e = torch.where((top > 0) & (top * torch.exp2(-(e - 1)) <= 448.0), e - 1, e).clamp(-126, 127)
    return (x.double() * torch.exp2(-e)).float().to(torch.float8_e4m3fn).double() * torch.exp2(e)


def exact(case, seed):
    c = case
    have, chunk, dec = _lengths(c)
    n, g = c["sessions"], c["hq"] // c["hkv"]
    longest = max(h + m + k for h, m, k in zip(have, chunk, dec))
    kh = torch.zeros((n, longest, c["layers"], c["hkv"], c["d"]), dtype=_io(c), device=DEV)
    vh = torch.zeros_like(kh)
    inputs, done = _Inputs(c, seed), [0] * n

    def put(idx, nt, k, v):
        si = torch.tensor([i for i, m in zip(idx, nt) for _ in range(m)], device=DEV)
        pi = torch.tensor([done[i] + j for i, m in zip(idx, nt) for j in range(m)], device=DEV)
        kh[si, pi], vh[si, pi] = k.transpose(0, 1), v.transpose(0, 1)
        for i, m in zip(idx, nt):
            done[i] += m
    if c["api"] != "reprefill":
        for plan in inputs.history():
            put(*plan)
    f = inputs.frame()
    put(range(n), chunk, f["k_chunk"], f["v_chunk"])
    for j in range(max(dec)):
        idx = [i for i in range(n) if dec[i] > j]
        put(idx, [1] * len(idx), f["k_dec"][j][:, idx], f["v_dec"][j][:, idx])
    out = {"out_chunk": torch.zeros(f["q_chunk"].shape, dtype=torch.float64, device=DEV)}
    out["lse_chunk"] = torch.zeros(f["q_chunk"].shape[:3], dtype=torch.float64, device=DEV)
    if max(dec):
        out["out_dec"] = torch.zeros(f["q_dec"].shape, dtype=torch.float64, device=DEV)
        out["lse_dec"] = torch.zeros(f["q_dec"].shape[:4], dtype=torch.float64, device=DEV)
    off = 0
    for i in range(n):
        p, m, k = have[i], chunk[i], dec[i]
        end = p + m + k
        pos = torch.arange(end, device=DEV)
        t = pos[p:, None]
        hide = pos[None] > t
        if c["api"] != "reprefill":
            hide = hide | ((pos[None] >= c["sinks"]) & (pos[None] <= t - c["window"]))
        hide = hide.repeat_interleave(g, 0)  # rows are (token, head of the group)
        for l in range(c["layers"]):
            q = f["q_chunk"][l, off:off + m]
            if k:
                q = torch.cat([q, f["q_dec"][:k, l, i]])
            q = _rotate(q, pos[p:]).view(m + k, c["hkv"], g, c["d"]).transpose(0, 1)
            kr, vr = _rotate(kh[i, :end, l], pos), vh[i, :end, l].double()
            if c["dtype"] == "fp8":
                kr, vr = _e4m3(kr), _e4m3(vr)
            for h in range(c["hkv"]):
                sc = q[h].reshape(-1, c["d"]) @ kr[:, h].T / math.sqrt(c["d"])
                sc.masked_fill_(hide, -math.inf)
                lse = sc.logsumexp(-1)
                o = (sc.sub_(lse[:, None]).exp_() @ vr[:, h].contiguous()).view(m + k, g, c["d"])
                lse, hs = lse.view(m + k, g), slice(h * g, (h + 1) * g)
                out["out_chunk"][l, off:off + m, hs], out["lse_chunk"][l, off:off + m, hs] = o[:m], lse[:m]
                if k:
                    out["out_dec"][:k, l, i, hs], out["lse_dec"][:k, l, i, hs] = o[m:], lse[m:]
        off += m
    return out
