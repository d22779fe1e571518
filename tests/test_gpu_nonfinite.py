"""A key and its value reach the outputs of the queries that see that key and of
no others: with infinite or NaN elements in one of them, every row of the chunk
prefill that does not see that key is bitwise what it is with finite elements,
and, for a value, a row that does is so in every other dimension."""
import pytest
import torch

from tests._gpu_util import TDT, make_pool, say

pytestmark = pytest.mark.gpu

HKV, N = 2, 43          # KV heads, tokens of the chunk
BAD = {3: float("nan"), 17: float("inf"), 40: float("-inf"), 61: float("nan")}  # dim: value


def _history(S, W):
    """Tokens before the chunk: none, a part of the window, a turned ring."""
    return [0, W // 2, S + W + 29] if W else [0, 150]


def _run(pool, kw, have, bad, seed):
    """The chunk at positions have .. have + N - 1 of a fresh session, the key
    or value row (bad[0]) at position bad[1] bad: (out, lse)."""
    dt = TDT[kw["dtype"]]
    sid = pool.session_open()
    gen = torch.Generator(device="cuda").manual_seed(seed)
    draw = lambda *s: torch.randn(s, generator=gen, device="cuda").to(dt)
    at, out, lse = 0, None, None
    while at < have + N:
        n = min(N, have - at) if at < have else N
        k, v = draw(n, HKV, kw["d"]), draw(n, HKV, kw["d"])
        if bad and at <= bad[1] < at + n:
            for dim, x in BAD.items():
                # an infinite element would change the FP8 row's scale
                (k if bad[0] == "k" else v)[bad[1] - at, :, dim] = (
                    float("nan") if kw["dtype"] == "fp8" else x)
        pool.plan_begin([sid], [n])
        pool.frame_append_kv(0, k, v)
        if at == have:
            q = draw(n, kw["hq"], kw["d"])
            out = torch.empty_like(q)
            lse = torch.empty((n, kw["hq"]), dtype=torch.float32, device="cuda")
            pool.attend_chunk_prefill(0, q, out, lse)
        pool.plan_commit()
        at += n
    torch.cuda.synchronize()
    pool.session_close(sid)
    return out, lse


@pytest.mark.parametrize("dtype,d,g,S,W,rows", [
    ("f32", 128, 4, 4, 60, 0),        # one segment
    ("f32", 128, 8, 17, 700, 0),      # key segments and their merge
    ("f32", 64, 1, 0, 390, 0),
    ("f32", 64, 2, 20, None, 0),      # unbounded
    ("f32", 64, 8, 4, 20, 0),         # the chunk is longer than the window
    ("bf16", 64, 8, 4, 60, 0),
    ("bf16", 64, 4, 17, 700, 0),
    ("bf16", 64, 1, 0, 390, 256),     # two tiles a wave
    ("bf16", 64, 2, 20, None, 128),
    ("bf16", 64, 8, 4, 20, 0),
    ("bf16", 128, 8, 4, 60, 0),
    ("bf16", 128, 4, 17, 700, 256),
    ("bf16", 128, 1, 20, None, 0),
    ("bf16", 128, 2, 4, 20, 128),
    ("fp8", 128, 8, 4, 60, 0),
    ("fp8", 128, 1, 17, 700, 256),
    ("fp8", 128, 4, 20, None, 0),
])
def test_a_bad_key_or_value_stays_with_the_rows_that_see_it(dtype, d, g, S, W, rows):
    say(f"non-finite values {dtype} d={d} G={g} S={S} W={W} rows={rows}")
    kw = dict(n_layers=1, hq=HKV * g, hkv=HKV, d=d, S=S, W=W, dtype=dtype)
    blocks = -(-S // 16) + -(-(W + N - 1) // 16) if W else 32
    pool = make_pool(**kw, cmax=N, max_sessions=1, n_blocks=blocks, max_len=0 if W else 400)
    if rows:
        pool.set_prefill_pass_rows(rows)
    for have in _history(S, W):
        t = torch.arange(have, have + N)
        clean = _run(pool, kw, have, None, have + 1)
        assert torch.isfinite(clean[0]).all()
        dims = torch.zeros(d, dtype=torch.bool, device="cuda")
        dims[list(BAD)] = True
        # the last token, one inside the chunk, a sink when the chunk writes it,
        # and keys that leave the window inside the chunk
        cand = {have + N - 1, have + 20, have + 1, have + N // 2 - W if W else -1,
                have + 1 - W if W else -1}
        for p in sorted(x for x in cand if 0 <= x < have + N):
            sees = p <= t if W is None or p < S else (p <= t) & (p > t - W)
            sees = sees.cuda()
            for kind in ("v", "k"):
                out, lse = _run(pool, kw, have, (kind, p), have + 1)
                what = f"{have} tokens before the chunk, bad {kind} at {p}"
                assert torch.equal(out[~sees], clean[0][~sees]), what
                assert torch.equal(lse[~sees], clean[1][~sees]), what
                if kind == "k":
                    assert not torch.isfinite(out[sees]).any(), what
                    continue
                assert torch.equal(lse, clean[1]), what
                assert not torch.isfinite(out[sees][..., dims]).any(), what
                if dtype != "fp8":  # every weight is above 0: an infinite value stays infinite
                    for dim, x in BAD.items():
                        if x == x:
                            assert (out[sees][..., dim] == x).all(), f"{what}, dim {dim}"
                if dtype != "fp8":  # (the row's scale may differ without those elements)
                    assert torch.equal(out[sees][..., ~dims], clean[0][sees][..., ~dims]), what


def test_a_bad_value_of_a_fused_chunk_stays_with_the_rows_that_see_it():
    """The fp8 frame whose chunk prefill stores the chunk itself: the tiles that
    are computed once more read the tokens that this launch has stored."""
    say("non-finite values, fused fp8 chunk")
    hkv, g, d, W, n = 4, 4, 128, 60, 40
    # enough one-pass sequences that the prefill is not split and carries the append
    ns = torch.cuda.get_device_properties(0).multi_processor_count // (2 * hkv) + 2
    kw = dict(n_layers=1, hq=hkv * g, hkv=hkv, d=d, S=4, W=W, dtype="fp8")
    outs = []
    for bad in (None, 0, 17, n - 1):
        pool = make_pool(**kw, cmax=n, max_sessions=ns, n_blocks=ns * 8)
        sids = [pool.session_open() for _ in range(ns)]
        gen = torch.Generator(device="cuda").manual_seed(8)
        draw = lambda h: torch.randn((1, ns * n, h, d), generator=gen, device="cuda").bfloat16()
        pool.set_timing(True)
        frames = []
        for f in range(3):
            q, k, v = draw(hkv * g), draw(hkv), draw(hkv)
            if bad is not None and f != 1:
                v.view(ns, n, hkv, d)[:, bad, :, 5] = float("nan")
            o = torch.empty_like(q)
            pool.frame_step(sids, [n] * ns, [0] * ns, q, k, v, o)
            frames.append(o.view(ns, n, hkv * g, d))
        torch.cuda.synchronize()
        assert pool.kernel_times()["append"][0] == 0, "the frames did not fuse the append"
        outs.append(frames)
        if bad is None:
            continue
        for f in range(3):
            t = torch.arange(f * n, (f + 1) * n)
            sees = torch.zeros(n, dtype=torch.bool)
            for p in (bad, 2 * n + bad):  # frames 0 and 2 bring a bad value
                sees |= (p <= t) & ((t < p + W) | (p < kw["S"]))
            got, clean = frames[f], outs[0][f]
            assert torch.equal(got[:, ~sees], clean[:, ~sees]), f"bad {bad}, frame {f}"
            assert torch.isnan(got[:, sees][..., 5]).all(), f"bad {bad}, frame {f}"
