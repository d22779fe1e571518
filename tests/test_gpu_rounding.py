"""What the attention kernels round, seen through scores that are exact: with a
RoPE base so large that the last rotation pair does not turn, queries and keys
that live in that one dimension have the score q' k, q' the scaled query as the
kernel holds it, and every expected result follows in float64."""
import math

import numpy as np
import pytest
import torch

from tests._gpu_util import TDT, make_pool, say

pytestmark = pytest.mark.gpu


def _scaled_query(q, d, dtype):
    """log2 units, rounded as the kernels round it."""
    f = np.float32
    x = torch.tensor(f(q) * (f(1.0 / math.sqrt(d)) * f(1.4426950408889634)))
    return float(x.to(TDT[dtype]))


def _attend(dtype, d, g, hkv, keys, v, q, how, sessions=1, kernel=0):
    """keys [n] values of the one dimension (every session and kv head alike),
    v [n, d], q one value per query: the last len(q) tokens are a chunk, or one
    decode for one query.  (out [sessions, len(q), hq, d], lse) and the float64
    expectation [len(q), d], [len(q)]."""
    n, nq, dt, e = len(keys), len(q), TDT[dtype], d // 2 - 1
    kw = dict(n_layers=1, hq=hkv * g, hkv=hkv, d=d, S=0, W=n + 16, dtype=dtype)
    pool = make_pool(**kw, cmax=n, max_sessions=sessions, theta=1e30,
                     n_blocks=sessions * (-(-(2 * n + 16) // 16) + 1))
    pool.set_decode_kernel(kernel)
    sids = [pool.session_open() for _ in range(sessions)]
    kt = torch.zeros((n, hkv, d), device="cuda")
    kt[..., e] = torch.tensor(keys, device="cuda", dtype=torch.float32)[:, None]
    vt = v.to(dt)[:, None].expand(n, hkv, d).cuda()
    qt = torch.zeros((nq, hkv * g, d), device="cuda")
    qt[..., e] = torch.tensor(q, device="cuda", dtype=torch.float32)[:, None]
    rep = lambda x: x.to(dt).repeat(sessions, 1, 1).contiguous()
    pool.plan_begin(sids, [n - nq] * sessions)
    pool.frame_append_kv(0, rep(kt[:n - nq]), rep(vt[:n - nq]))
    pool.plan_commit()
    qq, k2, v2 = rep(qt), rep(kt[n - nq:]), rep(vt[n - nq:])
    out = torch.empty_like(qq)
    lse = torch.empty(qq.shape[:2], dtype=torch.float32, device="cuda")
    pool.plan_begin(sids, [nq] * sessions)
    if how == "chunk":
        pool.frame_append_kv(0, k2, v2)
        pool.attend_chunk_prefill(0, qq, out, lse)
    else:
        pool.attend_decode_append(0, k2, v2, qq, out, lse, n_split=1)
    pool.plan_commit()
    torch.cuda.synchronize()
    ks = torch.tensor(keys, dtype=torch.float64).to(dt).double()
    eo, el = [], []
    for j in range(nq):
        s = ks[:n - nq + j + 1] * _scaled_query(q[j], d, dtype)
        p = torch.exp2(s - s.max())
        eo.append((p @ v.to(dt)[:len(s)].double()) / p.sum())
        el.append((s.max() + torch.log2(p.sum())) * math.log(2.0))
    shape = (sessions, nq, hkv * g)
    return out.view(*shape, d).double().cpu(), lse.view(shape).double().cpu(), torch.stack(eo), torch.stack(el)


def test_fp32_chunk_log_sum_exp_when_the_reference_lags():
    """Scores that stay just under 2^8 times the reference that a row's first
    keys set leave a sum of 2^17.  The expected error is that of the result's
    own last place (values of 8 to 16: 2.8e-7 rms) and a tenth of it from the
    sums; a logarithm of the whole sum adds 5e-7 of its own."""
    say("fp32 lse, lagging reference")
    rng = np.random.default_rng(3)
    hkv = 8
    # enough workgroups that the chunk runs in one segment
    n_sess = torch.cuda.get_device_properties(0).multi_processor_count // (2 * hkv) + 1
    err = []
    for n in (600, 653, 701, 760):
        keys = np.concatenate([np.zeros(16), rng.integers(152, 172, n - 16) / 32.0])
        v = torch.from_numpy(rng.standard_normal((n, 64)))
        q = 8.0 * (1.0 + rng.integers(-20, 6, 16) / 128.0)
        _, lse, _, want = _attend("f32", 64, 1, hkv, keys, v, q, "chunk", sessions=n_sess)
        err.append((lse[0] - want[:, None]).numpy())
    rms = float(np.sqrt(np.mean(np.concatenate(err) ** 2)))
    say(f"rms {rms:.2e}")
    assert rms < 4e-7


@pytest.mark.parametrize("g", [1, 8])
def test_head_dim_64_chunk_sums_unrounded_probabilities(g):
    """The log-sum-exp of bf16 chunks at head dimension 64: sums in fp32 of
    probabilities in fp32 (2e-6 covers 50 of them, the exponentials and the
    result's last place); probabilities rounded to bf16 first are up to 2e-3
    off each."""
    say(f"D=64 chunk row sums G={g}")
    rng = np.random.default_rng(g)
    for n in (24, 41, 50):
        keys = rng.integers(-256, 257, n) / 128.0
        v = torch.from_numpy(rng.standard_normal((n, 64)))
        _, lse, _, want = _attend("bf16", 64, g, 2, keys, v, [8.0, 7.0, 6.5, 8.0], "chunk")
        err = float((lse[0] - want[:, None]).abs().max())
        say(f"n={n} err {err:.2e}")
        assert err < 2e-6


def _dominant(dtype, d, q):
    """A key whose probability 2^(q' k) is as far from bf16 as they get, just
    under 2^8."""
    qs, best = _scaled_query(q, d, dtype), (0.0, 0.0)
    for i in range(256):
        k = float(torch.tensor(4.0 + i / 32).bfloat16())
        p = 2.0 ** (qs * k)
        if 64.0 < p < 250.0:
            best = max(best, (abs(float(torch.tensor(p).bfloat16()) / p - 1.0), k))
    assert best[0] > 0.002
    return best[1], 2.0 ** (qs * best[1])


@pytest.mark.parametrize("how,d,g,kernel", [
    ("chunk", 64, 1, 0), ("chunk", 64, 8, 0),
    # the matrix-core decode where it took over from the vector kernel
    ("decode", 64, 1, 0), ("decode", 64, 4, 0), ("decode", 64, 8, 0),
    ("decode", 128, 1, 0), ("decode", 128, 2, 0), ("decode", 128, 4, 0),
    ("decode", 128, 4, 1),
])
def test_the_largest_probability_is_exact(how, d, g, kernel):
    """One key carries nearly all of the weight, and a key of 2^-7 of it sets
    the reference a block before.  With the reference at the maximum the large
    probability is 1, and the output is the float64 one rounded once: within
    half a unit in its last place and the small weight's own rounding.  Against
    the earlier reference it would be rounded too, by 2e-3."""
    say(f"dominant key {how} d={d} G={g}")
    rng = np.random.default_rng(d + g)
    n, step = 416, 32 if how == "chunk" else 16
    top, weight = _dominant("bf16", d, 8.0)
    for at in range(4):
        keys = np.full(n, -30.0)
        pos = 133 + at * step
        keys[pos - step], keys[pos] = 0.0, top
        v = torch.from_numpy(rng.uniform(1.0, 2.0, (n, d)) * rng.choice([-1.0, 1.0], (n, d)))
        q = [8.0] * (3 if how == "chunk" else 1)
        out, _, want, _ = _attend("bf16", d, g, 2, keys, v, q, how, kernel=kernel)
        ulp = torch.exp2(torch.floor(torch.log2(want.abs())) - 7)
        err = ((out[0] - want[:, None]).abs() - 0.5 * ulp[:, None]).max()
        say(f"position {pos}: {float(err):.2e} past half a unit")
        assert err <= 2.0 / weight * 2.0 ** -8 + 1e-6
