"""GPU parity of the bf16 decode kernels on both sides of the automatic choice
at G < 8 (the matrix-core kernel up to two, at head dim 64 four, (query, KV
head) pairs per CU, the vector kernel beyond), and of the vector kernel at the
small batches that only a forced choice gives it."""
import random

import pytest
import torch

from tests._gpu_util import Harness, make_pool, say

pytestmark = pytest.mark.gpu


def _kw(g, hkv, d):
    return dict(n_layers=1, hq=hkv * g, hkv=hkv, d=d, S=4, W=70, dtype="bf16")


def _run(g, hkv, n, kind, frames, decodes, d=128, every=False):
    """Frames against the oracle; every: all sessions decode in every round."""
    say(f"bf16 decode d={d} G={g} hkv={hkv} sessions={n} kernel={kind}")
    kw = _kw(g, hkv, d)
    pool = make_pool(**kw, cmax=9, max_sessions=n, n_blocks=n * 6)
    h = Harness(pool, n_sessions=n, **kw)
    pool.set_decode_kernel(kind)
    rnd = random.Random(g * 10 + n)
    for f in range(frames):
        dec = [decodes if every else rnd.randint(0, decodes) for _ in range(n)]
        h.frame([rnd.randint(5, 9) for _ in range(n)], dec,
                n_split=(0, 2, 0, 5)[f % 4], check=f % 3 != 1)
    say(f"max err {h.max_err:.2e}")


@pytest.mark.parametrize("g,d", [(1, 128), (2, 128), (4, 128), (1, 64), (4, 64), (8, 64)])
def test_vector_decode_forced(g, d):
    _run(g, 2, 3, 1, 14, 4, d)


@pytest.mark.parametrize("g", [1, 8])
def test_matrix_core_decode_head_dim_64_stores_what_the_append_stores(g):
    """The fused append of the matrix-core decode at head dim 64 (one dim per
    lane) leaves the pool bytes of append + decode."""
    say(f"d64 fused append G={g}")
    kw = dict(n_layers=2, hq=2 * g, hkv=2, d=64, S=4, W=50, dtype="bf16")
    pools = [make_pool(**kw, cmax=5, max_sessions=3, n_blocks=20) for _ in range(2)]
    for p in pools:
        p.kv.zero_()
    hs = [Harness(p, n_sessions=3, **kw) for p in pools]
    rnd = random.Random(g)
    for f in range(12):
        cl, nd = [rnd.randint(1, 5) for _ in range(3)], [rnd.randint(0, 5) for _ in range(3)]
        hs[0].frame(cl, nd, use_frame_step=True)
        hs[1].frame(cl, nd, use_frame_step=False, fused=False)
        assert torch.equal(pools[0].kv, pools[1].kv), f"pool bytes differ after frame {f}"


def _decode_outputs(g, hkv, n, d, kind):
    """One decode of n sessions of 65 keys: (out, lse)."""
    kw = _kw(g, hkv, d)
    pool = make_pool(**kw, cmax=64, max_sessions=n, n_blocks=n * 10)
    pool.set_decode_kernel(kind)
    sids = [pool.session_open() for _ in range(n)]
    gen = torch.Generator(device="cuda").manual_seed(g)
    draw = lambda t, h: torch.randn((t, h, d), generator=gen, device="cuda").bfloat16()
    pool.plan_begin(sids, [64] * n)
    pool.frame_append_kv(0, draw(64 * n, hkv), draw(64 * n, hkv))
    pool.plan_commit()
    q, k, v = draw(n, hkv * g), draw(n, hkv), draw(n, hkv)
    out, lse = torch.empty_like(q), torch.empty((n, hkv * g), dtype=torch.float32, device="cuda")
    pool.plan_begin(sids, [1] * n)
    pool.attend_decode_append(0, k, v, q, out, lse)
    pool.plan_commit()
    torch.cuda.synchronize()
    return out, lse


@pytest.mark.parametrize("past", [0, 1])
@pytest.mark.parametrize("g,d", [(1, 128), (2, 128), (4, 128), (1, 64), (4, 64)])
def test_automatic_choice_around_its_line(g, d, past):
    """As many sessions of 32 KV heads as make two (head dim 64: four) pairs per
    CU, which the matrix-core kernel takes, and one session more, which the
    vector kernel takes: every session decodes in every round, and one launch is
    bitwise that of the kernel expected and not that of the other one (the
    matrix-core kernel can be forced at head dim 128 only)."""
    hkv = 32
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    n = (4 if d == 64 else 2) * cu // hkv + past
    _run(g, hkv, n, 0, 3, 2, d, every=True)
    auto = _decode_outputs(g, hkv, n, d, 0)
    for kind in (1, 2) if d == 128 else (1,):
        forced = _decode_outputs(g, hkv, n, d, kind)
        same = torch.equal(auto[0], forced[0]) and torch.equal(auto[1], forced[1])
        assert same == (kind == (1 if past else 2)), f"kernel {kind} forced against automatic"


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("n_split", [8, 9, 16, 17, 32])
def test_merge_round_sizes(n_split, dtype, d):
    """Splits at the edges of the merge's rounds of 8, 16 and 32."""
    say(f"merge {n_split} splits {dtype} d={d}")
    kw = dict(n_layers=1, hq=8, hkv=2, d=d, S=4, W=600, dtype=dtype)
    pool = make_pool(**kw, cmax=200, max_sessions=2, n_blocks=110)
    h = Harness(pool, n_sessions=2, **kw)
    for f in range(4):
        h.frame([200, 187], [2, 3], n_split=n_split)
