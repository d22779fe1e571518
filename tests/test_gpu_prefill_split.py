"""GPU parity of the chunk prefill's launch shapes against the float64 oracle:
launches with few workgroups cut each pass's keys into segments joined by the
merge, launches with more workgroups than CUs run their passes longest first.
Tolerances as in the other parity tests (bf16 in, fp32 accumulate, bf16 out)."""
import random

import pytest
import torch

from tests._gpu_util import Harness, make_pool, say

pytestmark = pytest.mark.gpu


def _setup(dtype, hq, hkv, S, W, cmax, n, L=1, d=128):
    kw = dict(n_layers=L, hq=hq, hkv=hkv, d=d, S=S, W=W, dtype=dtype)
    blocks = n * (-(-S // 16) + -(-(W + cmax - 1) // 16)) if W else n * 48
    pool = make_pool(**kw, cmax=cmax, max_sessions=n, n_blocks=blocks, max_len=0 if W else 760)
    return pool, Harness(pool, n_sessions=n, **kw)


@pytest.mark.parametrize("dtype,g,S,W,rows", [
    ("bf16", 8, 4, 520, 0),      # 4+ segments once the window is full, ring wraps
    ("bf16", 8, 4, 520, 256),
    ("bf16", 4, 20, 400, 0),     # sinks span two blocks, all in the first segment
    ("bf16", 1, 0, 390, 0),
    ("bf16", 8, 4, None, 0),     # unbounded: segments grow with the session
    ("fp8", 8, 4, 520, 0),
    ("fp8", 2, 17, 400, 256),
    ("bf16-d64", 8, 4, 520, 0),  # head dim 64: half the slices, another LDS swizzle
    ("bf16-d64", 2, 20, None, 256),
    ("bf16-d64", 1, 0, 390, 128),
    ("f32", 8, 4, 390, 0),       # fp32: 64-row passes, several per chunk
    ("f32", 1, 20, None, 0),
    ("f32-d64", 4, 17, 400, 0),
    ("f32-d64", 2, 0, 33, 0),    # chunks longer than the window
])
def test_split_prefill_matches_oracle(dtype, g, S, W, rows):
    """Two sessions of very different lengths in one plan: the short one has
    segments that hold no stage, and single-stage ones; every frame's outputs
    and log-sum-exps are checked from an empty pool on, so the number of
    segments runs from one to the largest this window gives."""
    say(f"split prefill {dtype} G={g} S={S} W={W} rows={rows}")
    dtype, _, d64 = dtype.partition("-")
    pool, h = _setup(dtype, 2 * g, 2, S, W, 60, 2, d=64 if d64 else 128)
    if rows:
        pool.set_prefill_pass_rows(rows)
    pool.set_timing(True)
    pool.kernel_times()
    rnd = random.Random(g * 100 + S)
    for f in range(12):
        pool.kernel_times()
        h.frame([rnd.randint(40, 60), rnd.randint(2, 9)], [1, 0], n_split=1, use_frame_step=f % 3 > 0)
        merges = pool.kernel_times()["merge"][0]
    assert merges == (W != 33), "the last frame's prefill ran unsplit"
    say(f"max err {h.max_err:.2e}")


@pytest.mark.parametrize("dtype,g,d,W,n,c,split", [
    ("bf16", 4, 128, None, 1, 700, False),  # a long chunk's partial rows cost more than the segments save
    ("bf16", 4, 128, 400, 16, 25, False),   # so do those of many sessions over a short window
    ("bf16", 4, 128, None, 1, 60, False),   # two stages: nothing to cut
    ("bf16", 4, 128, 2000, 2, 25, True),    # few rows over a long window
    ("f32", 1, 128, 128, 1, 25, True),      # ten slow blocks
    ("f32", 1, 64, 128, 1, 25, False),      # ten that cost about a merge and its launch
])
def test_segments_are_cut_where_they_save_more_than_the_merge_costs(dtype, g, d, W, n, c, split):
    say(f"prefill split {dtype} G={g} d={d} W={W} sessions={n} chunk={c}")
    kw = dict(n_layers=1, hq=8 * g, hkv=8, d=d, S=0, W=W, dtype=dtype)
    io = torch.float32 if dtype == "f32" else torch.bfloat16
    blocks = n * -(-((W or 0) + c + 31) // 16)
    pool = make_pool(**kw, cmax=c, max_sessions=n, n_blocks=blocks, max_len=0 if W else c)
    sids = [pool.session_open() for _ in range(n)]
    q = torch.zeros((n * c, 8 * g, d), dtype=io, device="cuda")
    k, o = torch.zeros((n * c, 8, d), dtype=io, device="cuda"), torch.empty_like(q)
    for _ in range(-(-(W or 0) // c)):
        pool.plan_begin(sids, [c] * n)
        pool.frame_append_kv(0, k, k)
        pool.plan_commit()
    pool.set_timing(True)
    pool.plan_begin(sids, [c] * n)
    pool.frame_append_kv(0, k, k)
    pool.attend_chunk_prefill(0, q, o)
    pool.plan_commit()
    assert (pool.kernel_times()["prefill_merge"][0] == 1) == split


def test_merge_times_tell_the_chunk_from_the_decode():
    """One split chunk and two split decodes of two layers: class 3 holds the
    merges of both, the chunk's share is told apart, and both reset."""
    say("merge times")
    pool, h = _setup("bf16", 16, 2, 4, 520, 60, 1, L=2)
    for _ in range(9):
        h.frame([60], [0], check=False)
    pool.set_timing(True)
    h.frame([60], [2], n_split=3)
    t = pool.kernel_times()
    assert (t["prefill"][0], t["decode"][0]) == (2, 4)
    assert (t["merge"][0], t["prefill_merge"][0]) == (2 + 4, 2)
    assert 0 < t["prefill_merge"][1] < t["merge"][1]
    assert pool.kernel_times()["merge"] == pool.kernel_times()["prefill_merge"] == (0, 0.0)


def test_many_ragged_passes_longest_first():
    """40 sessions x 8 KV heads: more passes than CUs, of mixed lengths."""
    say("longest first, 40 sessions")
    pool, h = _setup("bf16", 8, 8, 4, 70, 9, 40)
    rnd = random.Random(5)
    for f in range(6):
        h.frame([rnd.randint(2, 9) for _ in range(40)], [0] * 40)
    say(f"max err {h.max_err:.2e}")


def test_fused_append_of_a_large_fp8_batch_stores_what_the_append_stores():
    """Enough workgroups that the fp8 prefill is not split and carries the
    append: pool bytes equal those of append + prefill while the sessions grow
    past the stages a workgroup copies first and through the window's wrap."""
    say("fp8 fused append, 34 sessions x 4 kv heads")
    n, W, cmax = 34, 300, 32
    pools = []
    for fused in (True, False):
        pool, h = _setup("fp8", 32, 4, 4, W, cmax, n, L=2)
        pool.kv.zero_()
        pool.poison_dead()
        pools.append((pool, h, fused))
        pool.set_timing(True)
    rnd = random.Random(2)
    for f in range(13):
        cl = [rnd.randint(25, 32) for _ in range(n)]
        gen = torch.Generator(device="cuda").manual_seed(f)
        q, k, v = (torch.randn((2, sum(cl), hh, 128), generator=gen, device="cuda").bfloat16()
                   for hh in (32, 4, 4))
        outs = []
        for pool, h, fused in pools:
            o = torch.empty_like(q)
            if fused:
                pool.frame_step(h.sids, cl, [0] * n, q, k, v, o)
            else:
                pool.plan_begin(h.sids, cl)
                for l in range(2):
                    pool.frame_append_kv(l, k[l], v[l])
                    pool.attend_chunk_prefill(l, q[l], o[l])
                pool.plan_commit()
            outs.append(o)
        torch.cuda.synchronize()
        assert torch.equal(pools[0][0].kv, pools[1][0].kv), f"pool bytes differ after frame {f}"
        assert torch.equal(*outs)
    assert pools[0][0].kernel_times()["append"][0] == 0, "the frames did not fuse the append"
