"""Plan uploads back to back: small plans are read by the plan kernel from a
ring of pinned buffers, large ones copied from another; neither may be
overwritten before the GPU has read it.  A backlog of matrix products on the
stream holds the plan kernels back while the host goes round each ring."""
import random

import pytest
import torch

from tests._gpu_util import make_pool, say

pytestmark = pytest.mark.gpu

SMALL_SLOTS, LARGE_STAGES = 16, 4   # buffers of the two rings


def test_unsynchronized_plans_store_what_synchronized_ones_store():
    say("plan upload ring")
    n, cmax = 120, 9
    kw = dict(n_layers=1, hq=4, hkv=2, d=64, S=4, W=30, cmax=cmax, max_sessions=n,
              n_blocks=n * 4, dtype="bf16")
    pools = [make_pool(**kw) for _ in range(2)]
    for p in pools:
        p.kv.zero_()
    sids = [[p.session_open() for _ in range(n)] for p in pools]
    gen = torch.Generator(device="cuda").manual_seed(1)
    rows = torch.randn((2, n * cmax, 2, 64), generator=gen, device="cuda").bfloat16()
    a = torch.randn((8192, 8192), generator=gen, device="cuda").bfloat16()
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    rnd = random.Random(4)
    bursts = []
    for i in range(6):
        burst = []
        for j in range(2 * SMALL_SLOTS + 4 if i % 2 == 0 else 2 * LARGE_STAGES + 1):
            k = rnd.choice([1, 7, n]) if i % 2 == 0 else n
            nt = [1] * k if i % 2 == 0 else [rnd.randint(cmax - 3, cmax) for _ in range(k)]
            burst.append((nt, rnd.sample(range(n), k), j % 5 == 4))
        bursts.append(burst)
    for p, ids, sync in zip(pools, sids, (False, True)):
        for i, burst in enumerate(bursts):
            if not sync:
                for _ in range(12):     # about 10 ms
                    torch.mm(a, a, out=b)
                held = torch.cuda.Event()
                held.record()
            for j, (nt, who, on_side) in enumerate(burst):
                if not sync and j == (SMALL_SLOTS // 2 if i % 2 == 0 else LARGE_STAGES - 1):
                    assert not held.query(), "the backlog ended before the host was round the ring"
                s = (side if on_side else torch.cuda.current_stream()).cuda_stream
                p.plan_begin([ids[x] for x in who], nt, stream=s)
                p.frame_append_kv(0, rows[0], rows[1], stream=s)
                p.plan_commit()
                if sync:
                    torch.cuda.synchronize()
            torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
    assert torch.equal(pools[0].kv, pools[1].kv)
