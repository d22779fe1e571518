"""Plan uploads back to back: small plans are read by the plan kernel from a
ring of pinned buffers, large ones copied from another; neither may be
overwritten before the GPU has read it."""
import random

import pytest
import torch

from tests._gpu_util import make_pool, say

pytestmark = pytest.mark.gpu


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
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    rnd = random.Random(4)
    plans = []
    for i in range(90):   # one token each (small), a few sessions, or the whole batch (large)
        k = rnd.choice([1, 7, n, n])
        top = 1 if rnd.random() < 0.6 else cmax
        plans.append(([rnd.randint(1, top) for _ in range(k)], rnd.sample(range(n), k), i % 5 == 4))
    for p, ids, sync in zip(pools, sids, (False, True)):
        for nt, who, on_side in plans:
            s = (side if on_side else torch.cuda.current_stream()).cuda_stream
            p.plan_begin([ids[i] for i in who], nt, stream=s)
            p.frame_append_kv(0, rows[0], rows[1], stream=s)
            p.plan_commit()
            if sync:
                torch.cuda.synchronize()
        torch.cuda.synchronize()
    assert torch.equal(pools[0].kv, pools[1].kv)
