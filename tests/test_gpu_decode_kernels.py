"""GPU parity of the bf16 decode kernels on both sides of the automatic choice
at G < 8 (the matrix-core kernel up to two, at head dim 64 four, (query, KV
head) pairs per CU, the vector kernel beyond), and of the vector kernel at the small batches that only
a forced choice gives it."""
import random

import pytest
import torch

from tests._gpu_util import Harness, make_pool, say

pytestmark = pytest.mark.gpu


def _run(g, hkv, n, kind, frames, decodes, d=128):
    say(f"bf16 decode d={d} G={g} hkv={hkv} sessions={n} kernel={kind}")
    kw = dict(n_layers=1, hq=hkv * g, hkv=hkv, d=d, S=4, W=70, dtype="bf16")
    pool = make_pool(**kw, cmax=9, max_sessions=n, n_blocks=n * 6)
    h = Harness(pool, n_sessions=n, **kw)
    pool.set_decode_kernel(kind)
    rnd = random.Random(g * 10 + n)
    for f in range(frames):
        h.frame([rnd.randint(5, 9) for _ in range(n)], [rnd.randint(0, decodes) for _ in range(n)],
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


@pytest.mark.parametrize("g,n,d", [(1, 16, 128), (1, 17, 128), (2, 16, 128), (1, 32, 64),
                                   (1, 33, 64)])
def test_automatic_choice_around_its_line(g, n, d):
    """16 and 17 (head dim 64: 32 and 33) sessions of 32 KV heads: two (four)
    pairs per CU of 256, and one session more."""
    _run(g, 32, n, 0, 3, 2, d)


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
