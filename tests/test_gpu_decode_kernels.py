"""GPU parity of the bf16 decode kernels on both sides of the automatic choice
at G < 8 (the matrix-core kernel up to two (query, KV head) pairs per CU, the
vector kernel beyond), and of the vector kernel at the small batches that only
a forced choice gives it."""
import random

import pytest

from tests._gpu_util import Harness, make_pool, say

pytestmark = pytest.mark.gpu


def _run(g, hkv, n, kind, frames, decodes):
    say(f"bf16 decode G={g} hkv={hkv} sessions={n} kernel={kind}")
    kw = dict(n_layers=1, hq=hkv * g, hkv=hkv, d=128, S=4, W=70, dtype="bf16")
    pool = make_pool(**kw, cmax=9, max_sessions=n, n_blocks=n * 6)
    h = Harness(pool, n_sessions=n, **kw)
    pool.set_decode_kernel(kind)
    rnd = random.Random(g * 10 + n)
    for f in range(frames):
        h.frame([rnd.randint(5, 9) for _ in range(n)], [rnd.randint(0, decodes) for _ in range(n)],
                n_split=(0, 2, 0, 5)[f % 4], check=f % 3 != 1)
    say(f"max err {h.max_err:.2e}")


@pytest.mark.parametrize("g", [1, 2, 4])
def test_vector_decode_forced(g):
    _run(g, 2, 3, 1, 14, 4)


@pytest.mark.parametrize("g,n", [(1, 16), (1, 17), (2, 16)])
def test_automatic_choice_around_its_line(g, n):
    """16 and 17 sessions of 32 KV heads: 512 and 544 pairs."""
    _run(g, 32, n, 0, 3, 2)
