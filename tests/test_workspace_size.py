"""A call that may take wide KV tiles needs no more workspace than narrow ones
do, so that a workspace or the fixed scratch that served a shape still does."""
import random

import pytest

from paper_2601_21824_amd import binding as dash


def narrow_size(B, H, N, d, sched):
    up = lambda x: (x + 255) // 256 * 256
    bc, bh, nblk = (64 if d == 256 else 128), B * H, -(-N // 64)
    tc = -(-N // bc)
    copies = tc if sched == "partials" else 1
    size = 256 + up(copies * bh * nblk * 64 * d * 4) + 2 * up(bh * N * 4) + up(bh * nblk * 128)
    pad = tc + (tc & 1)  # Symmetric Shift
    g = bc // 64
    cap = max(1 + g * tc + 1, 1 + (pad + 1) * g, 1 + (tc + 1) * g)
    chains = pad + 1
    return size + up(chains * cap * 4) + up((bh + 16) * chains * 8)


@pytest.mark.parametrize("d", [128, 256])
def test_no_more_than_narrow_tiles_need(d):
    rng = random.Random(d)
    for _ in range(3000):
        B, H = rng.choice([1, 2, 4]), int(2 ** rng.uniform(0, 10))
        N = int(2 ** rng.uniform(0, 15))
        for sched in ("auto", "shift", "descending", "partials"):
            assert dash.dash_bwd_workspace_size(B, H, N, d, sched) <= narrow_size(B, H, N, d, sched), (B, H, N, sched)
