"""A tile asked for by option is a tile of the VALU engine's encryption kernels,
at every count: results and, from the time they take, the kernels."""
from __future__ import annotations

import random

import pytest
import torch

from tests.gpu_helpers import dev
from tests.test_gpu_rns import _key, _valu
from workload.limbs import to_limbs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lanes", [2, 4])
@pytest.mark.parametrize("count", [500, 9000])
def test_tile_at_both_sides_of_the_other_engines(gpu_ctx, lanes, count):
    from paper_2601_14980_amd import pc2
    sk, _, _ = _key(gpu_ctx, 1024)
    rng = random.Random(count)
    ms, rs = ([rng.randrange(1, sk.n) for _ in range(50)] for _ in range(2))
    m, r = (dev(to_limbs(v, sk.L)).repeat(count // 50, 1) for v in (ms, rs))

    def go():
        c = torch.zeros((count, 2 * sk.L), dtype=torch.int32, device="cuda")
        times = []
        for _ in range(4):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            pc2.pc2_encrypt(sk.public, m, r, c)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        assert gpu_ctx.sync() == 0
        return c, min(times[1:])

    want, free = go()
    gpu_ctx.set_option(pc2.PC2_OPT_TILE, lanes)
    try:
        got, tiled = go()
        with _valu(gpu_ctx):
            _, valu = go()
    finally:
        gpu_ctx.set_option(pc2.PC2_OPT_TILE, 0)
    assert torch.equal(got, want)
    # 1024 bits: 9.5 ms and more on the VALU engine, 1.6 and 4.8 on the others
    assert 0.8 * valu < tiled < 1.25 * valu and free < 0.8 * valu
