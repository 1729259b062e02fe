"""Device memory of batches and runners on the RNS engine: bounded whatever the
jobs' lengths, and without room for the engine's tables the jobs run on the
persistent kernels."""
from __future__ import annotations

import random

import pytest
import torch

from tests.gpu_helpers import dev
from tests.test_gpu_rns import _key, _valu
from workload.limbs import to_limbs

pytestmark = pytest.mark.gpu


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _jobs(pc2, sk, counts, op):
    """Jobs over 50 elements repeated, and the outputs they have to give."""
    rng = random.Random(len(counts))
    ms, rs = ([rng.randrange(1, sk.n) for _ in range(50)] for _ in range(2))
    m, r = dev(to_limbs(ms, sk.L)), dev(to_limbs(rs, sk.L))
    c = torch.zeros((50, 2 * sk.L), dtype=torch.int32, device="cuda")
    pc2.pc2_encrypt(sk.public, m, r, c)
    jobs, want = [], []
    for count in counts:
        a, b, d = (t.repeat(-(-count // 50), 1)[:count].contiguous() for t in (m, r, c))
        if op == "decrypt":
            jobs.append(dict(op=pc2.PC2_OP_DECRYPT, sk=sk, c=d, out=torch.zeros_like(a)))
            want.append(a)
        else:
            jobs.append(dict(op=pc2.PC2_OP_ENCRYPT, pk=sk.public, m=a, r=b,
                             out=torch.zeros_like(d)))
            want.append(d)
    return jobs, want


def _make(pc2, ctx, sk, jobs, kind):
    """(run, handle, bytes that the handle took)"""
    free = _free()
    if kind == "batch":
        b = pc2.Batch(ctx, jobs)
        return b.run, b, free - _free()
    size = pc2.runner_group_size(sk.public, jobs[0]["op"])
    n = [-(-j["out"].shape[0] // size) for j in jobs]
    r = pc2.Runner(ctx, jobs[0]["op"], sk.nbits, len(jobs), sum(n))
    return (lambda: r.launch(jobs, [0] * len(jobs), n)), r, free - _free()


def _check(ctx, run, jobs, want):
    run()
    assert ctx.sync() == 0
    for j, w in zip(jobs, want):
        assert torch.equal(j["out"], w)


# one job and several past the 2^18 positions of a part, cut inside a job and
# between two
@pytest.mark.parametrize("op", ["encrypt", "decrypt"])
@pytest.mark.parametrize("counts", [(262144,), (262145,), (262100, 40, 7), (200000, 400000)])
def test_long_jobs(gpu_ctx, op, counts):
    from paper_2601_14980_amd import pc2
    sk, _, _ = _key(gpu_ctx, 1024)
    jobs, want = _jobs(pc2, sk, counts, op)
    for kind in ("batch", "runner"):
        run, handle, _ = _make(pc2, gpu_ctx, sk, jobs, kind)
        _check(gpu_ctx, run, jobs, want)
        handle.close()
        for j in jobs:
            j["out"].zero_()


@pytest.mark.parametrize("op", ["encrypt", "decrypt"])
def test_memory_does_not_grow_with_the_jobs(gpu_ctx, op):
    from paper_2601_14980_amd import pc2
    sk, _, _ = _key(gpu_ctx, 1024)
    took = []
    for count in (1 << 18, 1 << 20):
        jobs, _ = _jobs(pc2, sk, (count,), op)
        _, handle, nbytes = _make(pc2, gpu_ctx, sk, jobs, "batch")
        handle.close()
        took.append(nbytes)
    assert took[1] < took[0] + (64 << 20)


@pytest.mark.parametrize("op", ["encrypt", "decrypt"])
@pytest.mark.parametrize("kind", ["batch", "runner"])
def test_without_room_for_the_engine(gpu_ctx, op, kind):
    """All but a little of the device's memory is taken: what is left holds the
    persistent kernels' scratch, not the engine's."""
    from paper_2601_14980_amd import pc2
    sk, _, _ = _key(gpu_ctx, 2048)
    jobs, want = _jobs(pc2, sk, (9000, 300), op)
    _, handle, full = _make(pc2, gpu_ctx, sk, jobs, kind)
    handle.close()
    with _valu(gpu_ctx):
        _, handle, _ = _make(pc2, gpu_ctx, sk, jobs, "batch")
    handle.close()
    torch.cuda.empty_cache()
    hog = torch.empty(_free() - full + (96 << 20), dtype=torch.uint8, device="cuda")
    try:
        run, handle, _ = _make(pc2, gpu_ctx, sk, jobs, kind)
        _check(gpu_ctx, run, jobs, want)
        handle.close()
    finally:
        del hog
        torch.cuda.empty_cache()
