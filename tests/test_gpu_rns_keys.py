"""Batches and runner launches of jobs under many keys, where the engine is
chosen for the launch: results against the one-call entry points and the
plaintexts, and no slower than the persistent kernel that holds all keys."""
from __future__ import annotations

import random

import pytest
import torch

from tests.gpu_helpers import dev, host_ints
from tests.test_gpu_rns import _prime, _valu
from workload.limbs import to_limbs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def keys(gpu_ctx):
    from paper_2601_14980_amd import pc2
    ps = [_prime(1024, s) for s in range(10, 19)]
    return [pc2.SecretKey(gpu_ctx, 2048, a, b) for a, b in zip(ps, ps[1:])]


def _jobs(pc2, keys, counts, op, seed=1):
    rng = random.Random(seed)
    jobs, want = [], []
    for sk, count in zip(keys, counts):
        ms = [rng.randrange(sk.n) for _ in range(min(count, 50))]
        rs = [rng.randrange(1, sk.n) for _ in ms]
        reps = -(-count // len(ms))
        m, r = dev(to_limbs(ms, sk.L)), dev(to_limbs(rs, sk.L))
        c = torch.zeros((len(ms), 2 * sk.L), dtype=torch.int32, device="cuda")
        pc2.pc2_encrypt(sk.public, m, r, c)
        m, r, c = (t.repeat(reps, 1)[:count].contiguous() for t in (m, r, c))
        if op == "decrypt":
            jobs.append(dict(op=pc2.PC2_OP_DECRYPT, sk=sk, c=c, out=torch.zeros_like(m)))
            want.append(m)
        else:
            jobs.append(dict(op=pc2.PC2_OP_ENCRYPT, pk=sk.public, m=m, r=r,
                             out=torch.zeros_like(c)))
            want.append(c)
    return jobs, want


def _launcher(pc2, ctx, jobs, kind):
    """A function that runs the jobs, and what to close."""
    if kind == "batch":
        b = pc2.Batch(ctx, jobs)
        return b.run, b
    size = [pc2.runner_group_size(j["sk"].public if "sk" in j else j["pk"], j["op"]) for j in jobs]
    n = [-(-j["out"].shape[0] // s) for j, s in zip(jobs, size)]
    r = pc2.Runner(ctx, jobs[0]["op"], 2048, len(jobs), sum(n))
    return (lambda: r.launch(jobs, [0] * len(jobs), n)), r


# few elements under every key; one key that the engine takes beside small ones;
# all large
@pytest.mark.parametrize("kind", ["batch", "runner"])
@pytest.mark.parametrize("op,counts", [
    ("decrypt", (16,) * 8), ("decrypt", (1, 40, 7)), ("decrypt", (20000, 16, 5, 33)),
    ("decrypt", (16, 5000, 3, 9001, 2, 1)), ("encrypt", (16,) * 8), ("encrypt", (3900,) * 4),
    ("encrypt", (100, 9000, 7)), ("encrypt", (9000, 8500))])
def test_results(gpu_ctx, keys, kind, op, counts):
    from paper_2601_14980_amd import pc2
    jobs, want = _jobs(pc2, keys, counts, op)
    run, handle = _launcher(pc2, gpu_ctx, jobs, kind)
    for _ in range(2):
        run()
        assert gpu_ctx.sync() == 0
        for j, w in zip(jobs, want):
            assert torch.equal(j["out"], w)
            j["out"].zero_()
    handle.close()
    assert host_ints(want[0][:1])  # (the inputs were not overwritten)


@pytest.mark.parametrize("kind", ["batch", "runner"])
def test_many_keys_of_few_elements_are_not_a_sequence_each(gpu_ctx, keys, kind):
    """Eight keys x 16 decryptions: 27 ms as eight launch sequences, 16.5 in the
    persistent kernel."""
    from paper_2601_14980_amd import pc2

    def ms():
        jobs, _ = _jobs(pc2, keys, (16,) * 8, "decrypt")
        run, handle = _launcher(pc2, gpu_ctx, jobs, kind)
        times = []
        for _ in range(4):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            torch.cuda.synchronize()
            a.record()
            run()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        handle.close()
        return min(times[1:])

    got = ms()
    with _valu(gpu_ctx):
        want = ms()
    assert got < 1.25 * want


# keys of other classes beside one that the engine takes: on the VALU kernel, and
# with the matrix cores asked for
@pytest.mark.parametrize("modmul,other,counts", [
    ("AUTO", 256, (9000, 700)), ("AUTO", 1024, (9000, 700)), ("AUTO", 1024, (4000, 20000)),
    ("MFMA", 512, (9000, 9000)), ("MFMA", 512, (100, 5000)), ("MFMA", 256, (4000, 5000))])
def test_other_classes(gpu_ctx, keys, modmul, other, counts):
    from paper_2601_14980_amd import pc2
    a, b = _prime(other // 2, 40), _prime(other // 2, 41)
    sk = pc2.SecretKey(gpu_ctx, other, a, b)
    jobs, want = _jobs(pc2, [keys[0], sk], counts, "encrypt")
    gpu_ctx.set_option(pc2.PC2_OPT_MODMUL, getattr(pc2, "PC2_MODMUL_" + modmul))
    try:
        for kind in ("batch", "runner") if other != 512 else ("batch",):
            run, handle = _launcher(pc2, gpu_ctx, jobs, kind)
            run()
            assert gpu_ctx.sync() == 0
            for j, w in zip(jobs, want):
                assert torch.equal(j["out"], w)
                j["out"].zero_()
            handle.close()
    finally:
        gpu_ctx.set_option(pc2.PC2_OPT_MODMUL, pc2.PC2_MODMUL_AUTO)


def test_class_without_element_groups(gpu_ctx, keys):
    """512-bit keys have no persistent kernel: with the matrix cores asked for, a
    batch of few elements under one is refused, and so is a runner's launch."""
    from paper_2601_14980_amd import pc2
    sk = pc2.SecretKey(gpu_ctx, 512, _prime(256, 40), _prime(256, 41))
    jobs, _ = _jobs(pc2, [keys[0], sk], (100, 100), "encrypt")
    r = pc2.Runner(gpu_ctx, pc2.PC2_OP_ENCRYPT, 2048, 2, 64)
    gpu_ctx.set_option(pc2.PC2_OPT_MODMUL, pc2.PC2_MODMUL_MFMA)
    try:
        for call in (lambda: pc2.Batch(gpu_ctx, jobs), lambda: pc2.Batch(gpu_ctx, jobs[1:]),
                     lambda: r.launch(jobs[1:], [0], [1])):
            with pytest.raises(pc2.PC2Error) as e:
                call()
            assert e.value.status == pc2.PC2_E_UNSUPPORTED
    finally:
        gpu_ctx.set_option(pc2.PC2_OPT_MODMUL, pc2.PC2_MODMUL_AUTO)
    r.close()
