"""Encryptions of few elements (a workgroup of several wavefronts per element):
every key class that has the kernel, counts on both sides of one round of its
workgroups, every table width, and the ends of the input ranges, against the
oracle and the VALU engine.  Results are integers: equal or wrong."""
from __future__ import annotations

import random

import pytest

from oracle import paillier as O
from tests.gpu_helpers import gpu_encrypt
from workload import gen

pytestmark = pytest.mark.gpu


def _case(ctx, nbits, count):
    from paper_2601_14980_amd import pc2
    p, q = gen.primes_for(41, nbits)
    opk, _ = O.derive_keys(p, q)
    n = opk.n
    rng = random.Random(nbits + count)
    ms = ([n - 1, 0, 1, n // 3] + [rng.randrange(n) for _ in range(count)])[:count]
    rs = ([n - 1, 1, n - 1, 2] + [rng.randrange(1, n) for _ in range(count)])[:count]
    return pc2.SecretKey(ctx, nbits, p, q), opk, ms, rs


@pytest.mark.parametrize("nbits", [1024, 1120, 1536, 2048, 3072, 4096])
@pytest.mark.parametrize("count", [1, 5])
def test_few_match_oracle(gpu_ctx, nbits, count):
    sk, opk, ms, rs = _case(gpu_ctx, nbits, count)
    got, st = gpu_encrypt(gpu_ctx, sk.public, ms, rs)
    assert st == 0 and got == [O.encrypt(opk, m, r) for m, r in zip(ms, rs)]


@pytest.mark.parametrize("nbits,count", [(1024, 512), (1024, 513), (2048, 256), (2048, 257),
                                         (3072, 256), (4096, 257)])
def test_rounds_match_valu_engine(gpu_ctx, nbits, count):
    from paper_2601_14980_amd import pc2
    sk, opk, ms, rs = _case(gpu_ctx, nbits, count)
    ms[7], rs[8], rs[count - 1] = opk.n, 0, opk.n + 1
    got, st = gpu_encrypt(gpu_ctx, sk.public, ms, rs)
    gpu_ctx.set_option(pc2.PC2_OPT_MODMUL, pc2.PC2_MODMUL_VALU)
    try:
        want, st2 = gpu_encrypt(gpu_ctx, sk.public, ms, rs)
    finally:
        gpu_ctx.set_option(pc2.PC2_OPT_MODMUL, pc2.PC2_MODMUL_AUTO)
    assert st == st2 == pc2.PC2_E_RANGE and got == want
    assert got[7] == got[8] == got[count - 1] == 0


@pytest.mark.parametrize("window", [2, 3, 4, 5, 6])
def test_windows(gpu_ctx, window):
    from paper_2601_14980_amd import pc2
    sk, opk, ms, rs = _case(gpu_ctx, 1024, 4)
    gpu_ctx.set_option(pc2.PC2_OPT_WINDOW, window)
    try:
        got, st = gpu_encrypt(gpu_ctx, sk.public, ms, rs, m_limbs=sk.L)
    finally:
        gpu_ctx.set_option(pc2.PC2_OPT_WINDOW, 0)
    assert st == 0 and got == [O.encrypt(opk, m, r) for m, r in zip(ms, rs)]
