"""Moduli that the RNS engine does not take, because one of the two primes'
squares shares a factor with a channel of its bases: every call runs on the
engine that it would run on without it, with equal results and statuses."""
from __future__ import annotations

import random

import pytest
import torch

from tests.gpu_helpers import dev, gpu_decrypt, host_ints
from tests.test_gpu_rns import _prime, _valu
from workload.limbs import to_limbs

pytestmark = pytest.mark.gpu

CHANNEL = 32749  # the first channel of the bases for p^2 of 2048 bits


@pytest.mark.parametrize("larger", [True, False])
def test_one_half_refused(gpu_ctx, larger):
    from paper_2601_14980_amd import pc2
    a, b = CHANNEL * _prime(1009, 5), _prime(1024 if not larger else 1023, 6)
    assert (a > b) == larger
    n = a * b
    sk = pc2.SecretKey(gpu_ctx, 2048, a, b)
    rng = random.Random(9)
    cs = [rng.randrange(1, n * n) for _ in range(40)]
    ms, rs = [rng.randrange(n) for _ in cs], [rng.randrange(1, n) for _ in cs]

    def calls():
        c = torch.zeros((40, 2 * sk.L), dtype=torch.int32, device="cuda")
        pc2.pc2_encrypt_sk(sk, dev(to_limbs(ms, sk.L)), dev(to_limbs(rs, sk.L)), c)
        st = gpu_ctx.sync()
        return host_ints(c), st, gpu_decrypt(gpu_ctx, sk, cs)

    got = calls()
    with _valu(gpu_ctx):
        assert got == calls()
