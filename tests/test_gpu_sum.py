"""K-way aggregation at the edges of its digit and word tiles: every key class
(odd limb counts among them), counts around a wavefront's elements, factors
at the ends of the range, and factors past it, against the oracle."""
from __future__ import annotations

import random

import pytest

from oracle import paillier as O
from tests.gpu_helpers import gpu_hom_sum
from workload import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbits", [20, 54, 64, 96, 128, 250, 256, 480, 512, 1000, 1024, 1120, 1536,
                                   2016, 2048, 3072, 4096])
@pytest.mark.parametrize("count,K", [(1, 1), (15, 2), (33, 3), (67, 9)])
def test_sum_matches_oracle(gpu_ctx, nbits, count, K):
    from paper_2601_14980_amd import pc2
    p, q = gen.primes_for(51, nbits)
    opk, _ = O.derive_keys(p, q)
    sk = pc2.SecretKey(gpu_ctx, nbits, p, q)
    n2 = opk.n2
    rng = random.Random(nbits + K)
    cvs = [[rng.randrange(n2) for _ in range(count)] for _ in range(K)]
    for j, v in enumerate([1, n2 - 1, 0, n2 - 2]):   # products that end at N - 1, 0, 1 ..
        if j < count:
            for k in range(K):
                cvs[k][j] = v if k == 0 else [1, n2 - 1, 1, 1][j]
    got, st = gpu_hom_sum(gpu_ctx, sk.public, cvs)
    assert st == 0
    want = [O.hom_sum(opk, [cv[j] for cv in cvs]) for j in range(count)]
    assert got == want
    top = (1 << (64 * sk.L)) - 1
    for j, v in ((0, n2), (count - 1, top)):
        cvs[K - 1][j] = v
    got, st = gpu_hom_sum(gpu_ctx, sk.public, cvs)
    assert st == pc2.PC2_E_RANGE
    assert got == [0 if j in (0, count - 1) else want[j] for j in range(count)]
