"""Keys whose modulus is shorter than the size that they are declared with
(15 <= n < 2^nbits, pq < 2^nbits), on the RNS engine, in every call that ends in
its output conversion: against the oracle and the VALU engine.  Results are
integers: equal or wrong."""
from __future__ import annotations

import random

import numpy as np
import pytest
import torch

from oracle import paillier as O
from tests.gpu_helpers import (dev, gpu_decrypt, gpu_enc_sum_dec, gpu_encrypt, gpu_scalar_mul,
                               host_ints)
from tests.test_gpu_rns import _prime, _valu
from workload.limbs import to_limbs

pytestmark = pytest.mark.gpu


# n^2's 28-bit limbs end, in blocks of eight, where the last word of the declared
# size begins, just below it, or far below
@pytest.mark.parametrize("nbits,bits", [
    (512, 434), (512, 430), (512, 260), (1024, 994), (1024, 990), (1024, 700),
    (2048, 2010), (2048, 2002), (2048, 1990), (2048, 1800), (2048, 600),
    (3072, 3010), (3072, 2900), (4096, 4018), (4096, 3000)])
def test_short_public_key(gpu_ctx, nbits, bits):
    from paper_2601_14980_amd import pc2
    rng = random.Random(nbits + bits)
    n = rng.getrandbits(bits) | 1 | (3 << (bits - 2))
    n2 = n * n
    pk = pc2.PublicKey(gpu_ctx, nbits, n)
    L = pk.L
    # encryptions, of a count that takes the engine, alone and as a batch
    count = {512: 4100, 1024: 3600, 2048: 3850, 3072: 6660, 4096: 7430}[nbits]
    ms = [0, 1, n - 1] + [rng.randrange(n) for _ in range(37)]
    rs = [n - 1, 1, 2] + [rng.randrange(1, n) for _ in range(37)]
    want = [(1 + m * n) * pow(r, n, n2) % n2 for m, r in zip(ms, rs)]
    reps = -(-count // 40)
    got, st = gpu_encrypt(gpu_ctx, pk, ms * reps, rs * reps)
    assert st == 0 and got == want * reps
    if nbits != 512:  # (no batches under 512-bit keys)
        job = dict(op=pc2.PC2_OP_ENCRYPT, pk=pk, m=dev(to_limbs(ms * reps, L)),
                   r=dev(to_limbs(rs * reps, L)),
                   out=torch.zeros((40 * reps, 2 * L), dtype=torch.int32, device="cuda"))
        b = pc2.Batch(gpu_ctx, [job])
        b.run()
        assert gpu_ctx.sync() == 0 and host_ints(job["out"]) == want * reps
        b.close()
    # scalar products and a mat-vec
    cs = [0, 1, n2 - 1] + [rng.randrange(n2) for _ in range(33)]
    ks = [3, 0, (1 << 64) - 1] + [rng.getrandbits(64) for _ in range(33)]
    got, st = gpu_scalar_mul(gpu_ctx, pk, cs, ks)
    assert st == 0 and got == [pow(c, k, n2) for c, k in zip(cs, ks)]
    B = np.random.default_rng(bits).integers(0, 1 << 20, size=(5, 3), dtype=np.uint64)
    mv = pc2.MatVec(pk, 3, 20, 8)
    mv.load(dev(to_limbs(cs[2:5], 2 * L)))
    out = torch.full((5, 2 * L), -1, dtype=torch.int32, device="cuda")
    mv.apply(torch.from_numpy(B.view(np.int64)).cuda(), out)
    assert gpu_ctx.sync() == 0
    assert host_ints(out) == [
        pow(cs[2], int(r[0]), n2) * pow(cs[3], int(r[1]), n2) * pow(cs[4], int(r[2]), n2) % n2
        for r in B]
    mv.close()


# a q^2 whose limbs end below the last word of p^2
@pytest.mark.parametrize("nbits,pbits,qbits", [
    (1024, 512, 430), (1024, 512, 300), (2048, 1024, 990), (2048, 1024, 950),
    (2048, 1024, 900), (2048, 1024, 600), (4096, 2048, 1900)])
def test_short_second_prime(gpu_ctx, nbits, pbits, qbits):
    from paper_2601_14980_amd import pc2
    p, q = _prime(pbits, 1), _prime(qbits, 2)
    n = p * q
    opk, _ = O.derive_keys(p, q)
    sk = pc2.SecretKey(gpu_ctx, nbits, p, q)
    rng = random.Random(qbits)
    ms = [0, 1, n - 1] + [rng.randrange(n) for _ in range(37)]
    rs = [n - 1, 1, 2] + [rng.randrange(1, n) for _ in range(37)]
    cs = [O.encrypt(opk, m, r) for m, r in zip(ms, rs)]
    assert gpu_decrypt(gpu_ctx, sk, cs) == (ms, 0)
    job = dict(op=pc2.PC2_OP_DECRYPT, sk=sk, c=dev(to_limbs(cs, 2 * sk.L)),
               out=torch.zeros((40, sk.L), dtype=torch.int32, device="cuda"))
    b = pc2.Batch(gpu_ctx, [job])
    b.run()
    assert gpu_ctx.sync() == 0 and host_ints(job["out"]) == ms
    b.close()
    bad = [cs[0], p * 3, q * q, cs[1]]
    got = gpu_decrypt(gpu_ctx, sk, bad)
    with _valu(gpu_ctx):
        assert got == gpu_decrypt(gpu_ctx, sk, bad)


def test_short_key_fused(gpu_ctx):
    from paper_2601_14980_amd import pc2
    p, q = _prime(1000, 3), _prime(990, 4)
    n = p * q
    sk = pc2.SecretKey(gpu_ctx, 2048, p, q)
    rng = random.Random(7)
    reps = 97  # 3880 elements: encryptions on the engine
    ms = [[rng.randrange(n // 4) for _ in range(40)] * reps for _ in range(3)]
    rs = [[rng.randrange(1, n) for _ in range(40)] * reps for _ in range(3)]
    got, st = gpu_enc_sum_dec(gpu_ctx, sk, ms, rs)
    assert st == 0 and got == [sum(v) for v in zip(*ms)]
