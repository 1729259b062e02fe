"""The residue-number-system engine (keys from 512 bits) against the VALU
engine on the same context and against the oracle: counts on both sides of
a block of 32 elements and of every choice that a call's shape depends on, key
sizes of every tile count, and the values at the ends of the input ranges.
Results are integers: equal or wrong."""
from __future__ import annotations

import random

import numpy as np
import pytest
import torch

from oracle import paillier as O
from tests.gpu_helpers import (dev, gpu_decrypt, gpu_encrypt, gpu_scalar_mul, host_ints)
from workload import gen
from workload.limbs import to_limbs

pytestmark = pytest.mark.gpu


def _key(ctx, nbits, seed=31):
    from paper_2601_14980_amd import pc2
    p, q = gen.primes_for(seed, nbits)
    opk, osk = O.derive_keys(p, q)
    return pc2.SecretKey(ctx, nbits, p, q), opk, osk


class _valu:
    """Every product of the calls inside on the VALU engine."""

    def __init__(self, ctx):
        self.ctx = ctx

    def __enter__(self):
        from paper_2601_14980_amd import pc2
        self.ctx.set_option(pc2.PC2_OPT_MODMUL, pc2.PC2_MODMUL_VALU)

    def __exit__(self, *a):
        from paper_2601_14980_amd import pc2
        self.ctx.set_option(pc2.PC2_OPT_MODMUL, pc2.PC2_MODMUL_AUTO)


def _ms_rs(n, count, seed):
    rng = random.Random(seed)
    ms = [0, 1, n - 1, n // 2][:count] + [rng.randrange(n) for _ in range(count - 4)]
    rs = [n - 1, 1, n - 1, 2][:count] + [rng.randrange(1, n) for _ in range(count - 4)]
    return ms, rs


# counts from which a public-key encryption takes the engine (one element
# below, at it), and a ragged one of several groups
@pytest.mark.parametrize("nbits,count", [
    (512, 4096), (512, 4097), (480, 9001), (1024, 3583), (1024, 3584), (1120, 3617),
    (1024, 12001), (1536, 3871), (2048, 3839), (2048, 3841),
    (2048, 16385), (2048, 20001), (3072, 6657), (4096, 7425)])
def test_encrypt_counts(gpu_ctx, nbits, count):
    sk, opk, _ = _key(gpu_ctx, nbits)
    ms, rs = _ms_rs(opk.n, count, count)
    got, st = gpu_encrypt(gpu_ctx, sk.public, ms, rs)
    assert st == 0
    with _valu(gpu_ctx):
        want, st = gpu_encrypt(gpu_ctx, sk.public, ms, rs)
    assert st == 0 and got == want
    for i in (0, 1, 2, count - 1):
        assert got[i] == O.encrypt(opk, ms[i], rs[i])


@pytest.mark.parametrize("window", [2, 3, 4, 5, 6])
def test_encrypt_windows(gpu_ctx, window):
    from paper_2601_14980_amd import pc2
    sk, opk, _ = _key(gpu_ctx, 1024)
    ms, rs = _ms_rs(opk.n, 4000, window)
    want, st = gpu_encrypt(gpu_ctx, sk.public, ms, rs)
    gpu_ctx.set_option(pc2.PC2_OPT_WINDOW, window)
    try:
        got, st2 = gpu_encrypt(gpu_ctx, sk.public, ms, rs)
        dec, st3 = gpu_decrypt(gpu_ctx, sk, got[:40])
    finally:
        gpu_ctx.set_option(pc2.PC2_OPT_WINDOW, 0)
    assert st == st2 == st3 == 0 and got == want and dec == ms[:40]


@pytest.mark.parametrize("nbits,count", [
    (512, 1), (512, 5632), (512, 5633), (1024, 1), (1024, 33), (1120, 31), (1536, 65),
    (2048, 32), (2048, 129), (2048, 5000), (2048, 8193),
    (2048, 10001), (3072, 31), (3072, 4097), (4096, 5)])
def test_decrypt_and_key_holder_counts(gpu_ctx, nbits, count):
    from paper_2601_14980_amd import pc2
    sk, opk, osk = _key(gpu_ctx, nbits)
    n, n2 = opk.n, opk.n2
    ms, rs = _ms_rs(n, count, nbits + count)
    c = torch.zeros((count, 2 * sk.L), dtype=torch.int32, device="cuda")
    pc2.pc2_encrypt_sk(sk, dev(to_limbs(ms, sk.L)), dev(to_limbs(rs, sk.L)), c)
    assert gpu_ctx.sync() == 0
    cs = host_ints(c)
    for i in {0, min(2, count - 1), count - 1}:
        assert cs[i] == O.encrypt(opk, ms[i], rs[i])
    got, st = gpu_decrypt(gpu_ctx, sk, cs)
    assert st == 0 and got == ms
    # values that are no ciphertexts: what the VALU engine makes of them
    odd = ([n2 - 1, 1, n + 1, n2 - n] + cs)[:count]
    got, st = gpu_decrypt(gpu_ctx, sk, odd)
    with _valu(gpu_ctx):
        want, st2 = gpu_decrypt(gpu_ctx, sk, odd)
    assert st == st2 and got == want


@pytest.mark.parametrize("nbits", [1024, 2048, 4096])
def test_bad_inputs(gpu_ctx, nbits):
    """Out of range m, r and c, alone among good ones: zeros and the same
    error on both engines."""
    from paper_2601_14980_amd import pc2
    sk, opk, _ = _key(gpu_ctx, nbits)
    n, n2, L = opk.n, opk.n2, sk.L
    full = (1 << (32 * L)) - 1
    ms, rs = _ms_rs(n, 40, 3)
    ms[5], rs[6], ms[33], rs[39] = full, 0, n, n
    cs = [n2, 0, (1 << (64 * L)) - 1, 1] + [random.Random(4).randrange(n2) for _ in range(36)]

    def both(f):
        a = f()
        with _valu(gpu_ctx):
            b = f()
        assert a == b
        return a

    def enc_sk():
        c = torch.full((40, 2 * L), -1, dtype=torch.int32, device="cuda")
        pc2.pc2_encrypt_sk(sk, dev(to_limbs(ms, L)), dev(to_limbs(rs, L)), c)
        return host_ints(c), gpu_ctx.sync()

    out, st = both(enc_sk)
    assert st == pc2.PC2_E_RANGE and [out[i] for i in (5, 6, 33, 39)] == [0] * 4
    big = 40 * 200  # an encryption on the engine
    both(lambda: gpu_encrypt(gpu_ctx, sk.public, ms * (big // 40), rs * (big // 40)))
    both(lambda: gpu_decrypt(gpu_ctx, sk, cs))
    out, st = both(lambda: gpu_scalar_mul(gpu_ctx, sk.public, cs, list(range(40))))
    assert st == pc2.PC2_E_RANGE and out[0] == out[2] == 0


@pytest.mark.parametrize("nbits,count", [
    (400, 33), (512, 65), (512, 20001), (1024, 1), (1024, 33), (1120, 32), (1536, 65),
    (2048, 31), (2048, 97), (2048, 16400),
    (3072, 33), (4096, 32)])
def test_scalar_mul_counts(gpu_ctx, nbits, count):
    sk, opk, _ = _key(gpu_ctx, nbits)
    n2 = opk.n2
    rng = random.Random(count)
    cs = ([n2 - 1, 0, 1, opk.n] + [rng.randrange(n2) for _ in range(count)])[:count]
    ks = ([(1 << 64) - 1, 3, 5, 7, 0, 1, 1 << 60, 15, 1 << 63] +
          [rng.getrandbits(64) for _ in range(count)])[:count]
    got, st = gpu_scalar_mul(gpu_ctx, sk.public, cs, ks)
    assert st == 0
    idx = range(count) if count <= 100 else [0, 1, 4, 8, count // 2, count - 1]
    assert [got[i] for i in idx] == [pow(cs[i], ks[i], n2) for i in idx]
    with _valu(gpu_ctx):
        assert gpu_scalar_mul(gpu_ctx, sk.public, cs, ks) == (got, 0)


# rows: one group, both numbers of column blocks, several row batches (the last
# two are more rows than the plan's staging holds at once)
@pytest.mark.parametrize("nbits,rows,cols,ebits,window,hint,with_alpha", [
    (512, 33, 5, 50, 0, 33, True), (512, 700, 40, 50, 0, 700, True),
    (1024, 1, 1, 1, 0, 0, True), (1024, 33, 3, 64, 0, 33, False), (1120, 32, 5, 17, 0, 1, True),
    (1536, 65, 4, 50, 4, 65, True), (2048, 31, 33, 7, 0, 31, True),
    (2048, 700, 40, 50, 0, 700, True), (2048, 700, 40, 50, 0, 0, False),
    (3072, 40, 6, 33, 12, 40, True), (4096, 33, 3, 50, 0, 33, True),
    (1024, 17000, 2, 9, 0, 64, True), (1024, 17000, 2, 9, 0, 17000, False)])
def test_matvec_shapes(gpu_ctx, nbits, rows, cols, ebits, window, hint, with_alpha):
    from paper_2601_14980_amd import pc2
    sk, opk, _ = _key(gpu_ctx, nbits)
    n2, L2 = opk.n2, 2 * sk.L
    rng = random.Random(rows + cols)
    cs = ([0, n2 - 1] + [rng.randrange(n2) for _ in range(cols)])[-cols:]
    alpha = [rng.randrange(n2) for _ in range(rows)]
    B = np.random.default_rng(rows).integers(0, 1 << ebits, size=(rows, cols), dtype=np.uint64)
    B[0] = 0
    B[-1] = (1 << ebits) - 1
    if rows > 100:
        B[32:96] = 0                     # groups with nothing to do
    bad_row, bad_col = (5, 1) if rows > 30 and cols > 1 else (None, None)
    if bad_row is not None:
        if ebits < 64:
            B[bad_row, 0] = np.uint64(1 << ebits)
        if with_alpha:
            alpha[6] = n2
        cs[bad_col] = n2 + 1
        B[7:12, bad_col] = 0             # rows that do not use the bad column
    Bd = torch.from_numpy(B.view(np.int64)).cuda()
    cd, ad = dev(to_limbs(cs, L2)), dev(to_limbs(alpha, L2)) if with_alpha else None

    def go():
        mv = pc2.MatVec(sk.public, cols, ebits, window, hint)
        mv.load(cd)
        out = torch.full((rows, L2), -1, dtype=torch.int32, device="cuda")
        mv.apply(Bd, out, ad)
        res = (out.cpu(), gpu_ctx.sync(), mv.window, mv.table_bytes)
        if ad is not None:               # alpha in place
            io = ad.clone()
            mv.apply(Bd, io, io)
            assert torch.equal(io.cpu(), res[0]) and gpu_ctx.sync() == res[1]
        mv.close()
        return res

    got = go()
    with _valu(gpu_ctx):
        want = go()
    assert torch.equal(got[0], want[0]) and got[1:] == want[1:]
    if bad_row is None:
        few = [0, rows // 2, rows - 1]
        ref = O.hom_matvec(opk, [[int(v) for v in B[i]] for i in few], cs,
                           [alpha[i] for i in few] if with_alpha else None)
        assert [host_ints(got[0][i:i + 1].cuda())[0] for i in few] == ref


def test_matvec_two_streams(gpu_ctx):
    """One plan's rows on two streams: the second call's staging waits for the
    first one's."""
    from paper_2601_14980_amd import pc2
    sk, opk, _ = _key(gpu_ctx, 1024)
    rng = random.Random(2)
    rows, cols = 300, 40
    c = dev(to_limbs([rng.randrange(opk.n2) for _ in range(cols)], 2 * sk.L))
    Bs = [torch.from_numpy(np.random.default_rng(i).integers(0, 1 << 50, size=(rows, cols),
                                                             dtype=np.uint64).view(np.int64)).cuda()
          for i in range(2)]
    mv = pc2.MatVec(sk.public, cols, 50, 0, rows)
    mv.load(c)
    want = []
    for B in Bs:
        out = torch.zeros((rows, 2 * sk.L), dtype=torch.int32, device="cuda")
        mv.apply(B, out)
        want.append(out)
    assert gpu_ctx.sync() == 0
    outs = [torch.zeros_like(w) for w in want]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(3):
        for B, out, s in zip(Bs, outs, streams):
            with torch.cuda.stream(s):
                mv.apply(B, out)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(outs, want))
    mv.close()


@pytest.mark.parametrize("op", ["encrypt", "decrypt"])
def test_batch_of_several_jobs(gpu_ctx, op):
    """Jobs of one key share launches: lengths at the edges of a block, two
    keys, and a job too small for the engine's own choice."""
    from paper_2601_14980_amd import pc2
    keys = [_key(gpu_ctx, 1024), _key(gpu_ctx, 2048, seed=32)]
    jobs, want = [], []
    for i, count in enumerate((1, 31, 32, 33, 4000, 64, 65, 4100)):
        sk, opk, _ = keys[i & 1]
        ms, rs = _ms_rs(opk.n, max(count, 4), i)
        ms, rs = ms[:count], rs[:count]
        with _valu(gpu_ctx):
            cs, st = gpu_encrypt(gpu_ctx, sk.public, ms, rs)
        assert st == 0
        if op == "encrypt":
            jobs.append(dict(op=pc2.PC2_OP_ENCRYPT, pk=sk.public, m=dev(to_limbs(ms, sk.L)),
                             r=dev(to_limbs(rs, sk.L)),
                             out=torch.zeros((count, 2 * sk.L), dtype=torch.int32, device="cuda")))
            want.append(cs)
        else:
            jobs.append(dict(op=pc2.PC2_OP_DECRYPT, sk=sk, c=dev(to_limbs(cs, 2 * sk.L)),
                             out=torch.zeros((count, sk.L), dtype=torch.int32, device="cuda")))
            want.append(ms)
    b = pc2.Batch(gpu_ctx, jobs)
    for _ in range(2):
        b.run()
        assert gpu_ctx.sync() == 0
        assert [host_ints(j["out"]) for j in jobs] == want
        for j in jobs:
            j["out"].zero_()
    b.close()


def _prime(bits, seed):
    rng = random.Random(seed)
    small = [p for p in range(3, 2000, 2) if all(p % d for d in range(3, int(p ** 0.5) + 1, 2))]
    while True:
        x = rng.getrandbits(bits) | 1 | (3 << (bits - 2))
        if all(x % p for p in small) and pow(2, x - 1, x) == 1 and pow(3, x - 1, x) == 1:
            return x


# primes of unequal lengths: limbs of p past a wavefront's (33 and 65 words),
# and a q^2 of fewer limbs than p^2
@pytest.mark.parametrize("pbits,qbits", [(1034, 1014), (2068, 2028)])
def test_unequal_primes(gpu_ctx, pbits, qbits):
    from paper_2601_14980_amd import pc2
    p, q = _prime(pbits, 1), _prime(qbits, 2)
    n = p * q
    opk, osk = O.derive_keys(p, q)
    sk = pc2.SecretKey(gpu_ctx, n.bit_length(), p, q)
    ms, rs = _ms_rs(n, 9, 5)
    cs, st = gpu_encrypt(gpu_ctx, sk.public, ms, rs)
    assert st == 0 and cs == [O.encrypt(opk, m, r) for m, r in zip(ms, rs)]
    assert gpu_decrypt(gpu_ctx, sk, cs) == (ms, 0)
    # not coprime to p: refused alike
    bad = [cs[0], p * 3, q * q, cs[1]]
    got = gpu_decrypt(gpu_ctx, sk, bad)
    with _valu(gpu_ctx):
        assert got == gpu_decrypt(gpu_ctx, sk, bad)
    assert got[0][0] == ms[0] and got[0][1] == got[0][2] == 0


# the last count on wavefronts of its own and the first on the engine from
# 3072-bit keys on, where two column blocks a workgroup take half of the units
@pytest.mark.parametrize("nbits,count", [
    (3072, 7168), (3072, 7169), (3072, 8193), (4096, 7168), (4096, 7169), (4096, 8193)])
def test_encrypt_engine_edges(gpu_ctx, nbits, count):
    sk, opk, _ = _key(gpu_ctx, nbits)
    ms, rs = _ms_rs(opk.n, 60, count)
    reps = -(-count // 60)
    ms, rs = (ms * reps)[:count], (rs * reps)[:count]
    got, st = gpu_encrypt(gpu_ctx, sk.public, ms, rs)
    assert st == 0 and got[:4] == [O.encrypt(opk, m, r) for m, r in zip(ms[:4], rs[:4])]
    with _valu(gpu_ctx):
        want, st = gpu_encrypt(gpu_ctx, sk.public, ms[:60], rs[:60])
    assert st == 0 and got == (want * reps)[:count]
