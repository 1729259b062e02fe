"""Mat-vec plans and the memory that they are made for: the tables take the bytes
that pc2_matvec_info reports, on either engine, and rows are right for every
number of digits that a window leaves room for."""
from __future__ import annotations

import random

import numpy as np
import pytest
import torch

from tests.gpu_helpers import dev, host_ints
from tests.test_gpu_rns import _key, _valu
from workload.limbs import to_limbs

pytestmark = pytest.mark.gpu


def _entry_bytes(nbits: int) -> int:
    return 64 * {1024: 9, 2048: 17, 4096: 34}[nbits]


@pytest.mark.parametrize("nbits,cols,ebits,window,hint", [
    (1024, 3000, 50, 1, 0), (2048, 3000, 50, 1, 0), (2048, 3000, 50, 2, 0),
    (2048, 1000, 50, 3, 0), (2048, 300, 50, 5, 300), (2048, 300, 64, 8, 0),
    (2048, 2000, 50, 0, 2000), (4096, 500, 20, 4, 0), (4096, 40, 50, 0, 9000)])
def test_plan_takes_the_bytes_it_reports(gpu_ctx, nbits, cols, ebits, window, hint):
    from paper_2601_14980_amd import pc2
    sk, _, _ = _key(gpu_ctx, nbits)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    mv = pc2.MatVec(sk.public, cols, ebits, window, hint)
    took = free - torch.cuda.mem_get_info()[0]
    w = mv.window
    assert window in (0, w)
    words = {1024: 320, 2048: 640, 4096: 1216}[nbits]
    if nbits != 4096:
        assert mv.table_bytes == cols * -(-ebits // w) * ((1 << w) - 1) * words
    assert took <= mv.table_bytes + mv.staging_bytes + (8 << 20)
    # the entries of a block's digits fit
    lo, x = divmod(-(-ebits // mv.blocks), mv.digits)
    entries = 1 + x * ((2 << lo) - 1) + (mv.digits - x) * ((1 << lo) - 1)
    assert mv.residues and cols * entries * _entry_bytes(nbits) <= mv.table_bytes
    mv.close()
    with _valu(gpu_ctx):
        mv = pc2.MatVec(sk.public, cols, ebits, window, hint)
        assert (mv.window, mv.residues, mv.blocks) == (w, False, 1)
        assert mv.digits == -(-ebits // w)
        mv.close()


@pytest.mark.parametrize("nbits", [512, 1024, 2048, 4096])
@pytest.mark.parametrize("ebits", [1, 7, 33, 50, 64])
@pytest.mark.parametrize("window", [1, 2, 3, 4, 6, 9, 12])
def test_rows_at_every_number_of_digits(gpu_ctx, nbits, ebits, window):
    from paper_2601_14980_amd import pc2
    sk, opk, _ = _key(gpu_ctx, nbits)
    n2, L2 = opk.n2, 2 * sk.L
    rng = random.Random(nbits + ebits + window)
    rows, cols = 37, 3
    cs = [n2 - 1, rng.randrange(n2), rng.randrange(n2)]
    top = (1 << ebits) - 1
    B = np.random.default_rng(window).integers(0, top, size=(rows, cols), dtype=np.uint64,
                                               endpoint=True)
    B[0], B[1] = top, 0
    B[2] = [1, 1 << (ebits - 1), 0]
    bad = 3
    if ebits < 64:
        B[bad] = [np.uint64(1) << np.uint64(ebits), top, (1 << 64) - 1]
    Bd, cd = torch.from_numpy(B.view(np.int64)).cuda(), dev(to_limbs(cs, L2))

    def go():
        mv = pc2.MatVec(sk.public, cols, ebits, window)
        mv.load(cd)
        out = torch.full((rows, L2), -1, dtype=torch.int32, device="cuda")
        mv.apply(Bd, out)
        res = host_ints(out), gpu_ctx.sync()
        mv.close()
        return res

    got = go()
    with _valu(gpu_ctx):
        assert got == go()
    for i in (0, 1, 2, 4, rows - 1):
        want = 1
        for c, b in zip(cs, B[i]):
            want = want * pow(c, int(b), n2) % n2
        assert got[0][i] == want
    if ebits < 64:
        assert got == (got[0], pc2.PC2_E_RANGE) and got[0][bad] == 0


# plans made for few rows (constants in blocks): one row and several, column chunks
# and one column, no alpha and one (also in place), more rows than they were made for,
# rows and columns of zeros, bad ones
@pytest.mark.parametrize("nbits,rows,cols,ebits,window,hint,with_alpha", [
    (512, 1, 200, 50, 0, 1, True), (1024, 1, 70, 50, 0, 1, False), (1024, 5, 33, 64, 0, 5, True),
    (1120, 40, 9, 50, 2, 1, True), (1536, 3, 300, 50, 0, 3, False), (2048, 1, 1, 50, 0, 1, True),
    (2048, 6, 435, 50, 0, 6, True), (2048, 33, 64, 64, 1, 1, False), (2048, 700, 40, 50, 0, 2, True),
    (2048, 70, 5, 4, 0, 1, True), (3072, 4, 40, 33, 0, 4, True), (4096, 2, 70, 50, 0, 2, True),
    (1024, 17000, 2, 9, 0, 1, True)])
def test_rows_with_constants_in_blocks(gpu_ctx, nbits, rows, cols, ebits, window, hint, with_alpha):
    from paper_2601_14980_amd import pc2
    sk, opk, _ = _key(gpu_ctx, nbits)
    n2, L2 = opk.n2, 2 * sk.L
    rng = random.Random(rows + cols)
    cs = ([0, n2 - 1] + [rng.randrange(n2) for _ in range(cols)])[-cols:]
    alpha = [rng.randrange(n2) for _ in range(rows)]
    B = np.random.default_rng(rows).integers(0, 1 << ebits, size=(rows, cols), dtype=np.uint64) \
        if ebits < 64 else np.random.default_rng(rows).integers(
            0, (1 << 64) - 1, size=(rows, cols), dtype=np.uint64, endpoint=True)
    B[-1] = (1 << ebits) - 1
    if rows > 2:
        B[0], B[1] = 0, 0
        B[1, 0] = 1
    if rows > 100:
        B[32:64] = 0                     # a group with nothing to do
    bad = rows > 32
    if bad and ebits < 64:
        B[5, 0], alpha[6], cs[-1] = np.uint64(1 << ebits), n2, n2 + 1
        B[7:12, -1] = 0                  # rows that do not use the bad column
    Bd = torch.from_numpy(B.view(np.int64)).cuda()
    cd, ad = dev(to_limbs(cs, L2)), dev(to_limbs(alpha, L2)) if with_alpha else None

    def go():
        mv = pc2.MatVec(sk.public, cols, ebits, window, hint)
        mv.load(cd)
        out = torch.full((rows, L2), -1, dtype=torch.int32, device="cuda")
        mv.apply(Bd, out, ad)
        res = out.cpu(), gpu_ctx.sync()
        if ad is not None:
            io = ad.clone()
            mv.apply(Bd, io, io)
            assert torch.equal(io.cpu(), res[0]) and gpu_ctx.sync() == res[1]
        blocks = mv.blocks
        mv.close()
        return res, blocks

    got, blocks = go()
    assert blocks > 1
    with _valu(gpu_ctx):
        want, _ = go()
    assert torch.equal(got[0], want[0]) and got[1] == want[1]
    if not bad:
        for i in {0, rows - 1}:
            v = alpha[i] if with_alpha else 1
            for c, b in zip(cs, B[i]):
                v = v * pow(c, int(b), n2) % n2
            assert host_ints(got[0][i:i + 1].cuda()) == [v]
