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
    if mv.residues:  # its digits' entries fit
        lo, x = divmod(ebits, mv.digits)
        entries = 1 + x * ((2 << lo) - 1) + (mv.digits - x) * ((1 << lo) - 1)
        assert cols * entries * _entry_bytes(nbits) <= mv.table_bytes
    else:
        assert mv.digits == -(-ebits // w)
    assert mv.residues == (window not in (1, 2))
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
