"""Uniform batches on whole interior tiles: results against the oracle and the
128 x 128 tile's bits, and guard regions around every instance of C that must
come back bit for bit."""
import contextlib
import itertools

import numpy as np
import pytest
import torch

import oracle
from paper_2203_09353_amd import bgemm, inputs

pytestmark = pytest.mark.gpu

GUARD = 16          # doubles, a whole 128-byte line; and as many columns behind C
SENTINEL = 0x7FF8_0BAD_5EED_0123
# every uniform tile shape: its number, rows and columns
SHAPES = [(0, 32, 32), (1, 64, 64), (2, 128, 128), (3, 128, 64), (4, 64, 32), (5, 32, 64),
          (6, 32, 16), (7, 128, 48)]


@pytest.fixture(scope="module")
def h():
    hd = bgemm.Handle()
    yield hd
    hd.close()


def guarded(batch, m, n, ldc, C):
    """A flat buffer of sentinels with the instances of C laid into it, GUARD
    columns and GUARD doubles apart; the buffer, the instances' starts (in
    doubles) and the (column, row) offsets of an instance."""
    step = (GUARD + (n + GUARD) * ldc + 15) // 16 * 16
    buf = torch.full((step * batch + GUARD,), SENTINEL, dtype=torch.int64)
    at = torch.arange(n)[:, None] * ldc + torch.arange(m)[None, :]
    start = GUARD + step * torch.arange(batch)
    buf[start[:, None, None] + at] = C.view(torch.int64)
    return buf.cuda().view(torch.float64), start, at


def run_guarded(call, batch, m, n, ldc, C):
    buf, start, at = guarded(batch, m, n, ldc, C)
    call(buf.data_ptr() + 8 * start.cuda())
    torch.cuda.synchronize()
    bits = buf.view(torch.int64).cpu()
    where = start[:, None, None] + at
    got = bits[where].view(torch.float64)
    bits[where] = SENTINEL
    assert bool((bits == SENTINEL).all()), "written outside C at %s" % (
        torch.nonzero(bits != SENTINEL)[:4].flatten().tolist())
    return got


@contextlib.contextmanager
def forced(h, shape):
    """The handle's batches on one tile shape (-1: as picked)."""
    assert bgemm.lib().bgi_force_tile(h._h, shape) == 0
    try:
        yield
    finally:
        assert bgemm.lib().bgi_force_tile(h._h, -1) == 0


def check(h, ta, tb, m, n, k, batch, alpha, beta, ldc, shapes):
    """Each shape's results: nothing outside C, the same bits as 128 x 128 tiles,
    and those within the binary64 bound of the oracle."""
    ra, ca = (m, k) if ta == "N" else (k, m)
    rb, cb = (k, n) if tb == "N" else (n, k)
    A, B = inputs.uniform_batch(51, 0, batch, ra, ca), inputs.uniform_batch(51, 1, batch, rb, cb)
    C = inputs.uniform_batch(51, 2, batch, m, n)
    C0 = torch.full_like(C, float("nan")) if beta == 0.0 else C
    Ad, Bd = A.cuda(), B.cuda()
    pA, pB = bgemm.pointer_array(Ad), bgemm.pointer_array(Bd)

    def call(pC):
        st = h.dgemm_batched_raw(ta, tb, m, n, k, alpha, pA.data_ptr(), ra, pB.data_ptr(), rb,
                                 beta, pC.data_ptr(), ldc, batch)
        assert st == 0

    with forced(h, 2):
        ref = run_guarded(call, batch, m, n, ldc, C0)
    for shape in shapes:
        with forced(h, shape):
            got = run_guarded(call, batch, m, n, ldc, C0)
        assert torch.equal(got.view(torch.int64), ref.view(torch.int64)), shape
    some = sorted({0, batch // 2, batch - 1})
    exp = C[some].numpy().copy()
    oracle.gemm_batched(ta, tb, m, n, k, alpha, A[some].numpy(), B[some].numpy(), beta, exp)
    err = np.linalg.norm(ref[some].numpy() - exp) / np.linalg.norm(exp)
    assert err <= 1e-13


@pytest.mark.parametrize("ta,tb", list(itertools.product("NT", "NT")))
@pytest.mark.parametrize("m,n,k,batch", [(128, 48, 64, 530), (256, 96, 256, 140), (256, 140, 80, 90),
                                         (336, 336, 336, 30), (500, 144, 100, 64)])
@pytest.mark.parametrize("pad", [0, 1])
def test_tiles_of_48_columns_stay_inside(h, ta, tb, m, n, k, batch, pad):
    check(h, ta, tb, m, n, k, batch, 1.25, 0.0, m + pad, [-1, 7])
    check(h, ta, tb, m, n, k, batch, -0.75, 1.5, m + pad, [-1, 7])


@pytest.mark.parametrize("ta,tb", list(itertools.product("NT", "NT")))
@pytest.mark.parametrize("shape,bm,bn", SHAPES)
@pytest.mark.parametrize("pad", [0, 1])
def test_every_shape_on_whole_and_cut_tiles(h, ta, tb, shape, bm, bn, pad):
    """Two by three whole tiles, whose C is in whole lines without padding; then
    cut ones behind whole ones, at a short and at a ragged k."""
    for alpha, beta in ((1.25, 0.0), (-0.75, 1.5)):
        check(h, ta, tb, 2 * bm, 3 * bn, 32, 3, alpha, beta, 2 * bm + pad, [shape])
        check(h, ta, tb, 2 * bm + 7, 2 * bn + 9, 15, 3, alpha, beta, 2 * bm + 7 + pad, [shape])
        check(h, ta, tb, 2 * bm - 1, 2 * bn - 1, 49, 3, alpha, beta, 2 * bm - 1 + pad, [shape])
