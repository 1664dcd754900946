"""Uniform batches on whole interior tiles: results against the oracle and the
128 x 128 tile's bits, and guard regions around every instance of C that must
come back bit for bit."""
import itertools

import numpy as np
import pytest
import torch

import oracle
from paper_2203_09353_amd import bgemm, inputs

pytestmark = pytest.mark.gpu

GUARD = 16          # doubles, a whole 128-byte line; and as many columns behind C
SENTINEL = 0x7FF8_0BAD_5EED_0123


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


def check(h, ta, tb, m, n, k, batch, alpha, beta, ldc, shapes, force):
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

    h.set_uniform_class(2)
    try:
        ref = run_guarded(call, batch, m, n, ldc, C0)
    finally:
        h.set_uniform_class(-1)
    for shape in shapes:
        with force(shape):
            got = run_guarded(call, batch, m, n, ldc, C0)
        assert torch.equal(got.view(torch.int64), ref.view(torch.int64)), shape
    some = sorted({0, batch // 2, batch - 1})
    exp = C[some].numpy().copy()
    oracle.gemm_batched(ta, tb, m, n, k, alpha, A[some].numpy(), B[some].numpy(), beta, exp)
    err = np.linalg.norm(ref[some].numpy() - exp) / np.linalg.norm(exp)
    assert err <= 1e-13


class as_picked:
    def __init__(self, shape):
        pass

    def __enter__(self):
        pass

    def __exit__(self, *exc):
        pass


@pytest.mark.parametrize("ta,tb", list(itertools.product("NT", "NT")))
@pytest.mark.parametrize("m,n,k,batch", [(128, 48, 64, 530), (256, 96, 256, 140), (256, 140, 80, 90),
                                         (336, 336, 336, 30), (500, 144, 100, 64)])
@pytest.mark.parametrize("pad", [0, 1])
def test_tiles_of_48_columns_stay_inside(h, ta, tb, m, n, k, batch, pad):
    check(h, ta, tb, m, n, k, batch, 1.25, 0.0, m + pad, [None], as_picked)
    check(h, ta, tb, m, n, k, batch, -0.75, 1.5, m + pad, [None], as_picked)
