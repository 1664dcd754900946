"""Batches so long that one launch would count 2^32 threads or more (a launch
drops those beyond without an error): every instance computed, exactly."""
import pytest
import torch

from paper_2203_09353_amd import bgemm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    hd = bgemm.Handle()
    yield hd
    hd.close()


@pytest.mark.parametrize("mode,slices,n,batch", [
    ("fp64", 0, 17, 33_600_000),      # 128 threads an instance
    ("fp64", 0, 1, 67_200_000),       # 64
    ("fp32", 0, 1, 16_800_000),       # 256
    ("bf16", 0, 1, 16_800_000),
    ("emu", 2, 1, 16_800_000),
    ("f32emu", 2, 1, 16_800_000),
    ("i8emu", 3, 1, 8_400_000),       # two exponent blocks of 256
    ("i8emu", 8, 1, 8_400_000),       # and 512 a tile
    ("complex", 0, 17, 16_800_000),   # 256
    ("complex", 0, 1, 67_200_000),    # 64
])
def test_every_instance_of_a_long_batch(h, mode, slices, n, batch):
    """1 x n products of one small integer each, another from instance to
    instance (exact in every mode)."""
    dt = torch.complex128 if mode == "complex" else torch.float64
    es = 16 if mode == "complex" else 8
    A = torch.arange(1, 101, device="cuda").to(dt)
    B = torch.arange(1, n + 1, device="cuda").to(dt)
    C = torch.zeros((batch, n), dtype=dt, device="cuda")
    i = torch.arange(batch, device="cuda")
    pA = A.data_ptr() + i % 100 * es
    pB = torch.full((batch,), B.data_ptr(), dtype=torch.int64, device="cuda")
    pC = C.data_ptr() + i * (n * es)
    args = (pA.data_ptr(), 1, pB.data_ptr(), 1, 0.0, pC.data_ptr(), 1, batch)
    if mode == "complex":
        st = h.zgemm_batched_raw("N", "N", 1, n, 1, 1.0, *args)
    else:
        st = h.gemm_batched_mode_raw(bgemm.MODES[mode], slices, "N", "N", 1, n, 1, 1.0, *args)
    torch.cuda.synchronize()
    assert st == 0
    wrong = 0
    for lo in range(0, batch, 1 << 22):
        j = i[lo:lo + (1 << 22)] % 100 + 1
        wrong += int((C[lo:lo + (1 << 22)] != j.to(dt)[:, None] * B).sum())
    assert wrong == 0
