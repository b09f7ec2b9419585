"""The column half step at the edges of its tiles: rows below, at and past a thread's batch (4 or 16) and a workgroup's
group of rows, rows enough for several batches a thread, columns below, at and past a tile of 1 to 64 lanes (16 bytes a
lane where rows are aligned to it, else one entry), and more words of signs than one launch joins."""
import numpy as np
import pytest
import torch

from helpers import to_dev_bits, to_np_bits

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 4), (1, 257), (2, 5), (3, 64), (4, 63), (15, 128), (16, 130), (17, 132), (31, 256), (32, 257), (33, 260),
         (127, 512), (128, 1000), (129, 1001), (2049, 7), (2048, 8), (4099, 2052), (4096, 4099), (5000, 100),
         (200001, 3), (600001, 4), (65, 32768), (66, 32769), (40000, 515)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n", SIZES)
def test_column_step_at_edges(oracle, m, n, dtype):
    from paper_2410_01799_amd import scd

    print(f"column step {m}x{n} {dtype.__name__}", flush=True)
    A = np.random.Generator(np.random.PCG64(m * 7 + n)).standard_normal((m, n)).astype(dtype)
    R = torch.from_numpy(A).cuda()
    words = oracle.rng_signs(3, 0, 0, m)
    v, t, c = scd.scd_col_signed_sum(R, to_dev_bits(words))
    bits = np.unpackbits(np.asarray(words, dtype="<u8").view(np.uint8), bitorder="little")[:m].astype(bool)
    A64 = A.astype(np.float64)
    ref = A64[~bits].sum(0) - A64[bits].sum(0)
    got = v.cpu().numpy()
    # m f64 additions in any order: (m - 1) 2^-53 of the sum of the magnitudes, for either side
    bound = 2.0 * m * 2.0 ** -53 * np.abs(A64).sum(0)
    assert (np.abs(got - ref) <= bound).all()
    back = np.unpackbits(to_np_bits(t).view(np.uint8), bitorder="little")
    assert np.array_equal(back[:n].astype(bool), got < 0) and not back[n:].any()
    assert float(c) == pytest.approx(np.abs(got).sum(), rel=n * 2.0 ** -52)
    again = scd.scd_col_signed_sum(R, to_dev_bits(words))
    assert torch.equal(v, again[0]) and torch.equal(t, again[1]) and torch.equal(c, again[2])


def test_infinities_past_the_last_row_of_a_batch_do_not_spread():
    from paper_2410_01799_amd import scd

    # a thread's missing rows are read from its first one: an infinity there counts once
    R = torch.ones((17, 8), device="cuda")
    R[16, 3] = float("inf")
    v, t, c = scd.scd_col_signed_sum(R, torch.zeros(1, dtype=torch.int64, device="cuda"))
    want = torch.full((8,), 17.0, dtype=torch.float64, device="cuda")
    want[3] = float("inf")
    assert torch.equal(v, want)
