"""The inner pass of the f32 product at the edges of what a workgroup takes: words of a chunk that fill no group of eight, no
quarter or one word more than a chunk; terms that fill no tile of 64, or one to four tiles a workgroup; largest entries that
are denormal, or of the largest exponents."""
import numpy as np
import pytest
import torch

from test_gpu_apply import check, random_factors, scd  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 64, 65, 511, 513, 1025, 2049, 3073, 4033, 4096, 4097, 8191])
@pytest.mark.parametrize("w", [1, 15, 63, 64, 65, 129])
def test_words_and_terms_at_edges(scd, oracle, n, w):  # noqa: F811
    check(scd, oracle, 70, n, w, 5 * n + w, np.float32, False)


@pytest.mark.parametrize("w", [16383, 16385, 32769, 49153, 65537])
def test_several_tiles_a_workgroup(scd, oracle, w):  # noqa: F811
    check(scd, oracle, 65, 130, w, w, np.float32, False)


@pytest.mark.parametrize("power", [-147, -127, -100, 0, 100, 120])
@pytest.mark.parametrize("nvec", [1, 2, 4])
def test_a_power_of_two_changes_no_bit(scd, power, nvec):  # noqa: F811
    m, n, w = 130, 700, 90
    S, T, c = random_factors(m, n, w, 7, np.float32)
    rs = np.random.Generator(np.random.PCG64(8))
    x = rs.integers(-7, 8, (nvec, n)).astype(np.float32)  # (exact at every scale)
    dev = lambda b: torch.from_numpy(b.view(np.int64)).cuda()
    s, t = dev(S), dev(T)

    def product(xs, cs):
        return scd.scd_apply(s, t, torch.from_numpy(cs).cuda(), m, n, torch.from_numpy(xs).cuda()).cpu().numpy()

    half = power // 2
    c1 = (c.astype(np.float64) * 2.0 ** -10).astype(np.float32)
    y = product(x, c1)
    scaled = product((x.astype(np.float64) * 2.0 ** power).astype(np.float32), (c1.astype(np.float64) * 2.0 ** -half).astype(np.float32))
    assert np.array_equal(scaled.astype(np.float64), y.astype(np.float64) * 2.0 ** (power - half))
