"""The words that the register-resident engine exchanges carry sums scaled by a power of two: a decomposition of 2^k A is that of
A with coefficients 2^k times as large, bit for bit, at every size of the entries; a context whose remainder changes between sizes
changes the type of its words with it."""
import numpy as np
import pytest
import torch

from helpers import CURVE_RTOL, dense

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scd():
    from paper_2410_01799_amd import scd as mod

    mod.lib()
    return mod


def gauss(shape, seed, dtype):
    return torch.from_numpy(np.random.Generator(np.random.PCG64(seed)).standard_normal(shape)).to(dtype).cuda()


def same_up_to(a, b, k):
    assert torch.equal(a["signs"][0], b["signs"][0]) and torch.equal(a["signs"][1], b["signs"][1])
    assert torch.equal(a["iters"], b["iters"])
    assert torch.equal(a["c"].double() * 2.0 ** k, b["c"].double())


# every number of lanes per 16-byte piece (4, 8, 16 partners; 64, 128 and 256 sums a slot), full and overhanging grids
SHAPES = [(300, 260), (512, 512), (257, 400), (1024, 1024), (1030, 520), (2048, 1000), (64, 4096), (4096, 512), (1501, 999), (301, 407)]


@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("dtype,powers", [(torch.float32, (-60, 40, 105)), (torch.float64, (-400, 400))], ids=["f32", "f64"])
def test_powers_of_two(scd, m, n, dtype, powers):
    w, seed = 6, 5
    A = gauss((m, n), m + n, dtype)
    base = scd.scd_decompose(A, w, seed)
    for k in powers:
        same_up_to(base, scd.scd_decompose(A * 2.0 ** k, w, seed), k)


@pytest.mark.parametrize("m,n", [(300, 260), (1024, 1024), (64, 4096)])
def test_sums_near_the_largest_f32(scd, m, n):
    """Entries of 1e36 and more: f64 words; norms as at any other size (up to near ties)."""
    w, seed = 6, 5
    A = gauss((m, n), 3, torch.float32)
    base = scd.scd_decompose(A, w, seed)
    big = scd.scd_decompose(A * 2.0 ** 121, w, seed)
    assert torch.isfinite(big["c"]).all()
    np.testing.assert_allclose(np.ldexp(big["trace"].cpu().numpy(), -121), base["trace"].cpu().numpy(), rtol=CURVE_RTOL)


@pytest.mark.parametrize("m,n", [(300, 260), (1024, 1024)])
def test_a_remainder_of_another_size(scd, m, n):
    """One context, remainders whose sums travel as f32, as f64 and as f32 again, an odd number of exchanges between."""
    w, seed = 3, 9
    A = gauss((m, n), 11, torch.float32)
    B = A * 2.0 ** 121
    with scd.ScdContext(A, 3 * w, seed) as ctx:
        for turn, X in enumerate((A, B, A)):
            if turn:
                ctx.set_remainder(X)
            assert ctx.engine()["engine"] == 1
            for _ in range(w):
                ctx.run(1)
        got = ctx.results()
    for turn, X in enumerate((A, B, A)):
        # the same terms in one launch of a context of its own, from the same keyed starts
        with scd.ScdContext(A, (turn + 1) * w, seed) as ctx:
            ctx.run(turn * w)
            ctx.set_remainder(X)
            ctx.run(w)
            want = ctx.results()
        for key in ("c", "iters"):
            assert torch.equal(got[key][turn * w:(turn + 1) * w], want[key][turn * w:])
        for mode in range(2):
            assert torch.equal(got["signs"][mode][turn * w:(turn + 1) * w], want["signs"][mode][turn * w:])


@pytest.mark.parametrize("m,n", [(300, 260), (1024, 1024), (1501, 999)])
def test_least_squares_powers_of_two(scd, m, n):
    w, seed = 5, 4
    A = gauss((m, n), 7, torch.float64)
    base = scd.scd_lsq_decompose(A, w, seed)
    for k in (-300, 300):
        same_up_to(base, scd.scd_lsq_decompose(A * 2.0 ** k, w, seed), k)


@pytest.mark.parametrize("options,engine", [({}, 1), ({"resident": 0, "sparse": 0}, 3)], ids=["resident", "stream"])
@pytest.mark.parametrize("dtype,low", [(torch.float32, -105), (torch.float64, -480)], ids=["f32", "f64"])
@pytest.mark.parametrize("m,n", [(512, 512), (300, 260)])
def test_small_sums_beside_large_ones(scd, m, n, dtype, low, options, engine):
    """Columns of size 2^low beside columns of size 1: within the range that the words keep, so the signs of their sums count.
    Odd whole numbers, so that the columns' sums are exact and those of the rows, over an odd number of large columns, not zero."""
    g = np.random.Generator(np.random.PCG64(1))
    x = 2.0 * g.integers(-4, 4, (m, n)) + 1.0
    size = np.where(np.arange(n) % 7 < 3, 2.0 ** low, 1.0)
    if (size == 1.0).sum() % 2 == 0:
        size[n - 1] = 2.0 ** low if size[n - 1] == 1.0 else 1.0
    A = torch.from_numpy(x * size).to(dtype).cuda()
    out = []
    for opts in (options, {"resident": 0, "sparse": 0, "persistent_stream": 0}):
        with scd.ScdContext(A, 1, 5, options=opts) as ctx:
            assert ctx.engine()["engine"] == (engine if opts is options else 0)
            ctx.set_max_iters(1)
            ctx.run(1)
            out.append(ctx.results())
    assert torch.equal(out[0]["signs"][0], out[1]["signs"][0]) and torch.equal(out[0]["signs"][1], out[1]["signs"][1])
    S = out[0]["signs"][0][0].cpu().numpy().view(np.uint64)
    T = out[0]["signs"][1][0].cpu().numpy().view(np.uint64)
    v = dense(S, m) @ x
    assert np.array_equal(dense(T, n), np.where(v < 0, -1.0, 1.0))
