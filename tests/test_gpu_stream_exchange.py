"""The persistent streaming engine's exchanges carry sums scaled by a power of two: 2^k times the input gives the same signs and 2^k
times the coefficients, bit for bit.  Shapes: every number of chunks a thread and every number of lanes across a slice, rows kept
in registers, in LDS and streamed, blocks that end in the middle of each."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

OPTS = {"resident": 0, "sparse": 0}
LAUNCH = {"resident": 0, "sparse": 0, "persistent_stream": 0}


@pytest.fixture(scope="module")
def scd():
    from paper_2410_01799_amd import scd as mod

    mod.lib()
    return mod


def gauss(shape, seed, dtype):
    return torch.from_numpy(np.random.Generator(np.random.PCG64(seed)).standard_normal(shape)).to(dtype).cuda()


def run(scd, A, w, share, opts, launches=1):
    with scd.ScdContext(A, w, 5, options=opts) as ctx:
        ctx.set_workgroups(share)
        assert ctx.engine()["engine"] == (3 if opts is OPTS else 0)
        for i in range(launches):
            ctx.run(w // launches)
        return ctx.results(), ctx.remainder()


# bytes of a row (1 to 8 chunks a thread), rows a workgroup (1 to 40), workgroups (256 down to 16: slices of 8 to 256 columns)
CASES = [((256, 256), torch.float64, 0), ((1300, 1000), torch.float64, 0), ((2560, 2048), torch.float32, 64), ((700, 4096), torch.float32, 0),
         ((900, 6000), torch.float32, 32), ((700, 8192), torch.float32, 0), ((640, 10000), torch.float32, 0), ((300, 12000), torch.float32, 64),
         ((600, 14000), torch.float32, 0), ((640, 16384), torch.float32, 64), ((400, 3968), torch.float32, 16), ((333, 3300), torch.float64, 32),
         ((3000, 300, 3), torch.float32, 0), ((500, 700, 4), torch.float64, 0), ((700, 3001, 4), torch.float32, 0)]


@pytest.mark.parametrize("dims,dtype,share", CASES)
def test_powers_of_two_and_the_launch_stream(scd, dims, dtype, share):
    w = 4
    A = gauss(dims, sum(dims), dtype)
    base, R = run(scd, A, w, share, OPTS)
    for k, launches in ((40, 2), (-30, 1)):
        res, Rk = run(scd, A * 2.0 ** k, w, share, OPTS, launches)
        for mode in range(len(dims)):
            assert torch.equal(res["signs"][mode], base["signs"][mode])
        assert torch.equal(res["iters"], base["iters"])
        assert torch.equal(res["c"].double(), base["c"].double() * 2.0 ** k)
        assert torch.equal(Rk, R * 2.0 ** k)
    if dtype is torch.float64:  # (f32 near ties may fall differently between engines)
        ref, Rr = run(scd, A, w, 0, LAUNCH)
        for mode in range(len(dims)):
            assert torch.equal(ref["signs"][mode], base["signs"][mode])
        np.testing.assert_allclose(base["c"].cpu().numpy(), ref["c"].cpu().numpy(), rtol=1e-12)
        assert float((R - Rr).abs().max()) < 1e-12


@pytest.mark.parametrize("dims", [(2000, 700, 3), (300, 5000, 3), (1200, 1500, 4), (90, 80, 2), (700, 3000, 1)])
def test_real_last_mode(scd, dims):
    A = gauss(dims, 3, torch.float32) + 2.0
    base = scd.scd_decompose_scalars(A, 5, 7)
    res = scd.scd_decompose_scalars(A * 2.0 ** 20, 5, 7)
    for mode in range(2):
        assert torch.equal(res["signs"][mode], base["signs"][mode])
    assert torch.equal(res["c"].double(), base["c"].double() * 2.0 ** 20)
    # the identity of Section 5's projection: ||R_{j+1}||^2 = ||R_j||^2 - mn sum_c c_j[c]^2
    t, c = base["trace"].cpu().numpy(), base["c"].double().cpu().numpy()
    np.testing.assert_allclose(t[1:] ** 2, t[:-1] ** 2 - dims[0] * dims[1] * (c ** 2).sum(1), rtol=1e-6)
