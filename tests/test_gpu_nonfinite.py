"""Infinities and NaNs stay visible in the results whatever engine serves the context: a remainder that holds some, and sums
that pass the largest f32."""
import numpy as np
import pytest
import torch

from helpers import C_RTOL, CURVE_RTOL

pytestmark = pytest.mark.gpu

RESIDENT = {}
SPARSE = {"resident": 0, "sparse_min_mib": 0}
STREAM = {"resident": 0, "sparse": 0}
LAUNCH = {"resident": 0, "sparse": 0, "persistent_stream": 0}


@pytest.fixture(scope="module")
def scd():
    from paper_2410_01799_amd import scd as mod

    mod.lib()
    return mod


def gauss(shape, seed, dtype):
    return torch.from_numpy(np.random.Generator(np.random.PCG64(seed)).standard_normal(shape)).to(dtype).cuda()


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("dims,dtype,options,engine", [
    ((512, 400), torch.float32, RESIDENT, 1), ((600, 400), torch.float64, RESIDENT, 1), ((64, 64), torch.float32, RESIDENT, 1),
    ((512, 512), torch.float64, SPARSE, 2), ((600, 400), torch.float32, STREAM, 3), ((300, 200, 3), torch.float64, STREAM, 3)])
def test_a_remainder_that_is_not_finite(scd, dims, dtype, options, engine, bad):
    """The call that gives it says so, later terms are not finite, and the next remainder is served as if it had not been."""
    A = gauss(dims, sum(dims), dtype)
    B = A.clone()
    B.view(-1)[A.numel() // 2 + 17] = bad
    out = []
    for detour in (True, False):
        with scd.ScdContext(A, 5, 3, options=options) as ctx:
            assert ctx.engine()["engine"] == engine
            ctx.run(2)
            ctx.set_max_iters(6)
            if detour:
                with pytest.raises(scd.ScdError) as e:
                    ctx.set_remainder(B)
                assert e.value.code == scd.ENONFINITE
            ctx.run(1)
            c = ctx.results()["c"]
            assert torch.isfinite(c[:2]).all()
            assert torch.isfinite(c[2]) != detour
            ctx.set_max_iters(4096)
            ctx.set_remainder(A * 0.5)
            assert ctx.engine()["engine"] == engine
            ctx.run(2)
            out.append(ctx.results())
    for key in ("c", "iters"):
        assert torch.equal(out[0][key][3:], out[1][key][3:])
    for mode in range(len(dims)):
        assert torch.equal(out[0]["signs"][mode][3:], out[1]["signs"][mode][3:])


# rows a workgroup: 64, 40, 64
TALL = [(16384, 8, 3), (10000, 12, 4), (16384, 24)]


def tall(dims):
    return gauss(dims, sum(dims), torch.float32) * 0.25 + 1.0


@pytest.mark.parametrize("dims", TALL)
def test_column_sums_past_the_largest_f32(scd, dims):
    """f32 sums of a workgroup's rows that overflow: infinite with one launch per alternation, and so with one for all of them."""
    A = tall(dims) * 2.0 ** 124
    for options in (STREAM, LAUNCH):
        with scd.ScdContext(A, 1, 3, options=options) as ctx:
            ctx.set_max_iters(6)
            ctx.run(1)
            assert not torch.isfinite(ctx.results()["c"]).any()


@pytest.mark.parametrize("dims", TALL)
def test_norms_on_either_side_of_the_streaming_engines_limit(scd, dims):
    A, w = tall(dims), 4
    fro, rows = float(A.double().norm()), -(-dims[0] // 256)
    top = int(np.floor(127 - np.log2(fro * rows ** 0.5)))  # largest power of two at which no sum can overflow
    with scd.ScdContext(A, w, 3, options=STREAM) as ctx:
        assert ctx.engine()["engine"] == 3
        ctx.run(w)
        base = ctx.results()
    for k, engine in ((top, 3), (top + 1, 0)):
        with scd.ScdContext(A * 2.0 ** k, w, 3, options=STREAM) as ctx:
            assert ctx.engine()["engine"] == engine
            ctx.run(w)
            res = ctx.results()
        np.testing.assert_allclose(np.ldexp(res["trace"].cpu().numpy(), -k), base["trace"].cpu().numpy(), rtol=CURVE_RTOL)
        np.testing.assert_allclose(np.ldexp(res["c"].double().cpu().numpy(), -k)[:1], base["c"].double().cpu().numpy()[:1], rtol=C_RTOL)
    if len(dims) == 3:
        base = scd.scd_decompose_scalars(A, w, 3)
        for k in (top, top + 1):
            res = scd.scd_decompose_scalars(A * 2.0 ** k, w, 3)
            np.testing.assert_allclose(np.ldexp(res["trace"].cpu().numpy(), -k), base["trace"].cpu().numpy(), rtol=CURVE_RTOL)
