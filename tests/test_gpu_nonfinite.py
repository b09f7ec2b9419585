"""Infinities and NaNs stay visible in the results whatever engine serves the context: a remainder that holds some, and sums
that pass the largest f32."""
import numpy as np
import pytest
import torch

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
