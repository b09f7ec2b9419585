"""Late alternations of the sparse engine run on one wave per workgroup.  Immediate updates (no list of pending terms) never take
them, so both must find the same terms: every number of members and words that the late exchanges are built for, slices of
one and two entries a lane, empty slices, half steps that one wave adds up alone and that it hands to the others."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scd():
    from paper_2410_01799_amd import scd as mod

    mod.lib()
    return mod


def gauss(shape, seed):
    return torch.from_numpy(np.random.Generator(np.random.PCG64(seed)).standard_normal(shape)).cuda()


def run(scd, A, w, share, launches, **options):
    with scd.ScdContext(A, w, 5, options=dict(resident=0, sparse_min_mib=0, persistent_stream=0, **options)) as ctx:
        for g, n in launches:
            ctx.set_workgroups(share if g is None else g)
            assert ctx.engine()["engine"] == 2
            ctx.run(n)
        return ctx.results(), ctx.sparse_flips()


def same(a, b):
    (ra, fa), (rb, fb) = a, b
    assert torch.equal(ra["signs"][0], rb["signs"][0]) and torch.equal(ra["signs"][1], rb["signs"][1])
    assert torch.equal(ra["iters"], rb["iters"])
    assert fa == fb
    np.testing.assert_allclose(ra["c"].cpu().numpy(), rb["c"].cpu().numpy(), rtol=1e-12)
    # (between flushes the norm follows from the cut value)
    np.testing.assert_allclose(ra["trace"].cpu().numpy(), rb["trace"].cpu().numpy(), rtol=1e-9)


# m, n, workgroups: slices of 8, 16, 24 .. 128 rows or columns; 4 to 512 words of a side; slices that are cut off and that own nothing
CASES = [(200, 200, 16), (512, 512, 32), (500, 1022, 16), (1024, 2048, 16), (2000, 600, 100), (2048, 2048, 0), (4096, 1030, 64),
         (4096, 4096, 0), (1024, 8000, 256), (264, 10000, 0), (8192, 264, 64)]


@pytest.mark.parametrize("m,n,share", CASES)
def test_late_alternations_find_the_same_terms(scd, m, n, share):
    A, w = gauss((m, n), m * 7 + n), 19 if m * n < 1 << 22 else 11
    same(run(scd, A, w, share, [(None, w)]), run(scd, A, w, share, [(None, w)], sparse_delay_width=0))


def test_launches_and_shares_of_one_context(scd):
    """Members that take no part for a while leave old words in their slots."""
    A = gauss((1000, 1500), 3)
    launches = [(256, 3), (32, 4), (256, 2), (64, 1), (256, 5), (32, 4)]
    w = sum(n for _, n in launches)
    same(run(scd, A, w, 0, launches), run(scd, A, w, 0, launches, sparse_delay_width=0))


def test_late_alternations_stop_on_the_iteration_cap(scd):
    A = gauss((600, 800), 8)
    out = []
    for width in (8, 0):
        with scd.ScdContext(A, 4, 5, options=dict(resident=0, sparse_min_mib=0, sparse_delay_width=width)) as ctx:
            ctx.set_max_iters(9)
            assert ctx.run(4) == scd.WMAXITER
            out.append((ctx.results(), ctx.sparse_flips()))
    assert int(out[0][0]["iters"].max()) == 9
    same(*out)
