"""Late alternations of the sparse engine run on one wave per workgroup.  Immediate updates (no list of pending terms) never take
them, so both must find the same terms: every form that the late loop is built in (slices of one and two entries a lane, up to
256 and up to 512 words of a side), empty slices, half steps that one wave adds up alone and that it hands to the others, loops
that end on many changed signs."""
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


def run(scd, A, w, share, launches, form=None, limit=-1, **options):
    """form: entries of a slice and words of a side that a lane of the late loop holds; limit: see scd_probe_late_limit."""
    with scd.ScdContext(A, w, 5, options=dict(resident=0, sparse_min_mib=0, persistent_stream=0, **options)) as ctx:
        ctx.late_limit(limit)
        for g, n in launches:
            ctx.set_workgroups(share if g is None else g)
            assert ctx.engine()["engine"] == 2
            ctx.run(n)
        late = ctx.late()
        if form:
            assert (late["entries"], late["words"]) == form
            assert w == 1 or (late["alternations"] > 0) == (form[0] > 0)
            if limit >= 0:
                assert (late["returns"] > 0) == (limit == 0)
        return ctx.results(), ctx.sparse_flips(), late["alternations"]


def same(a, b):
    (ra, fa, _), (rb, fb, _) = a, b
    assert torch.equal(ra["signs"][0], rb["signs"][0]) and torch.equal(ra["signs"][1], rb["signs"][1])
    assert torch.equal(ra["iters"], rb["iters"])
    assert fa == fb
    np.testing.assert_allclose(ra["c"].cpu().numpy(), rb["c"].cpu().numpy(), rtol=1e-12)
    # (between flushes the norm follows from the cut value)
    np.testing.assert_allclose(ra["trace"].cpu().numpy(), rb["trace"].cpu().numpy(), rtol=1e-9)


# m, n, workgroups, entries and words of a lane.  Slices of 8, 16, 24 .. 128 rows or columns, one that fills its entries in part
# (72, 96); 4 to 512 words of a side (500 and 384 of the longest here); slices that are cut off and that own nothing
CASES = [(200, 200, 16, 1, 4), (512, 512, 32, 1, 4), (500, 1022, 16, 1, 4), (1024, 2048, 16, 2, 4), (1100, 1500, 16, 2, 4), (2000, 600, 100, 1, 4),
         (2048, 2048, 0, 1, 4), (4096, 1030, 64, 1, 4), (4096, 4096, 0, 1, 4), (1024, 8000, 256, 1, 4), (1000, 10000, 0, 1, 8), (10000, 1000, 0, 1, 8),
         (1024, 12288, 128, 2, 8), (9000, 1200, 100, 2, 8)]


@pytest.mark.parametrize("m,n,share,entries,words", CASES)
def test_late_alternations_find_the_same_terms(scd, m, n, share, entries, words):
    A, w = gauss((m, n), m * 7 + n), 19 if m * n < 1 << 22 else 11
    same(run(scd, A, w, share, [(None, w)], (entries, words)), run(scd, A, w, share, [(None, w)], (0, 0), sparse_delay_width=0))


FORMS = [(512, 512, 32, 1, 4), (1100, 1500, 16, 2, 4), (1024, 2048, 16, 2, 4), (1000, 10000, 0, 1, 8), (2400, 9600, 100, 2, 8), (9000, 1200, 100, 2, 8)]


@pytest.mark.parametrize("m,n,share,entries,words", FORMS)
def test_late_alternations_of_f32(scd, m, n, share, entries, words):
    """Small whole numbers: the sums of a first term are exact in either order, and so are its signs."""
    late = 0
    for seed in range(12):
        A = torch.from_numpy(np.random.Generator(np.random.PCG64(seed)).integers(-9, 10, (m, n)).astype(np.float32)).cuda()
        got = run(scd, A, 1, share, [(None, 1)], (entries, words))
        same(got, run(scd, A, 1, share, [(None, 1)], (0, 0), sparse_delay_width=0))
        late += got[2]
    assert late > 0


@pytest.mark.parametrize("limit", [0, 1 << 20])
@pytest.mark.parametrize("m,n,share,entries,words", FORMS)
def test_late_alternations_that_end_early_and_lists_in_parts(scd, m, n, share, entries, words, limit):
    """What many changed signs do, with the limits lowered: the state goes back to the other waves, and the list of a half step is
    taken a word of every lane at a time."""
    A, w = gauss((m, n), m + n), 11
    same(run(scd, A, w, share, [(None, w)], (entries, words), limit), run(scd, A, w, share, [(None, w)], (0, 0), sparse_delay_width=0))


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
            out.append((ctx.results(), ctx.sparse_flips(), 0))
    assert int(out[0][0]["iters"].max()) == 9
    same(*out)
