"""The register-resident engine (whole remainder in the register files, one persistent launch) against
the oracle and against the launch-stream path, on every shape it is built for."""
import numpy as np
import pytest
import torch

from helpers import C_RTOL, CURVE_RTOL, ID_RTOL, to_np_bits
from test_gpu_parity import lockstep_check

pytestmark = pytest.mark.gpu

SHAPES = [(1024, 4096), (2048, 2048), (4096, 4096), (256, 256), (512, 512), (1024, 1024)]
# shapes the grid overhangs (zero rows and columns in the registers), or with an oblong thread tile
RAGGED = [(4096, 1024), (2048, 4096), (1000, 4096), (2052, 516), (100, 76), (8, 8), (5, 4096), (300, 260), (1, 4),
          (1030, 520), (4000, 4092), (64, 4096), (3000, 2000)]
# rows that are no multiple of 16 bytes: first and last lengths, one and two elements past a tile or a word, the
# largest; and the shapes whose 4 x 4 grid would need a tile that it does not take
UNALIGNED = [(7, 5), (1, 6), (64, 63), (65, 257), (513, 129), (333, 1025), (1501, 999), (4096, 4093), (4095, 4095)]
SMALL_OBLONG = [(128, 704), (200, 1024), (600, 256), (1024, 60)]


@pytest.fixture(scope="module")
def scd():
    from paper_2410_01799_amd import scd as mod

    mod.lib()
    return mod


RESIDENT = {"resident": 1}
STREAM = {"resident": 0, "sparse": 0, "persistent_stream": 0}


def gauss(shape, seed):
    return np.random.Generator(np.random.PCG64(seed)).standard_normal(shape).astype(np.float32)


@pytest.mark.parametrize("m,n", SHAPES + RAGGED + UNALIGNED + SMALL_OBLONG)
def test_resident_matches_oracle_in_lockstep(scd, oracle, m, n):
    w, seed = min(10, m * n), 17
    A = gauss((m, n), m + n)
    with scd.ScdContext(torch.from_numpy(A).cuda(), w, seed, options=RESIDENT) as ctx:
        assert ctx.engine()["engine"] == 1
        ctx.run(w)
        res = ctx.results()
        R = ctx.remainder()
    S, T = to_np_bits(res["signs"][0]), to_np_bits(res["signs"][1])
    c = res["c"].cpu().numpy().astype(np.float64)
    trace = res["trace"].cpu().numpy()
    iters = res["iters"].cpu().numpy()
    # (a 1 x 4 matrix is exhausted after three terms: the identity then compares rounding noise)
    np.testing.assert_allclose(trace[1:] ** 2, trace[:-1] ** 2 - m * n * c ** 2, rtol=ID_RTOL, atol=1e-12 * trace[0] ** 2)
    curve, _ = lockstep_check(oracle, A.astype(np.float64), seed, S, T, c, trace, iters, True)
    np.testing.assert_allclose(trace, curve, rtol=2e-5, atol=1e-6 * trace[0])
    np.testing.assert_allclose(trace / trace[0], curve / curve[0], rtol=CURVE_RTOL, atol=1e-6)
    E = scd.scd_expand(res["signs"], res["c"], (m, n)).double()
    resid = float((torch.from_numpy(A).cuda().double() - E).norm())
    assert resid == pytest.approx(trace[-1], rel=1e-4, abs=1e-6 * trace[0])
    # padding bits of the sign vectors are clear, and the remainder in memory is A - expand(S, T, c)
    if m % 64:
        assert np.all(S[:, -1] >> np.uint64(m % 64) == 0)
    if n % 64:
        assert np.all(T[:, -1] >> np.uint64(n % 64) == 0)
    assert float((torch.from_numpy(A).cuda() - E.float() - R).abs().max()) <= 2e-6 * float(np.abs(A).max())


def cancelling(m, n, seed):
    """Small integers, and in rows four by four two entries of 2^27 that cancel when summed with signs +1: a sum that rounds
    to 24 bits before they meet loses the small ones, which decide the sign.  The two lie in one block of 64 columns (the
    smallest a workgroup owns) and 16 or more apart, in different threads; no other rows have large entries in these
    columns."""
    rs = np.random.Generator(np.random.PCG64(seed))
    A = rs.integers(-3, 4, (m, n)).astype(np.float32)
    first = [c for c in range(n) if c % 64 < 16 and c + 16 < n]
    for g in range(min((m + 3) // 4, len(first))):
        r = slice(4 * g, min(4 * g + 4, m))
        A[r, first[g]] = 2.0 ** 27
        A[r, first[g] + 16] = -(2.0 ** 27)
    return A


@pytest.mark.parametrize("m,n", [(130, 21), (64, 63), (65, 257), (256, 129), (257, 127), (257, 129), (513, 129), (333, 1025), (1501, 999),
                                 (3000, 1999), (4095, 4093)])
def test_resident_sums_of_rows_without_16_byte_steps(scd, oracle, m, n):
    # f64 inside a workgroup; the words exchanged are f64 up to 256 rows or 128 columns, beyond f32, which rounds a sum of
    # large entries that do not cancel (in the columns; c then holds to one such rounding, its signs are exact)
    t0 = oracle.rng_signs(3, 0, 1, n)
    td = 1.0 - 2.0 * np.unpackbits(t0.view(np.uint8), bitorder="little")[:n].astype(np.float32)
    A = np.ascontiguousarray(cancelling(m, n, m + n) * td)     # (cancels under the start of the run's first term)
    ref = oracle.greedy_signed_cut(A.astype(np.float64), t0)
    with scd.ScdContext(torch.from_numpy(A).cuda(), 1, 3, options=RESIDENT) as ctx:
        assert ctx.engine()["engine"] == 1
        ctx.run(1)
        res = ctx.results()
    assert np.array_equal(to_np_bits(res["signs"][0])[0], ref["s"])
    assert np.array_equal(to_np_bits(res["signs"][1])[0], ref["t"])
    assert int(res["iters"][0]) == ref["iters"]
    if m <= 256 or n <= 128:
        assert float(res["c"][0]) == np.float32(ref["c"] / (m * n))
    else:
        assert float(res["c"][0]) == pytest.approx(ref["c"] / (m * n), rel=2.0 ** -23)


def test_resident_sums_near_the_largest_f32(scd, oracle):
    # all entries about 1e37: the sum of a workgroup's 64 columns is beyond f32, the c of a term is not
    A = (1e37 * (1.0 + 0.01 * gauss((300, 261), 7))).astype(np.float32)
    t0 = oracle.rng_signs(3, 0, 1, 261)
    ref = oracle.greedy_signed_cut(A.astype(np.float64), t0)
    for first in (A, A / np.float32(1e20)):    # given at the start, and later
        with scd.ScdContext(torch.from_numpy(first).cuda(), 1, 3, options=RESIDENT) as ctx:
            if first is not A:
                ctx.set_remainder(torch.from_numpy(A).cuda())
            ctx.run(1)
            assert ctx.engine()["engine"] == 1
            res = ctx.results()
        assert np.array_equal(to_np_bits(res["signs"][0])[0], ref["s"]) and np.array_equal(to_np_bits(res["signs"][1])[0], ref["t"])
        assert float(res["c"][0]) == pytest.approx(ref["c"] / A.size, rel=2.0 ** -23)


# f64: half the values a thread holds and two words a value, so its own tiles (each of them once, the largest on every
# grid) and its own limit, 4096x2048 or 2048x4096 values; odd row lengths end 16-byte reads of two values
F64_SHAPES = [(1, 4), (7, 5), (64, 63), (128, 64), (256, 512), (600, 400), (1024, 1024), (1501, 999), (100, 2048), (1024, 2048),
              (2048, 1024), (4096, 513), (1024, 4096), (2048, 2048), (4096, 2048), (4095, 2047), (2048, 4096), (1030, 4093)]


@pytest.mark.parametrize("m,n", F64_SHAPES)
def test_resident_f64_matches_oracle_in_lockstep(scd, oracle, m, n):
    w, seed = min(6, m * n // 2), 23  # (a 1 x 4 matrix is exhausted after three terms)
    A = gauss((m, n), m + n).astype(np.float64) * 1.5
    with scd.ScdContext(torch.from_numpy(A).cuda(), w, seed, options=RESIDENT) as ctx:
        assert ctx.engine()["engine"] == 1
        ctx.run(w)
        res = ctx.results()
        R = ctx.remainder()
    S, T = to_np_bits(res["signs"][0]), to_np_bits(res["signs"][1])
    c, trace = res["c"].cpu().numpy(), res["trace"].cpu().numpy()
    curve, _ = lockstep_check(oracle, A, seed, S, T, c, trace, res["iters"].cpu().numpy(), False)
    # sums of up to 2^23 values in another order: 2^23 * 2^-53 relative at the very worst, about its root in practice
    np.testing.assert_allclose(trace, curve, rtol=1e-9)
    if m % 64:
        assert np.all(S[:, -1] >> np.uint64(m % 64) == 0)
    if n % 64:
        assert np.all(T[:, -1] >> np.uint64(n % 64) == 0)
    E = scd.scd_expand(res["signs"], res["c"], (m, n))
    assert float((torch.from_numpy(A).cuda() - E - R).abs().max()) <= 2e-15 * w * float(np.abs(A).max())


# matrices that one workgroup holds: every tile, exact and with overhang, their ends and one row or column past them; odd f32
# rows end at 64 values a thread
SOLO = [(64, 64), (65, 68), (64, 128), (33, 132), (128, 64), (66, 61), (128, 128), (100, 126), (64, 256), (40, 255), (256, 64), (255, 62),
        (128, 256), (127, 253), (256, 128), (129, 127), (129, 132), (129, 129), (255, 252), (256, 260), (257, 256), (255, 255)]


@pytest.mark.parametrize("m,n", SOLO)
def test_one_workgroup_matches_oracle_in_lockstep(scd, oracle, m, n):
    test_resident_matches_oracle_in_lockstep(scd, oracle, m, n)
    test_resident_f64_matches_oracle_in_lockstep(scd, oracle, m, n)


def test_one_workgroup_takes_up_where_it_left(scd):
    # launches of one term, a remainder given back and a share of the device: the same bits as one launch
    A = torch.from_numpy(gauss((200, 240), 9)).cuda()
    whole = scd.scd_decompose(A, 8, 5)
    with scd.ScdContext(A, 8, 5) as ctx:
        ctx.set_workgroups(16)
        for k in range(8):
            if k == 4:
                ctx.set_remainder(ctx.remainder())
            ctx.step()
        parts = ctx.results()
    for x, y in zip(whole["signs"] + [whole["c"], whole["iters"]], parts["signs"] + [parts["c"], parts["iters"]]):
        assert torch.equal(x, y)
    np.testing.assert_allclose(whole["trace"].cpu().numpy(), parts["trace"].cpu().numpy(), rtol=1e-8)


def test_resident_f64_limit(scd):
    """One row or column past the registers: the next engine, as for every larger matrix."""
    for m, n in [(4097, 2048), (2049, 2049), (2048, 4097)]:
        with scd.ScdContext(torch.ones((m, n), dtype=torch.float64, device="cuda"), 1, 1) as ctx:
            assert ctx.engine()["engine"] != 1


@pytest.mark.parametrize("m,n", SHAPES[:2] + SHAPES[3:])
def test_resident_and_stream_paths_agree(scd, m, n):
    A = torch.from_numpy(gauss((m, n), 5)).cuda()
    a = scd.scd_decompose(A, 8, 3, options=RESIDENT)
    b = scd.scd_decompose(A, 8, 3, options=STREAM)
    ta, tb = a["trace"].cpu().numpy(), b["trace"].cpu().numpy()
    np.testing.assert_allclose(ta / ta[0], tb / tb[0], rtol=CURVE_RTOL)
    # same signs unless a near tie split the two summation orders: then the curves still agree (above)
    if torch.equal(a["signs"][0], b["signs"][0]) and torch.equal(a["signs"][1], b["signs"][1]):
        np.testing.assert_allclose(a["c"].cpu().numpy(), b["c"].cpu().numpy(), rtol=C_RTOL)
        assert torch.equal(a["iters"], b["iters"])
        np.testing.assert_allclose(ta, tb, rtol=1e-6)


def test_resident_chunking_determinism_and_handover(scd):
    m, n = 1024, 4096
    A = torch.from_numpy(gauss((m, n), 9)).cuda()
    one = scd.scd_decompose(A, 9, 4)
    two = scd.scd_decompose(A, 9, 4)
    for k in ("c", "trace", "iters"):
        assert torch.equal(one[k], two[k])
    with scd.ScdContext(A, 12, 4) as ctx:
        ctx.step()
        ctx.run(5)
        ctx.step()
        ctx.run(2)
        assert ctx.width == 9
        res = ctx.results()
        R = ctx.remainder()
        # hand-over to the launch-stream path: profiling sweeps continue the same decomposition
        ctx.profile_sweeps(40)
        k2 = ctx.width
        res2 = ctx.results()
    assert torch.equal(one["signs"][0], res["signs"][0]) and torch.equal(one["signs"][1], res["signs"][1])
    assert torch.equal(one["c"], res["c"]) and torch.equal(one["trace"], res["trace"])
    E = scd.scd_expand(res["signs"], res["c"], (m, n))
    assert float((A - E - R).abs().max()) <= 2e-6 * float(A.abs().max())
    assert k2 >= 9
    tr = res2["trace"].cpu().numpy()
    c2 = res2["c"].cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(tr[1:] ** 2, tr[:-1] ** 2 - m * n * c2 ** 2, rtol=ID_RTOL)


def test_resident_iteration_cap(scd):
    A = torch.from_numpy(gauss((2048, 2048), 2)).cuda()
    with scd.ScdContext(A, 3, 1) as ctx:
        assert ctx.engine()["engine"] == 1
        ctx.set_max_iters(2)
        assert ctx.run(3) == scd.WMAXITER
        r = ctx.results()
    assert r["iters"].cpu().tolist() == [2, 2, 2]
    tr = r["trace"].cpu().numpy()
    c = r["c"].cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(tr[1:] ** 2, tr[:-1] ** 2 - 2048 * 2048 * c ** 2, rtol=ID_RTOL)


@pytest.mark.parametrize("grid,group", [(256, 16), (64, 8), (16, 4), (256, 4), (64, 32)])
def test_exchange_probe_runs(scd, grid, group):
    t = scd.scd_probe_exchange(0, grid, group, 200)
    assert 0 < t < 1e-3


def test_a_context_that_loses_its_share_continues_on_the_launch_stream(scd):
    m = n = 1024
    A = torch.from_numpy(gauss((m, n), 21)).cuda()
    with scd.ScdContext(A, 8, 6, options={"sparse": 0, "persistent_stream": 0}) as ctx:
        assert ctx.engine()["engine"] == 1
        ctx.run(4)
        ctx.set_workgroups(16)            # the 8 x 8 grid no longer fits, the other persistent engines are switched off
        assert ctx.engine()["engine"] == 0
        ctx.run(4)
        mixed = ctx.results()
        R = ctx.remainder()
    whole = scd.scd_decompose(A, 8, 6)
    tr = mixed["trace"].cpu().numpy()
    c = mixed["c"].cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(tr[1:] ** 2, tr[:-1] ** 2 - m * n * c ** 2, rtol=ID_RTOL)
    tw = whole["trace"].cpu().numpy()
    np.testing.assert_allclose(tr / tr[0], tw / tw[0], rtol=CURVE_RTOL)
    assert torch.equal(mixed["c"][:4], whole["c"][:4])
    E = scd.scd_expand(mixed["signs"], mixed["c"], (m, n))
    assert float((A - E - R).abs().max()) <= 2e-6 * float(A.abs().max())
