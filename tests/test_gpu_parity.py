"""GPU parity tests: the HIP path (through the C ABI) against the f64 CPU oracle, element by element,
on the same seeded inputs.  Sizes span several tiles and ragged tails; both row-pass kernels
(the generic one and the register-tiled one) are exercised.

Tolerances (north-star): bit-exact for bitsets, random streams and expansion; signs identical except
where the reference value is within 1e-6 of a tie; c within 1e-5; Frobenius identity within 1e-6;
error curve within 1e-3.
"""
import ctypes as C
import math

import numpy as np
import pytest
import torch

from helpers import (C_RTOL, CURVE_RTOL, ID_RTOL, TIE_TOL, adoption_bound, assert_signs_match, dense, match_matrix_term,
                     match_tensor_term, sign_mismatch, to_dev_bits, to_np_bits)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scd():
    from paper_2410_01799_amd import scd as mod

    mod.lib()
    assert torch.cuda.is_available()
    return mod


@pytest.fixture(params=["tiled", "generic", "persistent"])
def variant(request):
    """Options that select the streaming engines: a launch per alternation with either row-pass kernel, or the
    one persistent launch (matrices; tensors then still take a launch per sweep)."""
    if request.param == "persistent":
        return {"resident": 0, "sparse": 0}
    return {"rowpass_kernel": 1 if request.param == "tiled" else 0, "resident": 0, "sparse": 0, "persistent_stream": 0}


def gauss(shape, seed, dtype=np.float32):
    return np.random.Generator(np.random.PCG64(seed)).standard_normal(shape).astype(dtype)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# ------------------------------------------------------------------ bit-exact pieces


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000, 4096, 14336 + 17])
def test_rng_stream_bit_exact(scd, oracle, n):
    for seed, term, mode in [(0, 0, 1), (2, 8191, 1), (2 ** 63 + 5, 3, 0), (77, 12345678, 2)]:
        got = to_np_bits(scd.scd_rng_signs(seed, term, mode, n))
        assert np.array_equal(got, oracle.rng_signs(seed, term, mode, n)), (seed, term, mode, n)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1, 64, 100, 8191, 100003])
def test_pack_unpack_bit_exact(scd, oracle, dtype, n):
    x = gauss(n, n, dtype)
    x[::7] = 0.0
    x[3::11] = -0.0
    bits = scd.scd_pack(dev(x))
    ref = oracle.pack(x.astype(np.float64))
    assert np.array_equal(to_np_bits(bits), ref)
    back = scd.scd_unpack(bits, n, torch.float32 if dtype == np.float32 else torch.float64).cpu().numpy()
    assert np.array_equal(back.astype(np.float64), oracle.unpack(ref, n))


@pytest.mark.parametrize("shape,w,dtype", [((70, 130), 33, np.float32), ((64, 64), 1, np.float64),
                                           ((257, 100), 200, np.float64), ((5, 3), 7, np.float32),
                                           ((33, 10, 3), 40, np.float32), ((6, 5, 4, 3), 25, np.float64)])
def test_expand_bit_exact(scd, oracle, shape, w, dtype):
    rs = np.random.Generator(np.random.PCG64(w))
    signs = [np.stack([oracle.pack(rs.standard_normal(d)) for _ in range(w)]) for d in shape]
    c = (rs.standard_normal(w) * 10.0 ** rs.uniform(-6, 6, w)).astype(dtype)
    got = scd.scd_expand([to_dev_bits(s) for s in signs], dev(c), shape).cpu().numpy()
    ref = oracle.expand(signs, c.astype(np.float64), shape).astype(dtype)
    assert got.dtype == dtype and np.array_equal(got, ref)


@pytest.mark.parametrize("shape,w", [((1, 1), 1), ((127, 63), 63), ((128, 64), 64), ((129, 65), 65), ((200, 300), 129),
                                     ((64, 129), 700), ((40, 9, 7), 66)])
@pytest.mark.parametrize("bits", [24, 30, 31, 38, 39, 60])
def test_expand_bit_exact_over_the_span_of_the_coefficients(scd, oracle, shape, w, bits):
    # f32 coefficients that span `bits` bits from the highest to the lowest one set: 30 is the last span of four int8
    # digits, 38 of five, above that the sums are f64; a span of 53 - log2(w) bits is the last with exact sums
    signs, c = spanning(oracle, shape, w, bits)
    got = scd.scd_expand([to_dev_bits(s) for s in signs], dev(c), shape).cpu().numpy()
    ref = oracle.expand(signs, c.astype(np.float64), shape).astype(np.float32)
    assert np.array_equal(got, ref)


def spanning(oracle, shape, w, bits):
    rs = np.random.Generator(np.random.PCG64(w + bits))
    signs = [np.stack([oracle.pack(rs.standard_normal(d)) for _ in range(w)]) for d in shape]
    mant = rs.integers(1 << 23, 1 << 24, w) | 1                    # 24 significant bits
    ex = rs.integers(0, bits - 23, w)
    ex[0], ex[-1] = 0, bits - 24
    c = (np.ldexp(mant.astype(np.float64), ex - 30) * rs.choice([-1.0, 1.0], w)).astype(np.float32)
    if w > 10:
        c[w // 2] = 0.0
        c[3] = 2.0 ** -20                                           # (a power of two: trailing zeros only)
    return signs, c


# large matrices and tensors (the last tiles ragged) in all three forms, whole and cut chunks of terms, more tiles than
# workgroups
@pytest.mark.parametrize("shape,w,bits", [((1470, 1500), 33, 30), ((1470, 1500), 129, 38), ((1409, 1537), 128, 60), ((1500, 1400), 32, 24),
                                          ((130, 127 * 127), 65, 30), ((2100, 2200), 191, 30), ((512, 17, 250), 70, 31)])
def test_expand_bit_exact_on_large_tiles(scd, oracle, shape, w, bits):
    test_expand_bit_exact_over_the_span_of_the_coefficients(scd, oracle, shape, w, bits)


# operands staged behind a launch for the digits: from 449 terms on, with 64 x 64 tiles and, for more than 128 of 128 x 128,
# with those; whole and cut chunks, cut pairs of chunks, the spans' ends
@pytest.mark.parametrize("shape,w", [((1, 1), 449), ((129, 63), 512), ((64, 129), 513), ((70, 200), 500), ((40, 9, 7), 577)])
@pytest.mark.parametrize("bits", [24, 30, 31, 38, 39, 60])
def test_expand_bit_exact_with_many_terms(scd, oracle, shape, w, bits):
    test_expand_bit_exact_over_the_span_of_the_coefficients(scd, oracle, shape, w, bits)


# (every f64 sum of these is exact, so a matrix product of any order has the bits of the definition)
@pytest.mark.parametrize("shape,w,bits", [((1470, 1500), 449, 30), ((1409, 1537), 513, 38), ((1500, 1400), 512, 24), ((130, 127 * 127), 500, 31),
                                          ((2100, 2200), 513, 30), ((2100, 2200), 640, 38)])
def test_expand_bit_exact_with_many_terms_on_large_tiles(scd, oracle, shape, w, bits):
    signs, c = spanning(oracle, shape, w, bits)
    assert bits + np.ceil(np.log2(w)) <= 53
    S, T = (np.stack([oracle.unpack(x, d) for x in s]) for s, d in zip(signs, shape))
    got = scd.scd_expand([to_dev_bits(s) for s in signs], dev(c), shape).cpu().numpy()
    assert np.array_equal(got, ((S * c.astype(np.float64)[:, None]).T @ T).astype(np.float32))


def test_expand_bit_exact_with_many_terms_on_large_tiles_of_the_f64_form(scd, oracle):
    test_expand_bit_exact_over_the_span_of_the_coefficients(scd, oracle, (1409, 1537), 450, 60)


# the last term that the f64 form takes at once and the next, by the size of the matrix; the last of one launch
@pytest.mark.parametrize("shape,w", [((1024, 1024), 48), ((1024, 1024), 49), ((1025, 1024), 32), ((1025, 1024), 33), ((2049, 2048), 20),
                                     ((2049, 2048), 21), ((300, 200), 448)])
def test_expand_bit_exact_where_the_form_changes(scd, oracle, shape, w):
    test_expand_bit_exact_over_the_span_of_the_coefficients(scd, oracle, shape, w, 30)


@pytest.mark.parametrize("w", [70, 460])
def test_expand_bit_exact_at_the_ends_of_the_exponents(scd, oracle, w):
    rs = np.random.Generator(np.random.PCG64(3))
    signs = [np.stack([oracle.pack(rs.standard_normal(d)) for _ in range(w)]) for d in (66, 70)]
    db = [to_dev_bits(s) for s in signs]
    for c in (rs.integers(1, 1 << 20, w).astype(np.float32) * np.float32(2.0 ** -149), np.float32(3e38) * rs.random(w).astype(np.float32),
              np.zeros(w, np.float32), rs.standard_normal(w) * 1e-309, rs.standard_normal(w) * 1e300):
        ref = oracle.expand(signs, c.astype(np.float64), (66, 70))
        with np.errstate(over="ignore"):
            ref = ref.astype(c.dtype)
        assert np.array_equal(scd.scd_expand(db, dev(c), (66, 70)).cpu().numpy(), ref)


def test_expand_past_two_to_the_23_terms(scd):
    # the same term 9 000 000 times with the largest digit: twice a column's sum of digits passes 2^31, its entries do not
    w, word = 9_000_000, 0x5A0F33C9_71E2846B
    bits = torch.full((w, 1), word, dtype=torch.int64, device="cuda")
    got = scd.scd_expand([bits, bits], torch.full((w,), 127.0, device="cuda"), (64, 64)).cpu().numpy()
    s = np.where((np.uint64(word) >> np.arange(64, dtype=np.uint64)) & np.uint64(1), -1.0, 1.0)
    assert np.array_equal(got, (127.0 * w * np.outer(s, s)).astype(np.float32))


def test_expand_zero_terms(scd):
    out = scd.scd_expand([torch.zeros((0, 1), dtype=torch.int64, device="cuda")] * 2,
                         torch.zeros(0, dtype=torch.float32, device="cuda"), (40, 50))
    assert float(out.abs().max()) == 0.0


# ------------------------------------------------------------------ half steps (Algorithm 4 lines 5, 6-7)


HALF_SHAPES = [(256, 256), (100, 77), (1024, 4096), (130, 8200), (3, 5), (2049, 64), (520, 14336)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n", HALF_SHAPES)
def test_half_steps(scd, oracle, m, n, dtype):
    R = gauss((m, n), 1000 * m + n, dtype)
    R64 = R.astype(np.float64)
    t = oracle.rng_signs(5, 0, 1, n)
    s = oracle.rng_signs(6, 0, 0, m)
    u_ref = oracle.row_signed_sum(R64, t)
    v_ref = oracle.col_signed_sum(R64, s)
    Rd = dev(R)
    u, sb = scd.scd_row_signed_sum(Rd, to_dev_bits(t))
    v, tb, c = scd.scd_col_signed_sum(Rd, to_dev_bits(s))
    tol = 2e-6 if dtype == np.float32 else 1e-13
    np.testing.assert_allclose(u.cpu().numpy(), u_ref, rtol=0, atol=tol * np.abs(u_ref).max())
    np.testing.assert_allclose(v.cpu().numpy(), v_ref, rtol=0, atol=tol * np.abs(v_ref).max())
    assert_signs_match(to_np_bits(sb), oracle.pack(u_ref), u_ref, m, "s = sgn(R t)")
    assert_signs_match(to_np_bits(tb), oracle.pack(v_ref), v_ref, n, "t = sgn(R^T s)")
    assert float(c) == pytest.approx(np.abs(v_ref).sum(), rel=C_RTOL)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("m", [7168, 7169, 9001, 66001])
@pytest.mark.parametrize("n", [1, 3, 4, 124, 128, 131, 1020, 1023, 1024])
def test_column_half_step_of_tall_matrices(scd, m, n, dtype):
    # seven and eight rows a group, groups whose signs straddle two words, a last group that is cut short, with and
    # without 16-byte chunks.  Small integers: every sum is exact, whatever its order.
    g = torch.Generator(device="cuda").manual_seed(m + n)
    R = torch.randint(-50, 51, (m, n), generator=g, device="cuda").to(dtype)
    s = scd.scd_rng_signs(9, 1, 0, m)
    sd = scd.scd_unpack(s, m, torch.float64)
    ref = (R.double() * sd[:, None]).sum(0)
    v, t, c = scd.scd_col_signed_sum(R, s)
    assert torch.equal(v, ref) and torch.equal(t, scd.scd_pack(ref)) and float(c) == float(ref.abs().sum())


@pytest.mark.parametrize("m", [(1 << 23) - 3, (1 << 23) + 5, (1 << 27) + 70])
def test_row_half_step_of_very_many_rows(scd, m):
    # 2^23 rows go into one launch; at 2^27 rows a single one would pass the limit on threads
    i = torch.arange(m, device="cuda", dtype=torch.int32)
    R = ((i * 7919) % 1009 - 504).to(torch.float32).reshape(m, 1)
    t = torch.ones(1, dtype=torch.int64, device="cuda")        # the one column counts negative
    u, s = scd.scd_row_signed_sum(R, t)
    assert bool((u == -R[:, 0].double()).all())
    neg = torch.zeros((m + 63) // 64 * 64, dtype=torch.bool, device="cuda")
    neg[:m] = R[:, 0] > 0
    got = ((s.view(torch.uint8).unsqueeze(1) >> torch.arange(8, device="cuda", dtype=torch.uint8)) & 1).reshape(-1).bool()
    assert torch.equal(got, neg)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,m", [(64, 64), (1024, 1024), (2500, 2500), (4096, 1000), (1000, 4096)])
def test_half_steps_in_one_sign_buffer(scd, oracle, m, n, dtype):
    # a caller that alternates in one buffer: the bitset written is the one that is read (or a part of it)
    Rd = dev(gauss((m, n), m + n, dtype))
    t = to_dev_bits(oracle.rng_signs(5, 0, 1, n))
    L, st = scd.lib(), C.c_void_p(torch.cuda.current_stream().cuda_stream)
    dt = scd.F32 if dtype == np.float32 else scd.F64
    u, s = scd.scd_row_signed_sum(Rd, t)
    v, t2, _ = scd.scd_col_signed_sum(Rd, s)
    mw, nw = (m + 63) // 64, (n + 63) // 64
    for shift in (0, min(mw, nw) - 1):      # the same words, or one word in common
        for want_u in (True, False):
            buf = torch.zeros(mw + nw + shift, dtype=torch.int64, device="cuda")
            buf[:nw] = t
            uu = torch.zeros(m, dtype=torch.float64, device="cuda")
            rc = L.scd_row_signed_sum(C.c_void_p(Rd.data_ptr()), dt, m, n, C.c_void_p(buf.data_ptr()), st,
                                      C.c_void_p(uu.data_ptr()) if want_u else None, C.c_void_p(buf.data_ptr() + 8 * shift))
            assert rc == 0 and torch.equal(buf[shift:shift + mw], s) and torch.equal(buf[:shift], t[:shift])
            assert not want_u or torch.equal(uu, u)
            buf[:mw] = s
            rc = L.scd_col_signed_sum(C.c_void_p(Rd.data_ptr()), dt, m, n, C.c_void_p(buf.data_ptr()), st, None,
                                      C.c_void_p(buf.data_ptr() + 8 * shift), None)
            assert rc == 0 and torch.equal(buf[shift:shift + nw], t2)


# ------------------------------------------------------------------ one term from the same remainder and start


def check_term(scd, oracle, A, seed, options):
    """scd_step_from vs Algorithm 4 + update of the oracle, same R and t_0."""
    m, n = A.shape
    A64 = A.astype(np.float64)
    t0 = oracle.rng_signs(seed, 0, 1, n)
    g = oracle.greedy_signed_cut(A64, t0)
    with scd.ScdContext(dev(A), 4, seed, options=options) as ctx:
        ctx.step_from([None, to_dev_bits(t0)])
        assert ctx.width == 1
        res = ctx.results()
        Rg = ctx.remainder().cpu().numpy().astype(np.float64)
    s_g, t_g = to_np_bits(res["signs"][0])[0], to_np_bits(res["signs"][1])[0]
    c_g = float(res["c"][0])
    trace = res["trace"].cpu().numpy()
    sd, td = dense(s_g, m), dense(t_g, n)
    c_from_signs = sd @ A64 @ td / (m * n)
    assert c_g == pytest.approx(c_from_signs, rel=C_RTOL)
    # identity of Section 3.2 on the GPU's own numbers
    assert trace[1] ** 2 == pytest.approx(trace[0] ** 2 - m * n * c_g ** 2, rel=ID_RTOL)
    assert trace[0] == pytest.approx(np.linalg.norm(A64), rel=ID_RTOL)
    # the stored remainder is R - c s t^T
    np.testing.assert_allclose(Rg, A64 - c_g * np.outer(sd, td), rtol=0,
                               atol=(1e-6 if A.dtype == np.float32 else 1e-14) * np.abs(A64).max())
    flips, _ = match_matrix_term(oracle, A64, t0, s_g, t_g, int(res["iters"][0]), A.dtype == np.float32, str(options))
    tie_free = g["margin"].min() >= TIE_TOL
    if flips == 0:
        assert c_g == pytest.approx(g["c"] / (m * n), rel=C_RTOL)
        # the literal run ends on a repeat: (s, t) is a fixed point of the alternation
        assert_signs_match(s_g, oracle.pack(A64 @ td), A64 @ td, m, "fixed point s")
    # t is always the sign of R^T s for the s that is returned (Algorithm 4 line 6)
    assert_signs_match(t_g, oracle.pack(A64.T @ sd), A64.T @ sd, n, "t = sgn(R^T s)")
    return tie_free


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("m,n", [(256, 256), (100, 77), (64, 1024), (1000, 4096), (130, 8200), (7, 5)])
def test_term_parity(scd, oracle, variant, m, n, dtype):
    A = gauss((m, n), 31 * m + n, dtype)
    check_term(scd, oracle, A, seed=m + n, options=variant)


# ------------------------------------------------------------------ whole decompositions


def lockstep_check(oracle, A64, seed, S, T, c, trace, iters, f32):
    """The oracle follows the GPU: term k is recomputed by Algorithm 4 on the oracle's own f64 remainder from
    the keyed start.  The GPU's term must be the literal outcome or one that differs from it only through
    near-tie decisions (match_matrix_term); the oracle then continues from the GPU's signs.  The number of
    such terms is bounded by what f32 rounding explains.  Returns the oracle's curve and that number."""
    m, n = A64.shape
    R = A64.copy()
    curve = [np.linalg.norm(R)]
    adopted = 0
    for k in range(len(c)):
        flips, g = match_matrix_term(oracle, R, oracle.rng_signs(seed, k, 1, n), S[k], T[k], iters[k], f32, f"term {k}")
        if flips == 0:
            assert c[k] == pytest.approx(g["c"] / (m * n), rel=C_RTOL), f"term {k}"
        else:
            adopted += 1
        sd, td = dense(S[k], m), dense(T[k], n)
        ck = sd @ R @ td / (m * n)
        assert c[k] == pytest.approx(ck, rel=C_RTOL), f"term {k}: c does not match <s,Rt>/(mn)"
        oracle.rank1_update(R, ck, S[k], T[k])
        curve.append(math.sqrt(oracle.fro2(R)))
    decisions = float(np.sum(iters[: len(c)])) * (m + n)
    assert adopted <= adoption_bound(decisions, f32), f"{adopted} of {len(c)} terms differ from the literal run"
    return np.array(curve), adopted


@pytest.mark.parametrize("m,n,w,dtype", [(256, 256, 64, np.float32), (256, 256, 64, np.float64),
                                         (200, 333, 40, np.float32), (77, 1024, 30, np.float32),
                                         (1030, 520, 24, np.float32)])
def test_decompose_lockstep_and_free_run(scd, oracle, variant, m, n, w, dtype):
    seed = 1
    A = gauss((m, n), 1 if (m, n) == (256, 256) else m * n, dtype)
    A64 = A.astype(np.float64)
    res = scd.scd_decompose(dev(A), w, seed, options=variant)
    assert res["status"] == 0
    S, T = to_np_bits(res["signs"][0]), to_np_bits(res["signs"][1])
    c = res["c"].cpu().numpy().astype(np.float64)
    trace = res["trace"].cpu().numpy()
    iters = res["iters"].cpu().numpy()
    # Frobenius identity on the GPU's own outputs, every term
    np.testing.assert_allclose(trace[1:] ** 2, trace[:-1] ** 2 - m * n * c ** 2, rtol=ID_RTOL)
    curve, adopted = lockstep_check(oracle, A64, seed, S, T, c, trace, iters, dtype == np.float32)
    np.testing.assert_allclose(trace / trace[0], curve / curve[0], rtol=CURVE_RTOL)
    np.testing.assert_allclose(trace, curve, rtol=2e-5 if dtype == np.float32 else 1e-11)
    # free run of the oracle on the same input and seed
    free = oracle.decompose(A64, w, seed)
    np.testing.assert_allclose(trace / trace[0], free["trace"] / free["trace"][0], rtol=CURVE_RTOL)
    if adopted == 0:
        assert np.array_equal(S, free["S"]) and np.array_equal(T, free["T"])
    # definition: A - expand(S,T,c) has the norm the trace reports
    E = scd.scd_expand(res["signs"], res["c"], (m, n)).cpu().numpy().astype(np.float64)
    assert np.linalg.norm(A64 - E) == pytest.approx(trace[-1], rel=1e-4 if dtype == np.float32 else 1e-10)


def test_step_run_results_agree_with_one_shot(scd, variant):
    A = dev(gauss((300, 260), 9))
    one = scd.scd_decompose(A, 12, 4, options=variant)
    with scd.ScdContext(A, 12, 4, options=variant) as ctx:
        ctx.step()
        ctx.run(5)
        assert ctx.width == 6
        for _ in range(6):
            ctx.step()
        with pytest.raises(scd.ScdError) as e:
            ctx.step()
        assert e.value.code == scd.EFULL
        res = ctx.results()
        R = ctx.remainder()
    for a, b in zip(one["signs"], res["signs"]):
        assert torch.equal(a, b)
    assert torch.equal(one["c"], res["c"]) and torch.equal(one["trace"], res["trace"])
    assert torch.equal(one["iters"], res["iters"])
    E = scd.scd_expand(res["signs"], res["c"], (300, 260))
    assert float((A - E - R).abs().max()) <= 2e-6 * float(A.abs().max())


def test_two_runs_are_bit_identical(scd):
    A = dev(gauss((512, 768), 10))
    a = scd.scd_decompose(A, 20, 7)
    b = scd.scd_decompose(A, 20, 7)
    for x, y in zip(a["signs"] + [a["c"], a["trace"], a["iters"]], b["signs"] + [b["c"], b["trace"], b["iters"]]):
        assert torch.equal(x, y)


def test_tiled_and_generic_kernels_agree(scd):
    A = dev(gauss((384, 1024), 12))
    out = [scd.scd_decompose(A, 10, 3, options={"rowpass_kernel": v, "resident": 0, "sparse": 0, "persistent_stream": 0})
           for v in (1, 0)]
    np.testing.assert_allclose(out[0]["trace"].cpu().numpy(), out[1]["trace"].cpu().numpy(), rtol=1e-5)


def test_set_remainder_resumes_exactly(scd, variant):
    A = dev(gauss((256, 512), 13))
    full = scd.scd_decompose(A, 8, 21, options=variant)
    with scd.ScdContext(A, 8, 21, options=variant) as ctx:
        ctx.run(5)
        R5 = ctx.remainder()
        ctx.set_remainder(R5)          # same remainder: the rest of the run must not change
        ctx.run(3)
        res = ctx.results()
    assert torch.equal(full["signs"][0], res["signs"][0]) and torch.equal(full["signs"][1], res["signs"][1])
    assert torch.equal(full["c"], res["c"])
    # trace[5] was recomputed by a pass of another kind (different rounding of the f32 partial sums)
    np.testing.assert_allclose(full["trace"].cpu().numpy(), res["trace"].cpu().numpy(), rtol=1e-8)


def test_one_term_recovery_and_iteration_cap(scd, oracle):
    rs = np.random.Generator(np.random.PCG64(3))
    m, n = 130, 257
    s, t = np.sign(rs.standard_normal(m)), np.sign(rs.standard_normal(n))
    A = (0.375 * np.outer(s, t)).astype(np.float32)
    res = scd.scd_decompose(dev(A), 1, 5)
    assert float(res["c"][0]) == pytest.approx(0.375, rel=1e-6)
    assert float(res["trace"][1]) <= 1e-6 * float(res["trace"][0])
    sg, tg = dense(to_np_bits(res["signs"][0])[0], m), dense(to_np_bits(res["signs"][1])[0], n)
    assert np.array_equal(np.outer(sg, tg), np.outer(s, t))
    # the cap is reported as a warning and the result is still a valid term
    B = dev(gauss((200, 200), 4))
    with scd.ScdContext(B, 2, 1) as ctx:
        ctx.set_max_iters(1)
        assert ctx.step() == scd.WMAXITER
        r = ctx.results()
        assert int(r["iters"][0]) == 1
        tr = r["trace"].cpu().numpy()
        assert tr[1] ** 2 == pytest.approx(tr[0] ** 2 - 200 * 200 * float(r["c"][0]) ** 2, rel=ID_RTOL)


def test_error_paths(scd):
    A = dev(gauss((64, 64), 1))
    bad = A.clone()
    bad[3, 5] = float("nan")
    with pytest.raises(scd.ScdError) as e:
        scd.ScdContext(bad, 2, 0)
    assert e.value.code == scd.ENONFINITE
    with scd.ScdContext(A, 2, 0) as ctx:
        inf = A.clone()
        inf[0, 0] = float("inf")
        with pytest.raises(scd.ScdError) as e:
            ctx.set_remainder(inf)
        assert e.value.code == scd.ENONFINITE
    res = scd.scd_decompose(A, 0, 0)
    assert res["trace"].numel() == 1 and float(res["trace"][0]) == pytest.approx(float(A.double().norm()), rel=1e-6)


# ------------------------------------------------------------------ tensors (Algorithms 12 and 13)


def kron_dense(sign_rows, shape):
    out = np.array([1.0])
    for b, d in zip(sign_rows, shape):
        out = np.multiply.outer(out, dense(b, d))
    return out.reshape(shape)


@pytest.mark.parametrize("shape,w,dtype", [((40, 30, 3), 16, np.float32), ((40, 30, 3), 16, np.float64),
                                           ((130, 64, 4), 12, np.float32), ((9, 8, 7, 6), 10, np.float32),
                                           ((300, 200, 3), 8, np.float32)])
def test_tensor_decompose(scd, oracle, variant, shape, w, dtype):
    seed = 4
    a = gauss(shape, int(np.prod(shape)), dtype)
    a64 = a.astype(np.float64)
    N = a.size
    res = scd.scd_decompose(dev(a), w, seed, options=variant)
    signs = [to_np_bits(s) for s in res["signs"]]
    c = res["c"].cpu().numpy().astype(np.float64)
    trace = res["trace"].cpu().numpy()
    iters = res["iters"].cpu().numpy()
    np.testing.assert_allclose(trace[1:] ** 2, trace[:-1] ** 2 - N * c ** 2, rtol=ID_RTOL)
    # lockstep against Algorithm 12 on the oracle's own remainder
    r = a64.copy()
    for k in range(w):
        s0 = [oracle.rng_signs(seed, k, i, d) for i, d in enumerate(shape)]
        mine = [sg[k] for sg in signs]
        flips, g = match_tensor_term(oracle, r, s0, mine, iters[k], dtype == np.float32, f"term {k}")
        if flips == 0:
            assert c[k] == pytest.approx(g["c"] / N, rel=C_RTOL)
        ck = (r * kron_dense(mine, shape)).sum() / N
        assert c[k] == pytest.approx(ck, rel=C_RTOL)
        oracle.tensor_update(r, ck, mine)
        assert trace[k + 1] == pytest.approx(np.linalg.norm(r), rel=2e-5 if dtype == np.float32 else 1e-11)
    E = scd.scd_expand(res["signs"], res["c"], shape).cpu().numpy().astype(np.float64)
    assert np.linalg.norm(a64 - E) == pytest.approx(trace[-1], rel=1e-4 if dtype == np.float32 else 1e-10)


def test_tensor_step_from(scd, oracle):
    shape = (50, 40, 3)
    a = gauss(shape, 99)
    s0 = [oracle.rng_signs(8, 0, i, d) for i, d in enumerate(shape)]
    g = oracle.axial_greedy_cut(a.astype(np.float64), s0)
    with scd.ScdContext(dev(a), 2, 123) as ctx:
        ctx.step_from([None] + [to_dev_bits(b) for b in s0[1:]])
        res = ctx.results()
    flips, _ = match_tensor_term(oracle, a.astype(np.float64), s0, [to_np_bits(res["signs"][i])[0] for i in range(3)],
                                 int(res["iters"][0]), True, "step_from")
    if flips == 0:
        assert float(res["c"][0]) == pytest.approx(g["c"] / a.size, rel=C_RTOL)
