// The kernel of the register-resident engine (shared by the decomposition and the least squares decomposition, each of
// which instantiates its own forms; the rule that picks the form is in scd_resident_shape.h).
#pragma once
#include <type_traits>

#include "scd_device.h"
#include "scd_exchange.h"
#include "scd_resident_shape.h"
#include "scd_rng.h"

namespace scd {

// ---- helpers of the engine

// Sum over the 64 lanes, the same bits in every lane, without LDS traffic (a chain of ds_bpermute would cost
// an LDS round trip per step): distances 1, 2, 4, 8 by the data-parallel lane modes (4 = mirror of half a row
// then reversed quads, 8 = mirror of a row then of half a row), 16 and 32 by the row-swap instructions of
// gfx950 (swapping the odd rows of one copy with the even rows of another leaves the two partners of every
// lane in the two results, in the same order for both partners).
template <int C0, int C1>
__device__ __forceinline__ double dpp_f64_res(double v)
{
    const long long b = __double_as_longlong(v);
    int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xFFFFFFFFll), C0, 0xF, 0xF, true);
    int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), C0, 0xF, 0xF, true);
    if constexpr (C1 != 0) {
        lo = __builtin_amdgcn_update_dpp(0, lo, C1, 0xF, 0xF, true);
        hi = __builtin_amdgcn_update_dpp(0, hi, C1, 0xF, 0xF, true);
    }
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
template <int D>
__device__ __forceinline__ double swap_sum_f64_res(double a)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(a);
    const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
    unsigned l0, l1, h0, h1;
    if constexpr (D == 16) {
        const auto rl = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto rh = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        l0 = rl[0], l1 = rl[1], h0 = rh[0], h1 = rh[1];
    } else {
        const auto rl = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto rh = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        l0 = rl[0], l1 = rl[1], h0 = rh[0], h1 = rh[1];
    }
    return __longlong_as_double((long long)(((unsigned long long)h0 << 32) | l0)) +
           __longlong_as_double((long long)(((unsigned long long)h1 << 32) | l1));
}
__device__ __forceinline__ double wave_sum_res(double a)
{
    a += dpp_f64_res<0xB1, 0>(a);       // lane ^ 1
    a += dpp_f64_res<0x4E, 0>(a);       // lane ^ 2
    a += dpp_f64_res<0x141, 0x1B>(a);   // lane ^ 4
    a += dpp_f64_res<0x140, 0x141>(a);  // lane ^ 8
    a = swap_sum_f64_res<16>(a);
    a = swap_sum_f64_res<32>(a);
    return a;
}


// =================================================================================================
// Register-resident engine.
//
// A 4096 x 4096 f32 remainder is 64 MiB; the 256 compute units of the chip hold 128 MiB of vector
// registers.  Workgroup (pr, pc) of a 16 x 16 grid keeps block (pr, pc) of R in its registers for the
// whole run, so an alternation of Algorithm 4 moves no matrix data at all: only 256 partial sums per
// workgroup and phase travel through memory.
//
//   row phase   p_i = sum over the block's columns of +-R_il (signs t), published to the 16
//               workgroups of the same block row; each adds the 16 partials in order -> u_i, s_i
//   col phase   q_l = sum over the block's rows of +-R_il (signs s), published to the 16 workgroups
//               of the same block column -> v_l, t_l, and this column block's share of c = sum |v_l|
//
// Exchange: values and tag travel in one 8-byte store (the datum is its own flag, see exchange_tag), read
// back with loads that bypass the non-coherent caches; no counter, no fence.  Slots alternate by the
// parity of the sequence number: a workgroup can only be one exchange ahead of the readers of its
// slot, because finishing exchange e+1 needs data its readers publish after they have read e.
// An alternation is bound by the latency of the two exchanges and by what lies between them on one workgroup per
// compute unit (two waves per SIMD, so every vector instruction costs 8 cycles of the chain).  Measured at 4096x4096
// (us per alternation): 6.33 with barriers that also join a predicate, full-width lane reductions (every lane ends
// with every sum) and the stop test ahead of the column sums; 5.42 with one plain barrier per exchange, reductions
// that halve the registers at each step, signs kept as factor bytes, scalar bases for the gathers and the test
// behind the column sums; 4.37 with two sums in a word and 16-byte reads (2048x2048 4.59 -> 3.43, 1024x1024 3.44 -> 3.10,
// 512x512 3.31 -> 2.87).
//
// f64 (TE = double): everything the exchanges carry and the tiles hold stays 64 bits wide, so a thread holds at most 64
// values (matrices up to 4096x2048 or 2048x4096) and a word is one sum.  Us per alternation with two words a sum / with one
// (and the best of the other engines on the same matrix): 600x400 4.56 / 3.23 (9.0), 1024x1024 4.78 / 3.44 (11.2), 1501x999
// 6.79 / 3.61 (19.4, launch stream), 1024x4096 7.68 / 4.72 (15.2), 2048x2048 6.95 / 4.03 (13.6), 4096x2048 8.00 / 4.89 (9.7,
// sparse), 2048x4096 7.70 / 5.16 (9.9, sparse).
// The sum of the 16 column-block shares of c rides on the next row-phase exchange, so the test of
// Algorithm 4 line 8 is taken one phase late: the row phase already done with the final t is then
// dropped.  ||R||_F^2 after an update travels the same way (block row sums, then the total).
// Every wait is bounded; on expiry all workgroups leave and the host reports an error.

// word offset of the slot of workgroup `wg` for exchange `seq` of kind 0 (rows) or 1 (columns)
__device__ __forceinline__ uint32_t res_slot_off(int kind, uint32_t seq, int wg)
{
    return (uint32_t)(((kind * 2 + (int)(seq & 1u)) * (kResGrid * kResGrid) + wg) * kResSlotWords);
}
__device__ __forceinline__ uint64_t* res_slot(const ResidentArgs& a, int kind, uint32_t seq, int wg)
{
    return a.xbuf + res_slot_off(kind, seq, wg);
}

__device__ __forceinline__ double uniform_f64(double v)
{
    // the value is the same in every lane: keep it in scalar registers
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)(b & 0xFFFFFFFFll));
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((unsigned long long)b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Words of an exchange.  A sum that is published is scaled by a power of two so that it stays below 2 (a.xexp; a sum of up to
// 256 entries is at most 16 ||R||_F), which leaves the top bit of its exponent clear: that bit carries the tag, so that
// two f32 sums or one f64 sum (see exchange_pack) fill an 8-byte word, every 32 bits of it tell whether they are fresh, and nothing
// else has to.  f32 sums below 2^-126 of that scale lose bits, f64 ones 2^-510; infinities and NaNs have no room (the host lets
// none come here).
// A slot is read 16 bytes a lane.  Us per exchange of 256 sums alone, among 16 partners on one die / on eight: one f32 and a
// 32-bit sequence number in a word, read 8 bytes a lane 1.55 / 1.85, read 16 bytes a lane 1.60 / 1.88, two f32 in a word
// read 16 bytes a lane 1.17 / 1.49; f64 as two such words 2.50 / 2.87, as one word 1.58 / 1.89 (before
// it had a tag in both halves, 0.03 us an alternation; read by 64-bit loads instead an alternation takes 0.3 to 0.8 us more).
__device__ __forceinline__ uint32_t res_tagged(uint32_t v, uint32_t tag) { return (v & ~kTagBit) | tag; }
__device__ __forceinline__ float res_scaled(float v, int e) { return __builtin_ldexpf(v, e); }
__device__ __forceinline__ double res_scaled(double v, int e) { return __builtin_ldexp(v, e); }

__device__ __forceinline__ void res_store(uint64_t* p, uint32_t lo, uint32_t hi)
{
    __hip_atomic_store(p, ((uint64_t)hi << 32) | (uint64_t)lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// two neighbouring sums, or one
__device__ __forceinline__ void res_publish(uint64_t* p, float v0, float v1, uint32_t tag)
{
    res_store(p, res_tagged(__float_as_uint(v0), tag), res_tagged(__float_as_uint(v1), tag));
}
__device__ __forceinline__ void res_publish(uint64_t* p, double v, uint32_t tag)
{
    uint32_t lo, hi;
    exchange_pack(v, tag, lo, hi);
    res_store(p, lo, hi);
}
// The share of c, a sum over up to 256 columns of up to 4096 entries each: below 2^10 ||R||_F, so that with kShareExp more than
// the f32 sums' scale it is below 1.  Its word is stored and read by 64-bit atomics, and the upper half alone has a tag.
constexpr int kShareExp = 12;
__device__ __forceinline__ void res_publish_share(uint64_t* p, double v, uint32_t tag)
{
    res_store(p, (uint32_t)__double2loint(v), res_tagged((uint32_t)__double2hiint(v), tag));
}
// a scalar of any size: two words of half of it and the exchange's sequence number, by 64-bit atomics too
__device__ __forceinline__ void res_publish_scalar(uint64_t* p, double v, uint32_t seq)
{
    res_store(p, (uint32_t)__double2loint(v), seq);
    res_store(p + 1, (uint32_t)__double2hiint(v), seq);
}

// How the 512 threads read a slot of N sums of P partners: 16 bytes a lane and partner, L neighbouring lanes on the same
// 16 bytes of different partners, H partners a lane.
template <typename TX, int N, int P>
struct ResRead {
    static constexpr int Q = 16 / (int)sizeof(TX), U = N / Q;  // sums in 16 bytes, 16-byte pieces of a slot
    static constexpr int fit = kResThreads / U;
    static constexpr int L = P < 2 ? 1 : fit < P ? fit : P, H = P / L;
    static constexpr int waves = U * L / 64;  // waves that read sums
    static_assert(P < 2 || (L >= 4 && L <= 16 && U * L % 64 == 0 && U * L <= kResThreads), "lanes of a piece");
};

// H partners' 16 bytes (none where `sums` is not set, the same for a wave), and of one partner, at xoff, its share of c (SHARE, as
// scaled) and a scalar (SCALAR, two words later or in its place; only what the phase at hand uses is published and read: every word
// is a trip through the fabric), all loads in flight together.  If any word of the wave is still from an earlier exchange, all are
// read again (re-reads are rare once the first read is delayed a little).  xbuf and rs are the slots; soff is the same for the whole
// workgroup and voff in every exchange: nothing is worked out between the wait and the first load.  s: the sums over the partners.
template <typename TX, int H, bool SHARE, bool SCALAR>
__device__ __forceinline__ bool res_gather(const uint64_t* xbuf, __amdgpu_buffer_rsrc_t rs, uint32_t soff, uint32_t voff, uint32_t stride, bool sums,
                                           uint32_t xoff, uint32_t seq, int max_spin, double (&s)[16 / sizeof(TX)], double& share, double& scalar, int& spin)
{
    constexpr int at = SHARE ? 2 : 0;  // words before the scalar
    const uint32_t tag = exchange_tag(seq), low = tag >> 30;
    const char* base = (const char*)xbuf + soff;
    auto load = [&](int word) { return __hip_atomic_load((const uint64_t*)(base + 8 * word + xoff), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    u32x4 w[H];
    uint64_t c = 0, x0 = 0, x1 = 0;
#pragma unroll
    for (int q = 0; q < H; ++q) w[q] = sizeof(TX) == 4 ? u32x4{tag, tag, tag, tag} : u32x4{low, tag, low, tag};
    for (;;) {
        if (sums) {
#pragma unroll
            for (int q = 0; q < H; ++q) w[q] = exchange_load16(rs, voff, soff + (uint32_t)q * stride);
        }
        if constexpr (SHARE) c = load(0);
        if constexpr (SCALAR) x0 = load(at), x1 = load(at + 1);
        uint32_t stale = 0, stale_low = 0;
#pragma unroll
        for (int q = 0; q < H; ++q) {
            stale |= (w[q].y ^ tag) | (w[q].w ^ tag);
            if constexpr (sizeof(TX) == 4) stale |= (w[q].x ^ tag) | (w[q].z ^ tag);
            else stale_low |= (w[q].x ^ low) | (w[q].z ^ low);
        }
        if constexpr (SHARE) stale |= (uint32_t)(c >> 32) ^ tag;
        stale = (stale & kTagBit) | (stale_low & 1u);
        if constexpr (SCALAR) stale |= ((uint32_t)(x0 >> 32) ^ seq) | ((uint32_t)(x1 >> 32) ^ seq);
        if (__ballot(stale != 0) == 0) break;
        if (++spin > max_spin) return false;
        __builtin_amdgcn_s_sleep(1);
    }
#pragma unroll
    for (int q = 0; q < H; ++q) {
        double v[16 / sizeof(TX)];
        if constexpr (sizeof(TX) == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (double)__uint_as_float(w[q][e] & ~kTagBit);
        } else {
            v[0] = exchange_unpack(w[q].x, w[q].y);
            v[1] = exchange_unpack(w[q].z, w[q].w);
        }
#pragma unroll
        for (int e = 0; e < (int)(16 / sizeof(TX)); ++e) s[e] = q == 0 ? v[e] : s[e] + v[e];
    }
    if constexpr (SHARE) share = __hiloint2double((int)((uint32_t)(c >> 32) & ~kTagBit), (int)(uint32_t)c);
    if constexpr (SCALAR) scalar = __hiloint2double((int)(uint32_t)x1, (int)(uint32_t)x0);
    return true;
}

// Sum over the L lanes of a 16-byte piece.  At distances 1 and 2 a lane keeps only the sums whose low index bits are its own:
// lane h ends with sum h mod Q, the same bits in every lane that holds it.
template <int L, int Q>
__device__ __forceinline__ double res_join(const double (&s)[Q], int lane)
{
    const bool odd1 = (lane & 1) != 0, odd2 = (lane & 2) != 0;
    double a = (odd1 ? s[1] : s[0]) + dpp_f64_res<0xB1, 0>(odd1 ? s[0] : s[1]);  // lane ^ 1
    if constexpr (Q == 4) {
        const double b = (odd1 ? s[3] : s[2]) + dpp_f64_res<0xB1, 0>(odd1 ? s[2] : s[3]);
        a = (odd2 ? b : a) + dpp_f64_res<0x4E, 0>(odd2 ? a : b);  // lane ^ 2
    } else {
        a += dpp_f64_res<0x4E, 0>(a);
    }
    if constexpr (L >= 8) a += dpp_f64_res<0x141, 0x1B>(a);    // lane ^ 4
    if constexpr (L >= 16) a += dpp_f64_res<0x140, 0x141>(a);  // lane ^ 8
    return a;
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}

template <int CTRL>
__device__ __forceinline__ float dpp_val(float v)
{
    return dpp_f32<CTRL>(v);
}
template <int CTRL>
__device__ __forceinline__ double dpp_val(double v)
{
    return dpp_f64_res<CTRL, 0>(v);
}
__device__ __forceinline__ float res_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double res_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
// the sign bit of a factor +-1.0, at the top of a word; ck with that word's top bit flipped in
__device__ __forceinline__ uint32_t sign_of(float f) { return __float_as_uint(f) & 0x80000000u; }
__device__ __forceinline__ uint32_t sign_of(double f) { return (uint32_t)__double2hiint(f) & 0x80000000u; }
__device__ __forceinline__ float flip_by(float ck, uint32_t top) { return __uint_as_float(__float_as_uint(ck) ^ top); }
__device__ __forceinline__ double flip_by(double ck, uint32_t top)
{
    return __hiloint2double((int)((uint32_t)__double2hiint(ck) ^ top), __double2loint(ck));
}

// 16 bytes of the matrix
template <typename TE>
struct ResVec;
template <>
struct ResVec<float> {
    typedef float4 type;
    static constexpr int N = 4;
    static __device__ __forceinline__ void get(const float* p, float* x)
    {
        const float4 v = *(const float4*)p;
        x[0] = v.x, x[1] = v.y, x[2] = v.z, x[3] = v.w;
    }
    static __device__ __forceinline__ void put(float* p, const float* x) { *(float4*)p = make_float4(x[0], x[1], x[2], x[3]); }
};
template <>
struct ResVec<double> {
    typedef double2 type;
    static constexpr int N = 2;
    static __device__ __forceinline__ void get(const double* p, double* x)
    {
        const double2 v = *(const double2*)p;
        x[0] = v.x, x[1] = v.y;
    }
    static __device__ __forceinline__ void put(double* p, const double* x) { *(double2*)p = make_double2(x[0], x[1]); }
};

// Sum over groups of N = 4, 8 or 16 neighbouring lanes, the same bits in every lane of a group.
template <int N>
__device__ __forceinline__ double group_sum_res(double a)
{
    a += dpp_f64_res<0xB1, 0>(a);                          // lane ^ 1
    a += dpp_f64_res<0x4E, 0>(a);                          // lane ^ 2
    if constexpr (N >= 8) a += dpp_f64_res<0x141, 0x1B>(a);    // lane ^ 4
    if constexpr (N >= 16) a += dpp_f64_res<0x140, 0x141>(a);  // lane ^ 8
    return a;
}

// A sign is kept in LDS as the top byte of the factor +-1.0 it stands for (the same byte in f32 and f64); byte k of a
// loaded word becomes the factor's (upper) word in one instruction.
constexpr uint8_t kPosByte = 0x3F, kNegByte = 0xBF;
template <int K>
__device__ __forceinline__ void sign_factor(uint32_t bytes, float& f)
{
    f = __uint_as_float(__builtin_amdgcn_perm(bytes, 0x00800000u, 0x00020100u | ((4u + K) << 24)));
}
template <int K>
__device__ __forceinline__ void sign_factor(uint32_t bytes, double& f)
{
    f = __hiloint2double((int)__builtin_amdgcn_perm(bytes, 0x00F00000u, 0x00020100u | ((4u + K) << 24)), 0);
}
template <typename TE, int N>
__device__ __forceinline__ void sign_factors(const uint8_t* p, TE (&f)[N])
{
    uint32_t w[(N + 3) / 4];
    if constexpr (N >= 4) {
#pragma unroll
        for (int i = 0; i < N / 4; ++i) w[i] = ((const uint32_t*)p)[i];
    } else {
        w[0] = *(const uint16_t*)p;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if ((i & 3) == 0) sign_factor<0>(w[i / 4], f[i]);
        else if ((i & 3) == 1) sign_factor<1>(w[i / 4], f[i]);
        else if ((i & 3) == 2) sign_factor<2>(w[i / 4], f[i]);
        else sign_factor<3>(w[i / 4], f[i]);
    }
}

// Least squares form: the block of A (f32 or f64 as the caller has it) in f64.  Overhang is zero.
template <typename TS, int TR, int TC>
__device__ __forceinline__ void res_load_block(const TS* __restrict__ A, int64_t m, int64_t n, int64_t row0, int64_t col0,
                                               double (&x)[TR][TC])
{
    constexpr int VS = ResVec<TS>::N;
    const TS* base = A + row0 * n + col0;
    if (n % VS == 0 && ((uintptr_t)A & 15u) == 0) {  // every row starts on a 16-byte boundary
#pragma unroll
        for (int r = 0; r < TR; ++r)
#pragma unroll
            for (int c = 0; c < TC; c += VS) {
                TS v[VS];
#pragma unroll
                for (int e = 0; e < VS; ++e) v[e] = 0;
                if (row0 + r < m && col0 + c < n) ResVec<TS>::get(base + (int64_t)r * n + c, v);
#pragma unroll
                for (int e = 0; e < VS; ++e) x[r][c + e] = (double)v[e];
            }
    } else {
#pragma unroll
        for (int r = 0; r < TR; ++r)
#pragma unroll
            for (int c = 0; c < TC; ++c) x[r][c] = (row0 + r < m && col0 + c < n) ? (double)base[(int64_t)r * n + c] : 0.0;
    }
}

// x <- x - sum_j c_j s_j t_j^T for the k terms so far, in their order: one fused multiply-add per entry and term (the product
// of -c_j s_j with t_j = +-1 is exact).  The block's words of 64 terms at a time go through LDS, the next ones on their way from
// memory meanwhile: with the words of four terms in a thread's registers the chain of trips to memory was the bound
// (ms a call, before / here: 1024x1024 to 512 terms 242 / 224, 256x128 to 512 211 / 181, to 1500 1918 / 1666, 100x900 to 1500 1540 / 1431).
template <int TR, int TC>
__device__ __forceinline__ void res_subtract_terms(const ResidentArgs& a, int64_t k, int pr, int pc, uint32_t* lds, double (&x)[TR][TC])
{
    constexpr int RW = TR / 2, CW = TC / 4, REC = 1 + RW + CW, NT = 64;  // a term: coefficient, words of rows and of columns
    constexpr int PER = (NT * REC + kResThreads - 1) / kResThreads;
    const int tid = threadIdx.x, tr = tid >> 4, tc = tid & 15;
    uint64_t w[PER];
    auto fetch = [&](int64_t j0) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int at = tid + i * kResThreads, f = at % REC;
            const int64_t j = j0 + at / REC;
            const int64_t row = (int64_t)pr * RW + f - 1, col = (int64_t)pc * CW + f - 1 - RW;
            w[i] = 0;  // (past the last term: +0.0)
            if (at < NT * REC && j < k) {
                if (f == 0) w[i] = (uint64_t)__double_as_longlong(a.coef[j]);
                else if (f <= RW) w[i] = row < a.mw ? a.S[j * a.mw + row] : 0;
                else w[i] = col < a.nw ? a.T[j * a.nw + col] : 0;
            }
        }
    };
    // a thread's rows lie in one half of a word, its columns in another
    const int hr = 2 + (tr * TR >> 5), br = tr * TR & 31, hc = 2 + 2 * RW + (tc * TC >> 5), bc = tc * TC & 31;
    if (k > 0) fetch(0);
    for (int64_t j0 = 0; j0 < k; j0 += NT) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (const int at = tid + i * kResThreads; at < NT * REC) lds[2 * at] = (uint32_t)w[i], lds[2 * at + 1] = (uint32_t)(w[i] >> 32);
        __syncthreads();
        if (j0 + NT < k) fetch(j0 + NT);
        const int n = k - j0 < NT ? (int)(k - j0) : NT;
#pragma unroll 2
        for (int j = 0; j < n; ++j) {
            const uint32_t* rec = lds + 2 * j * REC;
            const double c = __hiloint2double((int)rec[1], (int)rec[0]);
            const uint32_t sb = ~(rec[hr] >> br), tb = rec[hc] >> bc;
            double t[TC];
#pragma unroll
            for (int e = 0; e < TC; ++e) t[e] = __hiloint2double((int)(0x3FF00000u | (tb << (31 - e) & 0x80000000u)), 0);
#pragma unroll
            for (int r = 0; r < TR; ++r) {
                const double cs = flip_by(c, sb << (31 - r) & 0x80000000u);  // -c_j s_j
#pragma unroll
                for (int e = 0; e < TC; ++e) x[r][e] = __builtin_fma(cs, t[e], x[r][e]);
            }
        }
    }
    const int64_t row0 = (int64_t)pr * 32 * TR + tr * TR, col0 = (int64_t)pc * 16 * TC + tc * TC;
#pragma unroll
    for (int r = 0; r < TR; ++r)
#pragma unroll
        for (int c = 0; c < TC; ++c) x[r][c] = (row0 + r < a.m && col0 + c < a.n) ? x[r][c] : 0.0;
}

// PAD: the grid overhangs the matrix (a template parameter: the 128 row/column tests of a thread's tile are
// invariants of the whole launch, and a kernel that has to keep them takes twice the instructions and runs out of
// scalar registers even when no test ever fails).
// SOLO (P = 1): a matrix that one workgroup holds.  A thread adds at most eight entries one after the other; its row sums
// are f64 across threads, its column sums f32 across the four thread rows of a wave (f64 there too: 2.24 instead of 2.17 us
// per alternation at 256x256) and f64 across waves (emulated, rms error of the row and column sums against f64, 4 x 4 workgroups / one: 256x256
// 6.9e-8, 7.4e-8 / 6.1e-8, 7.0e-8; 64x64 7.1e-8, 7.6e-8 / 4.3e-8, 5.2e-8).  Nothing is published or waited for.
// TA: type of the sums inside a workgroup, TX: of the sums that it publishes (see resident_sums; SOLO: of a thread's sums).
// LSQ: one greedy cut of A - sum c_j s_j t_j^T for the coefficients that the refit of the last term left; the position of
// the loop is the device's (a.lsq), and the refit follows as a launch of its own.
template <typename TE, typename TA, typename TX, int TR, int TC, int P, bool PAD, bool LSQ = false>
__global__ void __launch_bounds__(kResThreads) resident_kernel(ResidentArgs a)
{
    constexpr int VE = ResVec<TE>::N;
    TE* const Rm = (TE*)a.R;
    constexpr bool SOLO = P == 1;         // one workgroup holds the matrix: its sums are the sums, nothing is exchanged
    static_assert(SOLO || P == 4 || P == 8 || P == 16, "grid side");
    constexpr bool kEarly = SOLO && TR * TC >= 32;  // (with less to save, the branch costs more: 61x67 1.44 us per alternation, with it 1.53)
    using TI = std::conditional_t<SOLO && sizeof(TX) == 4, float, TA>;  // of a thread's own sums
    constexpr int BM = 32 * TR, BN = 16 * TC;  // block of this workgroup
    static_assert(TR >= 2 && TR <= 16 && (TR % 2) == 0, "rows per thread");
    static_assert(TC >= 4 && TC <= 32 && (TC % 4) == 0, "columns per thread");
    using RowRead = ResRead<TX, BM, P>;
    using ColRead = ResRead<TX, BN, P>;
    constexpr int WM = BM * (int)sizeof(TX) / 8, WN = BN * (int)sizeof(TX) / 8;  // words of sums in a slot; the scalars follow
    static_assert(WM + 4 <= kResSlotWords && WN + 4 <= kResSlotWords, "slot size");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int tr = tid >> 4, tc = tid & 15;  // 32 x 16 threads, each TR x TC elements
    const int pr = blockIdx.x / P, pc = blockIdx.x % P;
    const int wg = blockIdx.x;

    constexpr int NWV = kResThreads / 64;
    __shared__ __align__(16) TA lds_q[NWV][BN];
    __shared__ __align__(16) uint8_t lds_s[2][BM];  // signs as the top bytes of +-1.0
    __shared__ __align__(16) uint8_t lds_t[BN];
    __shared__ double lds_red[NWV];
    __shared__ double lds_x[2][P];
    __shared__ int lds_fail;  // a wait ran out in some wave; read after the barrier that follows every exchange

    // ---- load the block.  The grid may overhang the matrix: rows and columns past its end are zeros in the
    // registers (they add nothing to any sum and stay zero through every update) and are never read or written.
    const int64_t row0 = (int64_t)pr * BM + tr * TR, col0 = (int64_t)pc * BN + tc * TC;
    constexpr bool padded = PAD;
    int64_t k = a.k_start;
    uint32_t seq_u = a.seq_u, seq_v = a.seq_v;
    TE x[TR][TC];
    if constexpr (LSQ) {
        if (a.lsq->done) return;
        k = a.lsq->k;
        seq_u = a.lsq->seq_u;
        seq_v = a.lsq->seq_v;
        if (a.a_f32) res_load_block<float, TR, TC>((const float*)a.A, a.m, a.n, row0, col0, x);
        else res_load_block<double, TR, TC>((const double*)a.A, a.m, a.n, row0, col0, x);
        static_assert(sizeof(lds_q) >= 64 * (1 + TR / 2 + TC / 4) * 8, "records of 64 terms");
        res_subtract_terms<TR, TC>(a, k, pr, pc, (uint32_t*)&lds_q[0][0], x);
    } else {
        const TE* base = Rm + row0 * a.n + col0;
        if (!padded || a.n % VE == 0) {
#pragma unroll
            for (int r = 0; r < TR; ++r)
#pragma unroll
                for (int c = 0; c < TC; c += VE) {
#pragma unroll
                    for (int e = 0; e < VE; ++e) x[r][c + e] = 0;
                    if (!padded || (row0 + r < a.m && col0 + c < a.n)) ResVec<TE>::get(base + (int64_t)r * a.n + c, &x[r][c]);
                }
        } else {
            // rows that are no multiple of 16 bytes: one element at a time, once per launch
#pragma unroll
            for (int r = 0; r < TR; ++r)
#pragma unroll
                for (int c = 0; c < TC; ++c) x[r][c] = (row0 + r < a.m && col0 + c < a.n) ? base[(int64_t)r * a.n + c] : (TE)0;
        }
    }
    if (tid == 0) lds_fail = 0;
    // Values that are widened for the sums are widened anew in each phase: kept from one to the next they would take twice
    // the registers again and go through scratch (4095x4093 f32, 8 terms: 23.3 ms instead of 5.9).
    auto keep_narrow = [&]() {
        if constexpr (sizeof(TI) != sizeof(TE)) {
#pragma unroll
            for (int r = 0; r < TR; ++r)
#pragma unroll
                for (int c = 0; c < TC; ++c) asm volatile("" : "+v"(x[r][c]));
        }
    };

    int alternations = 0, updates = 0;
    int j = 0, warn = 0, cur = 0;
    double c_prev = -INFINITY;
    double cpart = 0.0;      // wave 0: this column block's sum |v_l| of the last column phase (several workgroups: times 2^-xexp)
    double fsq_block = 0.0;  // wave 0: sum of squares of this block after the last update
    double frow = 0.0;       // ... of this block row
    int norm_stage = 0;      // 1: fsq_block to publish (row exchange); 2: frow to publish (col exchange)
    int64_t norm_k = 0;
    const double total = (double)a.m * (double)a.n;
    bool need_t0 = true;
    int spin = 0, spins = 0;
    // the exchange slots as a buffer, and a thread's offsets in the two gathers (bytes; the same in every exchange)
    const __amdgpu_buffer_rsrc_t xrs = __builtin_amdgcn_make_buffer_rsrc(a.xbuf, 0, SOLO ? 0 : (int)kResXbufBytes, 0x00027000);
    const uint32_t off_u = (uint32_t)(tid % RowRead::L * RowRead::H * kResSlotWords) * 8u + (uint32_t)(tid / RowRead::L) * 16u;
    const uint32_t off_v = (uint32_t)(tid % ColRead::L * ColRead::H * P * kResSlotWords) * 8u + (uint32_t)(tid / ColRead::L) * 16u;
    const int wave = __builtin_amdgcn_readfirstlane(wv);
    const int xexp = a.xexp + (sizeof(TX) == 8 ? kF64Exp : 0);  // sums are published times 2^-xexp

    for (;;) {
        if (!LSQ && k >= a.w_target && norm_stage == 0) break;
        if (need_t0) {
            // t_0 of term k from the keyed stream (Algorithm 4 line 2)
            if (tid < BN) {
                const int64_t col = (int64_t)pc * BN + tid;
                const bool neg = col < a.n && ((rng_word(a.seed, (uint64_t)k, 1u, (uint64_t)(col >> 6)) >> (col & 63)) & 1ull);
                lds_t[tid] = neg ? kNegByte : kPosByte;
            }
            need_t0 = false;
            __syncthreads();
        }
        // One workgroup knows c at once: a term that is complete forms no further sums (the block below flips cur back).
        const bool over = kEarly && j > 0 && (uniform_f64(cpart) <= c_prev || j >= a.max_iters || (LSQ && !(fabs(uniform_f64(cpart)) < INFINITY)));
        int failed = 0;
        double cx = 0.0;
        TA qv[TC / 4];
        if (!over) {
            // ================= row phase: u = R t (Algorithm 4 line 5)
            // The signs enter as +-1.0 multipliers of a fused multiply-add: x * (+-1) is exact, so each step
            // rounds exactly like the sign-flip-and-add of Section 3.4, in one instruction instead of two
            // (this engine is bound by vector instructions and latency, not by memory).
            keep_narrow();
            TA prow;  // the row sum this lane publishes: row tc of the thread row's TR rows (lanes tc < TR)
            {
                TI tf[TC];
                sign_factors(lds_t + tc * TC, tf);
                TA p[TR];
#pragma unroll
                for (int r = 0; r < TR; ++r) {
                    // (SOLO: two runs of at most eight, so that no f32 sum is longer than it is on a 4 x 4 grid)
                    constexpr int RUN = SOLO && TC > 4 ? TC / 2 : TC;
                    TI s[TC / RUN];
#pragma unroll
                    for (int h = 0; h < TC / RUN; ++h) {
                        s[h] = 0;
#pragma unroll
                        for (int c = h * RUN; c < (h + 1) * RUN; ++c) s[h] = res_fma((TI)x[r][c], tf[c], s[h]);
                    }
                    if constexpr (TC / RUN == 2) p[r] = (TA)(s[0] + s[1]);
                    else p[r] = (TA)s[0];
                }
                // Sum over the 16 lanes that share these rows, lane distances 1, 2, 4, 8.  At distances 1 and 2 a lane
                // keeps only the rows whose low index bits are its own (it hands the others to its neighbour), which
                // halves the registers each time: lane tc ends with rows tc mod 4 and 4 + tc mod 4.
                const bool odd1 = (lane & 1) != 0, odd2 = (lane & 2) != 0;
                TA a1[TR / 2];
#pragma unroll
                for (int i = 0; i < TR / 2; ++i) {
                    const TA keep = odd1 ? p[2 * i + 1] : p[2 * i], send = odd1 ? p[2 * i] : p[2 * i + 1];
                    a1[i] = keep + dpp_val<0xB1>(send);  // lane ^ 1
                }
                if constexpr (TR == 2) {
                    TA s = a1[0];
                    s += dpp_val<0x4E>(s);   // lane ^ 2
                    s += dpp_val<0x124>(s);  // row rotate 4
                    s += dpp_val<0x128>(s);  // row rotate 8
                    prow = s;
                } else {
                    TA a2[TR / 4];
#pragma unroll
                    for (int i = 0; i < TR / 4; ++i) {
                        const TA keep = odd2 ? a1[2 * i + 1] : a1[2 * i], send = odd2 ? a1[2 * i] : a1[2 * i + 1];
                        TA s = keep + dpp_val<0x4E>(send);  // lane ^ 2
                        s += dpp_val<0x124>(s);             // row rotate 4
                        s += dpp_val<0x128>(s);             // row rotate 8
                        a2[i] = s;
                    }
                    if constexpr (TR == 8) prow = (lane & 4) ? a2[1] : a2[0];
                    else prow = a2[0];
                }
            }
            ++alternations;
            if constexpr (SOLO) {
                if (tc < TR) lds_s[cur ^ 1][tr * TR + tc] = (prow < 0) ? kNegByte : kPosByte;
            } else {
                ++seq_u;
                {
                    uint64_t* mine = res_slot(a, 0, seq_u, wg);
                    const TX pv = res_scaled((TX)prow, -xexp);
                    if constexpr (sizeof(TX) == 4) {
                        const float next = dpp_f32<0xB1>(pv);  // lane ^ 1: the row after
                        if (tc < TR && !(lane & 1)) res_publish(mine + (tr * TR + tc) / 2, pv, next, exchange_tag(seq_u));
                    } else {
                        if (tc < TR) res_publish(mine + tr * TR + tc, pv, exchange_tag(seq_u));
                    }
                    if (tid == 0) {
                        res_publish_share(mine + WM, sizeof(TX) == 4 ? res_scaled(cpart, -kShareExp) : cpart, exchange_tag(seq_u));
                        if (norm_stage == 1) res_publish_scalar(mine + WM + 2, fsq_block, seq_u);  // (only the exchange after an update)
                    }
                }
                for (int d = 0; d < a.poll_delay; ++d) __builtin_amdgcn_s_sleep(1);
                {
                    // gather; the last wave also fetches the scalars (lane mod P = partner), in the same batch of loads
                    constexpr int L = RowRead::L, H = RowRead::H, Q = RowRead::Q;
                    const uint32_t soff = res_slot_off(0, seq_u, pr * P) * 8u;
                    double hs[Q], x0 = 0.0, x1 = 0.0;
                    bool ok = true;
                    if (wave == NWV - 1) {
                        constexpr bool sums = RowRead::waves == NWV;
                        const uint32_t xoff = (uint32_t)((lane & (P - 1)) * kResSlotWords + WM) * 8u;
                        if (norm_stage == 1) ok = res_gather<TX, H, true, true>(a.xbuf, xrs, soff, off_u, kResSlotWords * 8, sums, xoff, seq_u, a.max_spin, hs, x0, x1, spin);
                        else ok = res_gather<TX, H, true, false>(a.xbuf, xrs, soff, off_u, kResSlotWords * 8, sums, xoff, seq_u, a.max_spin, hs, x0, x1, spin);
                        if (lane < P) {
                            lds_x[0][lane] = res_scaled(x0, xexp + (sizeof(TX) == 4 ? kShareExp : 0));
                            if (norm_stage == 1) lds_x[1][lane] = x1;
                        }
                    } else if (wave < RowRead::waves) {
                        ok = res_gather<TX, H, false, false>(a.xbuf, xrs, soff, off_u, kResSlotWords * 8, true, 0, seq_u, a.max_spin, hs, x0, x1, spin);
                    }
                    if (wave < RowRead::waves) {
                        const double u = res_join<L, Q>(hs, lane);
                        if (tid % L < Q) lds_s[cur ^ 1][tid / L * Q + tid % L] = (u < 0.0) ? kNegByte : kPosByte;
                    }
                    if (!ok) lds_fail = 1;
                }
            }
            // One barrier per exchange: the give-up flag is an LDS word that only ever goes from 0 to 1 and is read
            // with the data behind the barrier (__syncthreads_or takes three barriers and two more LDS round trips).
            __syncthreads();
            failed = lds_fail;
            cx = lds_x[0][lane & (P - 1)];
            cur ^= 1;  // s_j = sgn(u)

            // ================= column phase: v = R^T s (Algorithm 4 line 6), c = sum |v| (line 7).  Its sums are formed
            // before the stop test below is looked at: the test's chain of additions hides behind them, and a term that
            // ends here has formed one half step too many (once per term).
            keep_narrow();
            {
                TI sf[TR];
                sign_factors(&lds_s[cur][tr * TR], sf);
                TI q[TC];
#pragma unroll
                for (int c = 0; c < TC; ++c) {
                    TI s = 0;
#pragma unroll
                    for (int r = 0; r < TR; ++r) s = res_fma((TI)x[r][c], sf[r], s);
                    q[c] = s;
                }
                // the four thread rows of this wave hold the same columns 16 lanes apart: lane row i ends with the sums
                // of columns i TC/4 .. (i + 1) TC/4 - 1
#pragma unroll
                for (int g = 0; g < TC / 4; ++g)
                    qv[g] = (TA)half32(half16(q[g], q[TC / 4 + g]), half16(q[TC / 2 + g], q[3 * (TC / 4) + g]));
            }
        } else {
            cur ^= 1;
            __syncthreads();  // (every wave has read lds_red, which the update writes)
        }
        double c_tot;
        if constexpr (SOLO) c_tot = uniform_f64(cpart);
        else c_tot = uniform_f64(group_sum_res<P>(cx));
        if (__builtin_amdgcn_readfirstlane(failed)) {
            if (tid == 0) atomicExch((unsigned*)&a.res->err, 1u);
            return;
        }
        spins += spin;
        spin = 0;
        if constexpr (!SOLO) {
            if (norm_stage == 1) {
                frow = uniform_f64(group_sum_res<P>(lds_x[1][lane & (P - 1)]));
                norm_stage = 2;
            }
        }
        if (j > 0) {
            const bool conv = (c_tot <= c_prev) || (j >= a.max_iters) || (LSQ && !(fabs(c_tot) < INFINITY));
            if (conv) {
                // ---- the term is (c_tot, s_{j-1}, t): append it (Algorithm 5 lines 7-9) and subtract it (line 10);
                // the s of the row phase just done (lds_s[cur]) is dropped
                cur ^= 1;
                if (!(c_tot <= c_prev)) warn = 1;
                const double ck = c_tot / total;
                const TE ckf = (TE)ck;
                if (pc == 0 && wv < BM / 64) {
                    const uint64_t word = __ballot(lds_s[cur][wv * 64 + lane] == kNegByte);
                    if (lane == 0 && pr * (BM / 64) + wv < a.mw) a.S[k * a.mw + pr * (BM / 64) + wv] = word;
                }
                if (pr == 0 && wv < BN / 64) {
                    const uint64_t word = __ballot(lds_t[wv * 64 + lane] == kNegByte);
                    if (lane == 0 && pc * (BN / 64) + wv < a.nw) a.T[k * a.nw + pc * (BN / 64) + wv] = word;
                }
                if constexpr (LSQ) {
                    // (every workgroup has read the position: this one has taken part in two row exchanges and the
                    // column exchange between them, which all others had to enter first)
                    if (wg == 0 && tid == 0) {
                        a.iters[k] = j;
                        a.lsq->c_prev = c_tot;
                        a.lsq->seq_u = seq_u;
                        a.lsq->seq_v = seq_v;
                        if (warn) a.lsq->warn = 1;
                    }
                    return;
                }
                if (wg == 0 && tid == 0) {
                    ((TE*)a.c)[k] = ckf;
                    a.iters[k] = j;
                }
                TE tf[TC];
                sign_factors(lds_t + tc * TC, tf);
                double f = 0.0;
#pragma unroll
                for (int r = 0; r < TR; ++r) {
                    const uint32_t sr = ((uint32_t)lds_s[cur][tr * TR + r] & 0x80u) << 24;
#pragma unroll
                    for (int c = 0; c < TC; ++c) {
                        // R_il - ck s_i t_l: the signs choose +ck or -ck
                        const TE d = flip_by(ckf, sr ^ sign_of(tf[c]));
                        x[r][c] = (!padded || (row0 + r < a.m && col0 + c < a.n)) ? x[r][c] - d : (TE)0;  // padding stays zero
                        f += (double)x[r][c] * (double)x[r][c];
                    }
                }
                f = wave_sum_res(f);
                if (lane == 0) lds_red[wv] = f;
                __syncthreads();
                if (wv == 0) {
                    double fb = 0.0;
#pragma unroll
                    for (int q = 0; q < NWV; ++q) fb += lds_red[q];
                    fsq_block = uniform_f64(fb);
                    if (SOLO && tid == 0) a.trace[k + 1] = sqrt(fsq_block);
                }
                ++k;
                ++updates;
                norm_stage = SOLO ? 0 : 1;
                norm_k = k;
                j = 0;
                c_prev = -INFINITY;
                cpart = 0.0;
                need_t0 = true;
                __syncthreads();  // lds_t and lds_red are rewritten next
                continue;
            }
            c_prev = c_tot;
        }
        {
            // lane (i, tc) holds TC/4 neighbouring columns
            constexpr int VA = ResVec<TA>::N;
            TA* dst = &lds_q[wv][tc * TC + (lane >> 4) * (TC / 4)];
            if constexpr (TC / 4 >= VA) {
#pragma unroll
                for (int g = 0; g < TC / 4; g += VA) ResVec<TA>::put(dst + g, qv + g);
            } else {
#pragma unroll
                for (int g = 0; g < TC / 4; ++g) dst[g] = qv[g];
            }
        }
        __syncthreads();
        double absv = 0.0;
        if constexpr (SOLO) {
            if (tid < BN) {
                TA w[NWV];
#pragma unroll
                for (int q = 0; q < NWV; ++q) w[q] = lds_q[q][tid];
                asm volatile("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(w[4]), "+v"(w[5]), "+v"(w[6]), "+v"(w[7]));
                const TA v = ((w[0] + w[1]) + (w[2] + w[3])) + ((w[4] + w[5]) + (w[6] + w[7]));
                lds_t[tid] = (v < 0) ? kNegByte : kPosByte;
                absv = fabs((double)v);
            }
        } else {
            ++seq_v;
            {
                uint64_t* mine = res_slot(a, 1, seq_v, wg);
                constexpr int C = 8 / (int)sizeof(TX);  // columns of a word
                if (tid < BN / C) {
                    // (all loads in flight together, then the adds in wave order: the empty asm keeps the compiler from
                    // loading two, waiting, adding two)
                    TA w[C][NWV];
#pragma unroll
                    for (int q = 0; q < NWV; ++q)
#pragma unroll
                        for (int e = 0; e < C; ++e) w[e][q] = lds_q[q][tid * C + e];
                    static_assert(NWV == 8, "operands of the asm");
                    TX s[C];
#pragma unroll
                    for (int e = 0; e < C; ++e) asm volatile("" : "+v"(w[e][0]), "+v"(w[e][1]), "+v"(w[e][2]), "+v"(w[e][3]), "+v"(w[e][4]), "+v"(w[e][5]), "+v"(w[e][6]), "+v"(w[e][7]));
#pragma unroll
                    for (int e = 0; e < C; ++e) {
                        TA t = 0;
#pragma unroll
                        for (int q = 0; q < NWV; ++q) t += w[e][q];
                        s[e] = res_scaled((TX)t, -xexp);
                    }
                    if constexpr (C == 2) res_publish(mine + tid, s[0], s[1], exchange_tag(seq_v));
                    else res_publish(mine + tid, s[0], exchange_tag(seq_v));
                }
                if (norm_stage == 2 && tid == kResThreads - 1) res_publish_scalar(mine + WN, frow, seq_v);
            }
            for (int d = 0; d < a.poll_delay_v; ++d) __builtin_amdgcn_s_sleep(1);
            {
                constexpr int L = ColRead::L, H = ColRead::H, Q = ColRead::Q;
                const uint32_t soff = res_slot_off(1, seq_v, pc) * 8u;
                double hs[Q], x0 = 0.0, x1 = 0.0;
                bool ok = true;
                if (norm_stage == 2 && wave == NWV - 1) {
                    // the block-row sums of squares travel on this exchange once per term
                    const uint32_t xoff = (uint32_t)((lane & (P - 1)) * P * kResSlotWords + WN) * 8u;
                    ok = res_gather<TX, H, false, true>(a.xbuf, xrs, soff, off_v, P * kResSlotWords * 8, ColRead::waves == NWV, xoff, seq_v, a.max_spin, hs, x0, x1, spin);
                    if (lane < P) lds_x[1][lane] = x1;
                } else if (wave < ColRead::waves) {
                    ok = res_gather<TX, H, false, false>(a.xbuf, xrs, soff, off_v, P * kResSlotWords * 8, true, 0, seq_v, a.max_spin, hs, x0, x1, spin);
                }
                if (wave < ColRead::waves) {
                    const double v = res_join<L, Q>(hs, lane);
                    if (tid % L < Q) {
                        lds_t[tid / L * Q + tid % L] = (v < 0.0) ? kNegByte : kPosByte;
                        absv = fabs(v);
                    }
                }
                if (!ok) lds_fail = 1;
            }
        }
        absv = wave_sum_res(absv);
        if (lane == 0) lds_red[wv] = absv;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(lds_fail)) {
            if (tid == 0) atomicExch((unsigned*)&a.res->err, 1u);
            return;
        }
        // this column block's share of c (in the exchange's scale) travels on the next row exchange (published by thread 0)
        if (SOLO || wv == 0) cpart = group_sum_res<8>(lds_red[lane & (NWV - 1)]);
        if constexpr (!SOLO) {
            if (norm_stage == 2) {
                const double ft = group_sum_res<P>(lds_x[1][lane & (P - 1)]);
                if (wg == 0 && tid == 0) a.trace[norm_k] = sqrt(ft);
                norm_stage = 0;
            }
        }
        ++j;
        spins += spin;
        spin = 0;
        // No barrier here: what was read above (lds_red, lds_x[1]) is next written after the two barriers of the
        // coming row and column phases (lds_x[1] in a row phase only right after an update, never right after
        // the column phase that read it), and what the coming row phase writes first (lds_s of the other
        // parity, lds_x[0]) was last read before this phase's barriers.
    }

    // ---- write the block back
    {
        TE* base = Rm + row0 * a.n + col0;
        if (!padded || a.n % VE == 0) {
#pragma unroll
            for (int r = 0; r < TR; ++r)
#pragma unroll
                for (int c = 0; c < TC; c += VE)
                    if (!padded || (row0 + r < a.m && col0 + c < a.n)) ResVec<TE>::put(base + (int64_t)r * a.n + c, &x[r][c]);
        } else {
#pragma unroll
            for (int r = 0; r < TR; ++r)
#pragma unroll
                for (int c = 0; c < TC; ++c)
                    if (row0 + r < a.m && col0 + c < a.n) base[(int64_t)r * a.n + c] = x[r][c];
        }
    }
    if (wg == 0 && tid == 0) {
        a.res->k = k;
        a.res->alternations = alternations;
        a.res->updates = updates;
        a.res->seq_u = seq_u;
        a.res->seq_v = seq_v;
        a.res->warn = warn;
        a.res->spins = spins;
    }
}

template <int P_, int TR_, int TC_>
struct ResTile {
    static constexpr int P = P_, TR = TR_, TC = TC_;
    static constexpr bool taken(scd_dtype dt, int form) { return kResForms.taken(dt, form, P, TR, TC); }
};
// f(ResTile) for the numbers that resident_shape gives
template <int P, int TR, typename F>
hipError_t res_with_columns(int tc, F& f)
{
    if (tc == 4) return f(ResTile<P, TR, 4>());
    return tc == 8 ? f(ResTile<P, TR, 8>()) : f(ResTile<P, TR, 16>());
}
template <int P, typename F>
hipError_t res_with_rows(int tr, int tc, F& f)
{
    if (tr == 2) return res_with_columns<P, 2>(tc, f);
    return tr == 4 ? res_with_columns<P, 4>(tc, f) : res_with_columns<P, 8>(tc, f);
}
template <typename F>
hipError_t res_with_tile(int p, int tr, int tc, F f)
{
    if (p == 1) return res_with_rows<1>(tr, tc, f);
    if (p == 4) return res_with_rows<4>(tr, tc, f);
    return p == 8 ? res_with_rows<8>(tr, tc, f) : res_with_rows<16>(tr, tc, f);
}

}  // namespace scd
