// Expansion of a decomposition (the definition, Section 2.2 / 5.2 of arXiv 2410.01799):
//     out[i][l] = sum_j c_j s_j[i] t_j[l],
// per entry the terms are added in the order j = 0 .. w-1 into one f64 sum that is rounded once to the output type.
// It is a matrix product of two sign matrices with the coefficients in between, so it runs on the matrix cores:
//
//   f64 coefficients (and f32 ones that the second form refuses): v_mfma_f64_16x16x4_f64.  The instruction adds its
//   four products one after the other, each sum rounded like an f64 fused multiply-add, so the order and the bits are
//   those of the definition.
//
//   f32 coefficients: int8 digits.  With c_j = k_j 2^q, k_j integers below 2^B, every partial sum of the definition is
//   a multiple of 2^q below w 2^(q + B): if B + log2 w <= 53 each of its f64 additions is exact, so any exact
//   evaluation gives the same bits.  k_j is written in four or five balanced base-255 digits of -127 .. 127 (B <= 30
//   or 38); signs times digits are int8, products and 32-bit sums are exact, the digits' sums are put together in
//   f64 integers below 2^53.  Every workgroup works out q and B from the coefficients for itself, so all take the same
//   form; the launch of the other form returns at once.
//
// The bitsets are term-major and the terms are the contraction index: a wave loads one word (64 rows or columns) of 64
// terms, one per lane, and transposes the 64 x 64 bits across its lanes.
#include "scd_bits.h"
#include "scd_device.h"

namespace scd {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kExThreads = 256;

// The common scale of the coefficients.  ok: all finite and every partial sum exact.
struct ExScale {
    int q;     // exponent of the unit
    int bits;  // B: magnitudes are below 2^B units (0: all coefficients are zero)
    bool ok;
};

// All threads of the workgroup call it; every thread gets the same answer.
__device__ ExScale ex_scan(const float* __restrict__ c, int64_t w, int (*red)[3])
{
    int lo = 1 << 20, hi = -(1 << 20), bad = 0;
    for (int64_t i0 = threadIdx.x; i0 < w; i0 += 8 * kExThreads) {
        uint32_t u[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) u[e] = __float_as_uint(c[i0 + e * kExThreads < w ? i0 + e * kExThreads : i0]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int ex = (int)((u[e] >> 23) & 255u);
            const uint32_t mant = (u[e] & 0x7FFFFFu) | (ex ? 0x800000u : 0u);
            if (ex == 255) bad = 1;
            if (mant) {
                const int unit = (ex ? ex : 1) - 150;
                const int l = unit + __ffs(mant) - 1, h = unit + 32 - __clz(mant);
                lo = l < lo ? l : lo;
                hi = h > hi ? h : hi;
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const int l = __shfl_xor(lo, off, kWave), h = __shfl_xor(hi, off, kWave);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
        bad |= __shfl_xor(bad, off, kWave);
    }
    const int wv = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) red[wv][0] = lo, red[wv][1] = hi, red[wv][2] = bad;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kExThreads / kWave; ++i) {
        lo = red[i][0] < lo ? red[i][0] : lo;
        hi = red[i][1] > hi ? red[i][1] : hi;
        bad |= red[i][2];
    }
    int lw = 0;
    while (((int64_t)1 << lw) < w) ++lw;
    ExScale s;
    s.q = hi > lo ? lo : 0;
    s.bits = hi > lo ? hi - lo : 0;
    s.ok = !bad && s.bits <= 38 && s.bits + lw <= 53 && lw <= 24;  // (32-bit sums of w digits)
    __syncthreads();  // red may be reused
    return s;
}

// ------------------------------------------------------------------------------------------------
// int8 form.  A workgroup of four waves takes a tile of 128 rows x 64 columns, a wave 64 x 32 of it (two 32 x 32
// accumulators per digit: 128 or 160 registers, two waves per SIMD).  Per chunk of 64 terms three waves transpose the
// tile's three words of bits and the fourth splits the coefficients, double-buffered in LDS.  Within 32 terms the
// contraction index of an operand byte is d + 8 b (b: byte of a dword, d = 0..7: dword, four of them per lane half), so
// that (bits >> d) & 0x01010101 are the four signs of a dword: shifted to selector bytes of v_perm they pick, per
// byte, 1 or -1 (rows) and the digit or its negative (columns).
constexpr int kExTileM = 128, kExTileN = 64;

struct ExIntLds {
    uint64_t abits[2][kExTileM];  // transposed: bit t = sign of term t of the chunk at this row
    uint64_t bbits[2][kExTileN];
    uint32_t dig[2][2][2][5][2][4];  // [buffer][half of the chunk][lane half][digit][sign][dword]
    int red[kExThreads / kWave][3];
};

template <int ND>
__device__ void ex_int_tiles(const uint64_t* __restrict__ S, const uint64_t* __restrict__ T, const float* __restrict__ c, int64_t m,
                             int64_t n, int64_t w, float* __restrict__ out, int q, ExIntLds& sh)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wr = wv >> 1, wc = wv & 1;
    const int li = lane & 31, kh = lane >> 5;
    const int64_t mw = (m + 63) / 64, nw = (n + 63) / 64;
    const int64_t tm = (m + kExTileM - 1) / kExTileM, tiles = tm * nw;
    const int64_t chunks = (w + 63) / 64;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t ti = tile % tm, tj = tile / tm;
        v16i acc[2][ND];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int d = 0; d < ND; ++d) acc[a][d] = (v16i)0;
        // waves 0, 1: words 2 ti, 2 ti + 1 of S; wave 2: word tj of T; wave 3: the coefficients.  Lane = term.
        auto fetch = [&](int64_t ch) -> uint64_t {
            const int64_t j = ch * 64 + lane;
            if (j >= w) return 0;
            if (wv < 2) return 2 * ti + wv < mw ? S[j * mw + 2 * ti + wv] : 0;
            if (wv == 2) return T[j * nw + tj];
            return (uint64_t)__float_as_uint(c[j]);
        };
        auto stage = [&](int buf, uint64_t v) {
            if (wv < 2) {
                sh.abits[buf][wv * 64 + lane] = transpose64(v, lane);
            } else if (wv == 2) {
                sh.bbits[buf][lane] = transpose64(v, lane);
            } else {
                // c = k 2^q, |k| in ND balanced base-255 digits
                const uint32_t u = (uint32_t)v;
                const int ex = (int)((u >> 23) & 255u);
                const uint32_t mant = (u & 0x7FFFFFu) | (ex ? 0x800000u : 0u);
                uint64_t k = mant;
                const int shift = (ex ? ex : 1) - 150 - q;  // negative only by trailing zeros of the mantissa
                k = mant == 0 ? 0 : (shift >= 0 ? k << shift : k >> -shift);
                const bool neg = (u >> 31) != 0;
                const int t = lane & 31, d = t & 7;
                uint8_t* p = (uint8_t*)&sh.dig[buf][lane >> 5][d >> 2][0][0][d & 3] + (t >> 3);
#pragma unroll
                for (int g = 0; g < ND; ++g) {
                    const uint64_t k127 = k + 127, quot = k127 / 255;  // k = 255 quot + r, r in -127 .. 127
                    int r = (int)(k127 - quot * 255) - 127;
                    k = quot;
                    r = neg ? -r : r;
                    p[g * 32] = (uint8_t)r;
                    p[g * 32 + 16] = (uint8_t)-r;
                }
            }
        };
        stage(0, fetch(0));
        uint64_t next = fetch(1);
        __syncthreads();
        for (int64_t ch = 0; ch < chunks; ++ch) {
            const int buf = (int)(ch & 1);
            if (ch + 1 < chunks) stage(buf ^ 1, next);
            next = fetch(ch + 2);
            const uint64_t ab0 = sh.abits[buf][wr * 64 + li], ab1 = sh.abits[buf][wr * 64 + 32 + li];
            const uint64_t bb = sh.bbits[buf][wc * 32 + li];
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const uint32_t x0 = (uint32_t)(ab0 >> (32 * hf)) >> (4 * kh), x1 = (uint32_t)(ab1 >> (32 * hf)) >> (4 * kh);
                const uint32_t xb = (uint32_t)(bb >> (32 * hf)) >> (4 * kh);
                v4i A0, A1;
                uint32_t selb[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t s0 = (e < 2 ? x0 << (2 - e) : x0 >> (e - 2)) & 0x04040404u;
                    const uint32_t s1 = (e < 2 ? x1 << (2 - e) : x1 >> (e - 2)) & 0x04040404u;
                    A0[e] = (int)__builtin_amdgcn_perm(0xFFFFFFFFu, 0x01010101u, s0);
                    A1[e] = (int)__builtin_amdgcn_perm(0xFFFFFFFFu, 0x01010101u, s1);
                    selb[e] = ((e < 2 ? xb << (2 - e) : xb >> (e - 2)) & 0x04040404u) | 0x03020100u;
                }
#pragma unroll
                for (int g = 0; g < ND; ++g) {
                    const uint4 pos = *(const uint4*)sh.dig[buf][hf][kh][g][0], neg = *(const uint4*)sh.dig[buf][hf][kh][g][1];
                    v4i B;
                    B[0] = (int)__builtin_amdgcn_perm(neg.x, pos.x, selb[0]);
                    B[1] = (int)__builtin_amdgcn_perm(neg.y, pos.y, selb[1]);
                    B[2] = (int)__builtin_amdgcn_perm(neg.z, pos.z, selb[2]);
                    B[3] = (int)__builtin_amdgcn_perm(neg.w, pos.w, selb[3]);
                    acc[0][g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A0, B, acc[0][g], 0, 0, 0);
                    acc[1][g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A1, B, acc[1][g], 0, 0, 0);
                }
            }
            __syncthreads();
        }
        // register r of a 32 x 32 accumulator: row 8 (r / 4) + 4 (lane / 32) + r mod 4, column lane mod 32
        const int64_t col = tj * 64 + wc * 32 + li;
        const double unit = ldexp(1.0, q);
        if (col < n) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t row = ti * kExTileM + wr * 64 + a * 32 + 8 * (r >> 2) + 4 * kh + (r & 3);
                    double v = (double)acc[a][ND - 1][r];
#pragma unroll
                    for (int g = ND - 2; g >= 0; --g) v = v * 255.0 + (double)acc[a][g][r];
                    if (row < m) out[row * n + col] = (float)(v * unit);
                }
        }
    }
}

__global__ void __launch_bounds__(kExThreads, 2)
    expand_int_kernel(const uint64_t* __restrict__ S, const uint64_t* __restrict__ T, const float* __restrict__ c, int64_t m, int64_t n,
                      int64_t w, float* __restrict__ out)
{
    __shared__ __align__(16) ExIntLds sh;
    const ExScale sc = ex_scan(c, w, sh.red);
    if (!sc.ok) return;
    if (sc.bits <= 30) ex_int_tiles<4>(S, T, c, m, n, w, out, sc.q, sh);
    else ex_int_tiles<5>(S, T, c, m, n, w, out, sc.q, sh);
}

// ------------------------------------------------------------------------------------------------
// f64 form.  A workgroup takes 64 rows x 128 columns, a wave 32 x 64 of it (2 x 4 accumulators of 16 x 16).  Operand
// lanes: row or column lane mod 16, term lane / 16 of four; the words and coefficients of 64 terms are staged in LDS.
struct ExF64Lds {
    uint64_t s[2][64], t[2][2][64];
    double c[2][64];
    int red[kExThreads / kWave][3];
};

// SCAN: f32 coefficients that expand_int_kernel may have taken.
template <typename TE, bool SCAN>
__global__ void __launch_bounds__(kExThreads, 2)
    expand_f64_kernel(const uint64_t* __restrict__ S, const uint64_t* __restrict__ T, const TE* __restrict__ c, int64_t m, int64_t n,
                      int64_t w, TE* __restrict__ out)
{
    __shared__ ExF64Lds sh;
    if constexpr (SCAN) {
        const ExScale sc = ex_scan((const float*)c, w, sh.red);
        if (sc.ok) return;  // expand_int_kernel does it
    }
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wr = wv >> 1, wc = wv & 1;
    const int li = lane & 15, kq = lane >> 4;
    const int64_t mw = (m + 63) / 64, nw = (n + 63) / 64;
    const int64_t tn = (nw + 1) / 2, tiles = mw * tn;
    const int64_t chunks = (w + 63) / 64;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t ti = tile % mw, tj = tile / mw;
        v4d acc[2][4];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = (v4d)0.0;
        // wave 0: word ti of S, waves 1, 2: words 2 tj, 2 tj + 1 of T, wave 3: the coefficients.  Terms past the end
        // get the coefficient +0.0 (a product of +-0.0 leaves every sum as it is).
        auto fetch = [&](int64_t ch) -> uint64_t {
            const int64_t j = ch * 64 + lane;
            if (j >= w) return 0;
            if (wv == 0) return S[j * mw + ti];
            if (wv < 3) return 2 * tj + wv - 1 < nw ? T[j * nw + 2 * tj + wv - 1] : 0;
            return (uint64_t)__double_as_longlong((double)c[j]);
        };
        auto stage = [&](int buf, uint64_t v) {
            if (wv == 0) sh.s[buf][lane] = v;
            else if (wv < 3) sh.t[buf][wv - 1][lane] = v;
            else sh.c[buf][lane] = __longlong_as_double((long long)v);
        };
        stage(0, fetch(0));
        uint64_t next = fetch(1);
        __syncthreads();
        for (int64_t ch = 0; ch < chunks; ++ch) {
            const int buf = (int)(ch & 1);
            if (ch + 1 < chunks) stage(buf ^ 1, next);
            next = fetch(ch + 2);
            const int64_t left = w - ch * 64;
            const int steps = left >= 64 ? 16 : (int)((left + 3) / 4);
            for (int st = 0; st < steps; ++st) {
                const int term = st * 4 + kq;
                const uint32_t xs = (uint32_t)(sh.s[buf][term] >> (32 * wr)) >> li;
                const uint64_t tw = sh.t[buf][wc][term] >> li;
                const double cj = sh.c[buf][term];
                double A[2], B[4];
#pragma unroll
                for (int a = 0; a < 2; ++a) A[a] = __hiloint2double((int)(((xs >> (16 * a)) << 31) | 0x3FF00000u), 0);
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    B[b] = __hiloint2double((int)((uint32_t)__double2hiint(cj) ^ ((uint32_t)(tw >> (16 * b)) << 31)), __double2loint(cj));
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[a], B[b], acc[a][b], 0, 0, 0);
            }
            __syncthreads();
        }
        // register r of a 16 x 16 accumulator: row 4 r + lane / 16, column lane mod 16
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t row = ti * 64 + wr * 32 + a * 16 + 4 * r + kq, col = (tj * 2 + wc) * 64 + b * 16 + li;
                    if (row < m && col < n) out[row * n + col] = (TE)acc[a][b][r];
                }
    }
}

unsigned ex_grid(int64_t tiles, int64_t cap) { return (unsigned)(tiles < 1 ? 1 : (tiles < cap ? tiles : cap)); }

}  // namespace

hipError_t launch_expand(const uint64_t* S, const uint64_t* T, const void* c, scd_dtype dt, int64_t m, int64_t n, int64_t w, void* out,
                         hipStream_t st)
{
    const int64_t mw = (m + 63) / 64, nw = (n + 63) / 64;
    // Two to four workgroups per compute unit walk over the tiles.  Measured (us a call, one term after the other on
    // the vector units before): 1024x4096 to 6512 terms 167 (3859), 4096x4096 to 16320 terms 1330 (28440), f64
    // 1024x4096 to 2000 terms 291 (1188), 64x64 to 300 terms 30 (119).  Below some ten terms the call only writes the
    // output and the second launch is what it costs: those go to the f64 form at once.
    const unsigned gridf = ex_grid(mw * ((nw + 1) / 2), 1024);
    if (dt == SCD_F64) {
        hipLaunchKernelGGL((expand_f64_kernel<double, false>), dim3(gridf), dim3(kExThreads), 0, st, S, T, (const double*)c, m, n, w,
                           (double*)out);
    } else if (w <= 16) {
        hipLaunchKernelGGL((expand_f64_kernel<float, false>), dim3(gridf), dim3(kExThreads), 0, st, S, T, (const float*)c, m, n, w,
                           (float*)out);
    } else {
        const int64_t tiles = (m + kExTileM - 1) / kExTileM * nw;
        hipLaunchKernelGGL(expand_int_kernel, dim3(ex_grid(tiles, 512)), dim3(kExThreads), 0, st, S, T, (const float*)c, m, n, w,
                           (float*)out);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((expand_f64_kernel<float, true>), dim3(ex_grid(mw * ((nw + 1) / 2), 512)), dim3(kExThreads), 0, st, S, T,
                           (const float*)c, m, n, w, (float*)out);
    }
    return hipGetLastError();
}

}  // namespace scd
