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
//   f64 integers below 2^53.  With few terms every workgroup works out q, B and the digits for itself; with many a launch
//   ahead does; the form that applies is taken on the device.
//
// The bitsets are term-major and the terms are the contraction index: a wave loads one word (64 rows or columns) of 64
// terms, one per lane, and transposes the 64 x 64 bits across its lanes.
#include <type_traits>

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

// All threads of a workgroup call it; every thread gets the same answer.
constexpr int kExScanThreads = 1024;  // of the launch that works out the digits
template <int THREADS>
__device__ ExScale ex_scan(const float* __restrict__ c, int64_t w, int (*red)[3])
{
    int lo = 1 << 20, hi = -(1 << 20), bad = 0;
    for (int64_t i0 = threadIdx.x; i0 < w; i0 += 8 * THREADS) {
        uint32_t u[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) u[e] = __float_as_uint(c[i0 + e * THREADS < w ? i0 + e * THREADS : i0]);
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
    for (int i = 0; i < THREADS / kWave; ++i) {
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

// A coefficient (its bits) as k 2^q, k in ND balanced base-255 digits.
template <int ND>
__device__ __forceinline__ void ex_digits(uint32_t u, int q, int (&r)[ND])
{
    const int ex = (int)((u >> 23) & 255u);
    const uint32_t mant = (u & 0x7FFFFFu) | (ex ? 0x800000u : 0u);
    uint64_t k = mant;
    const int shift = (ex ? ex : 1) - 150 - q;  // negative only by trailing zeros of the mantissa
    k = mant == 0 ? 0 : (shift >= 0 ? k << shift : k >> -shift);
    const bool neg = (u >> 31) != 0;
#pragma unroll
    for (int g = 0; g < ND; ++g) {
        const uint64_t k127 = k + 127, quot = k127 / 255;  // k = 255 quot + r, r in -127 .. 127
        const int d = (int)(k127 - quot * 255) - 127;
        k = quot;
        r[g] = neg ? -d : d;
    }
}

// ------------------------------------------------------------------------------------------------
// f64 form.  A workgroup takes 64 rows x 128 columns, a wave 32 x 64 of it (2 x 4 accumulators of 16 x 16).  Operand
// lanes: row or column lane mod 16, term lane / 16 of four; the words and coefficients of 64 terms are staged in LDS.
struct ExF64Lds {
    uint64_t s[2][64], t[2][2][64];
    double c[2][64];
};

// TEAMS: groups of kExThreads threads in a workgroup, a tile each.
template <typename TE, int TEAMS>
__device__ __forceinline__ void ex_f64_tiles(const uint64_t* __restrict__ S, const uint64_t* __restrict__ T, const TE* __restrict__ c, int64_t m,
                                             int64_t n, int64_t w, TE* __restrict__ out, ExF64Lds* lds)
{
    ExF64Lds& sh = lds[threadIdx.x / kExThreads];
    const int tid = threadIdx.x % kExThreads, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wr = wv >> 1, wc = wv & 1;
    const int li = lane & 15, kq = lane >> 4;
    const int64_t mw = (m + 63) / 64, nw = (n + 63) / 64;
    const int64_t tn = (nw + 1) / 2, tiles = mw * tn;
    const int64_t chunks = (w + 63) / 64;
    const int64_t first = (int64_t)blockIdx.x * TEAMS + threadIdx.x / kExThreads, step = (int64_t)gridDim.x * TEAMS;
    for (int64_t base = 0; base < tiles; base += step) {
        // (the teams of a workgroup share its barriers: one that is past the last tile works on it again)
        const bool mine = base + first < tiles;
        const int64_t tile = mine ? base + first : tiles - 1;
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
                    if (mine && row < m && col < n) out[row * n + col] = (TE)acc[a][b][r];
                }
    }
}

template <typename TE>
__global__ void __launch_bounds__(kExThreads, 2)
    expand_f64_kernel(const uint64_t* __restrict__ S, const uint64_t* __restrict__ T, const TE* __restrict__ c, int64_t m, int64_t n,
                      int64_t w, TE* __restrict__ out)
{
    __shared__ ExF64Lds sh;
    ex_f64_tiles<TE, 1>(S, T, c, m, n, w, out, &sh);
}

// ------------------------------------------------------------------------------------------------
// int8 form in one launch, for few terms.  Every workgroup scans the coefficients and forms their digits itself; tiles of
// 128 rows x 64 columns on four waves, 64 x 32 each (two 32 x 32 accumulators per digit), two workgroups per compute unit, so
// that the store of one tile overlaps with the products of another.  Per chunk of 64 terms three waves transpose the
// tile's three words of bits and the fourth splits the coefficients, double-buffered in LDS; operand bytes as below, a column's
// byte the digit or its negative.  Bound by the store of the output and the ends of the tiles (4096x4096 to 33 terms 34 us
// a call, staged operands 47; see launch_expand).
constexpr int kExDirectM = 128, kExDirectN = 64;

struct ExDirectLds {
    uint64_t abits[2][kExDirectM];   // transposed: bit t = sign of term t of the chunk at this row
    uint64_t bbits[2][kExDirectN];
    uint32_t dig[2][2][2][5][2][4];  // [buffer][half of the chunk][lane half][digit][sign][dword]
};

template <int ND>
__device__ __forceinline__ void ex_direct_tiles(const uint64_t* __restrict__ S, const uint64_t* __restrict__ T, const float* __restrict__ c,
                                                int64_t m, int64_t n, int64_t w, float* __restrict__ out, int q, ExDirectLds& sh)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wr = wv >> 1, wc = wv & 1;
    const int li = lane & 31, kh = lane >> 5;
    const int64_t mw = (m + 63) / 64, nw = (n + 63) / 64;
    const int64_t tm = (m + kExDirectM - 1) / kExDirectM, tiles = tm * nw;
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
                int r[ND];
                ex_digits<ND>((uint32_t)v, q, r);
                const int t = lane & 31, d = t & 7;
                uint8_t* p = (uint8_t*)&sh.dig[buf][lane >> 5][d >> 2][0][0][d & 3] + (t >> 3);
#pragma unroll
                for (int g = 0; g < ND; ++g) {
                    p[g * 32] = (uint8_t)r[g];
                    p[g * 32 + 16] = (uint8_t)-r[g];
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
                    A0[e] = (int)__builtin_amdgcn_perm(0xFFFFFFFFu, 0x01010101u, (e < 2 ? x0 << (2 - e) : x0 >> (e - 2)) & 0x04040404u);
                    A1[e] = (int)__builtin_amdgcn_perm(0xFFFFFFFFu, 0x01010101u, (e < 2 ? x1 << (2 - e) : x1 >> (e - 2)) & 0x04040404u);
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
                    const int64_t row = ti * kExDirectM + wr * 64 + a * 32 + 8 * (r >> 2) + 4 * kh + (r & 3);
                    double v = (double)acc[a][ND - 1][r];
#pragma unroll
                    for (int g = ND - 2; g >= 0; --g) v = v * 255.0 + (double)acc[a][g][r];
                    if (row < m) out[row * n + col] = (float)(v * unit);
                }
        }
    }
}

__global__ void __launch_bounds__(kExThreads, 2)
    expand_direct_kernel(const uint64_t* __restrict__ S, const uint64_t* __restrict__ T, const float* __restrict__ c, int64_t m, int64_t n,
                         int64_t w, float* __restrict__ out)
{
    __shared__ __align__(16) union {
        ExDirectLds d;
        ExF64Lds f;
        int red[kExThreads / kWave][3];
    } sh;
    const ExScale sc = ex_scan<kExThreads>(c, w, sh.red);
    if (!sc.ok) ex_f64_tiles<float, 1>(S, T, c, m, n, w, out, &sh.f);
    else if (sc.bits <= 30) ex_direct_tiles<4>(S, T, c, m, n, w, out, sc.q, sh.d);
    else ex_direct_tiles<5>(S, T, c, m, n, w, out, sc.q, sh.d);
}

// ------------------------------------------------------------------------------------------------
// int8 form.  expand_digits_kernel writes the scale and the digits once per call; the tile kernel then runs on three
// stages per chunk of 64 terms, one barrier apart:
//   chunk ch + 2  the tile's words of bits are transposed across a wave (lane = term -> lane = row or column), each wave
//                 32 terms of one word
//   chunk ch + 1  the operand bytes are formed, 16 terms of one row (1 or -1) and of one column (digit or zero,
//                 ND of them) per thread, and laid out in LDS as the instructions take them
//   chunk ch      a wave multiplies: AR x 1 accumulators of 32 x 32 per digit, operands straight from LDS
// Within 32 terms the contraction index of an operand byte is d + 8 b (b: byte of a dword, d = 0..7: dword, four of them
// per lane half), so that (bits >> d) & 0x01010101 are the four signs of a dword: shifted to selector bytes of v_perm they
// pick, per byte, 1 or -1.  With t = 1 - 2 u (u = 1 where the sign is -1), sum s d t = sum s d - 2 sum s d u: a
// column's byte is the digit or zero, one AND with a scalar, and the first sum, one per row, comes from four-byte dot
// products of the row's bytes while they are in registers.  Operands are read a half chunk ahead of the instructions that
// take them (three buffers).  Bound by the matrix unit and by what it does not overlap with: 1024x4096 to 6512 terms takes
// 114 us (166), of which 48 are products at the clock it runs at (2.15 GHz); the vector unit issues for 36 % of the time.
struct ExPlan {
    int32_t ok;      // the int8 form applies
    int32_t digits;  // 4 or 5
    int32_t q;       // exponent of the unit
    int32_t pad[13];
};
constexpr int kExDigits = 5;                                  // most digits
constexpr int kExChunkDwords = 2 * 2 * kExDigits * 4;         // [half of the chunk][lane half][digit][dword]

__global__ void __launch_bounds__(kExScanThreads)
    expand_digits_kernel(const float* __restrict__ c, int64_t w, ExPlan* __restrict__ plan, uint32_t* __restrict__ dig)
{
    __shared__ int red[kExScanThreads / kWave][3];
    const ExScale sc = ex_scan<kExScanThreads>(c, w, red);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        plan->ok = sc.ok ? 1 : 0;
        plan->digits = sc.bits <= 30 ? 4 : 5;
        plan->q = sc.q;
    }
    if (!sc.ok) return;
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int64_t chunks = (w + 127) / 128 * 2;
    for (int64_t ch = (int64_t)blockIdx.x * (kExScanThreads / kWave) + wv; ch <= chunks; ch += (int64_t)gridDim.x * (kExScanThreads / kWave)) {
        // terms past the end are zero
        const int64_t j = ch * 64 + lane;
        int r[kExDigits];
        ex_digits<kExDigits>(j < w ? __float_as_uint(c[j]) : 0u, sc.q, r);
        const int t = lane & 31, d = t & 7;
        uint8_t* p = (uint8_t*)(dig + ch * kExChunkDwords + (((lane >> 5) * 2 + (d >> 2)) * kExDigits) * 4 + (d & 3)) + (t >> 3);
#pragma unroll
        for (int g = 0; g < kExDigits; ++g) p[g * 16] = (uint8_t)r[g];
    }
}

// RW, CW: words of 64 rows and columns of a workgroup's tile; four waves per word pair.  AR: 32-row accumulators of a wave.
template <int RW, int CW>
struct ExTile {
    static constexpr int kM = 64 * RW, kN = 64 * CW, kWaves = 4 * (RW > CW ? RW : CW), kThreads = kWaves * kWave;
    static constexpr int kAcross = CW * 2;                       // waves side by side, 32 columns each
    static constexpr int kAR = RW * 2 / (kWaves / kAcross);      // 32-row blocks per wave
    static constexpr int kWords = RW + CW;
    struct Lds {
        uint32_t bits[2][2][RW + CW][kWave];  // [buffer][half][word][row or column]: bit t = sign of term t of the half
        uint4 a[3][2][2][kM];                 // [buffer][half][lane half][row]
        uint4 b[3][kExDigits][2][2][kN];      // [buffer][digit][half][lane half][column]
        int rows[kM][kExDigits];              // sums of s_j times digit over all terms
    };
};

template <int RW, int CW, int ND>
__device__ __forceinline__ void ex_int_tiles(const uint64_t* __restrict__ S, const uint64_t* __restrict__ T, const uint32_t* __restrict__ dig,
                                             int64_t m, int64_t n, int64_t w, float* __restrict__ out, int q,
                                             typename ExTile<RW, CW>::Lds& sh)
{
    typedef ExTile<RW, CW> Tile;
    constexpr int AR = Tile::kAR;
    static_assert(RW == CW && Tile::kWaves == 2 * Tile::kWords, "a wave: one row and one column item and half a word per chunk");
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wr = wv / Tile::kAcross, wc = wv % Tile::kAcross;
    const int li = lane & 31, kh = lane >> 5;
    const int my = wv >> 1, myh = wv & 1;                       // the wave's bits to transpose: word and half of the chunk
    const int ihf = (wv >> 1) & 1, ikh = wv & 1, iw = wv >> 2;  // the wave's operand bytes: terms and word
    const int64_t mw = (m + 63) / 64, nw = (n + 63) / 64;
    const int64_t tm = (mw + RW - 1) / RW, tn = (nw + CW - 1) / CW, tiles = tm * tn;
    const int chunks = (int)((w + 127) / 128) * 2;  // (w is at most 2^24 here; the digits of what is past the end are zero)
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t ti = tile % tm, tj = tile / tm;
        v16i acc[AR][ND];
#pragma unroll
        for (int a = 0; a < AR; ++a)
#pragma unroll
            for (int d = 0; d < ND; ++d) acc[a][d] = (v16i)0;
        // 32 terms of one word: lane = term, lower half of the lanes the lower half of the word.  Terms past the last one
        // re-read it, words past the end of a vector re-read the first (their rows and columns are not stored): the load has
        // no condition and nothing waits for it here.
        const bool row = my < RW;
        const int64_t words = row ? mw : nw, word = row ? ti * RW + my : tj * CW + (my - RW);
        const uint32_t* src = (const uint32_t*)((row ? S : T) + (word < words ? word : 0)) + kh;
        const uint32_t last = (uint32_t)(w - 1), stride = (uint32_t)(words * 8), mine = (uint32_t)(myh * 32 + li);
        auto fetch = [&](int ch) {
            const uint32_t j = (uint32_t)ch * 64u + mine;
            return *(const uint32_t*)((const char*)src + (uint64_t)(j < last ? j : last) * stride);
        };
        auto transpose = [&](uint32_t h) {
            h = bit_butterfly<16>(h, lane);
            h = bit_butterfly<8>(h, lane);
            h = bit_butterfly<4>(h, lane);
            h = bit_butterfly<2>(h, lane);
            return bit_butterfly<1>(h, lane);
        };
        // the digits of the wave's terms: the same for all lanes, in scalar registers
        const uint32_t* dbase = dig + (ihf * 2 + ikh) * kExDigits * 4;
        auto digits = [&](int ch, uint32_t (&d)[ND][4]) {
            const uint32_t* p = dbase + (ch < chunks ? ch : chunks) * kExChunkDwords;  // (one more chunk, all zero)
#pragma unroll
            for (int g = 0; g < ND; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) d[g][e] = p[g * 4 + e];
        };
        int usum[ND];
#pragma unroll
        for (int g = 0; g < ND; ++g) usum[g] = 0;
        auto build = [&](int par, int buf, const uint32_t (&d)[ND][4]) {
            const uint32_t xa = sh.bits[par][ihf][iw][lane] >> (4 * ikh), xb = sh.bits[par][ihf][RW + iw][lane] >> (4 * ikh);
            uint32_t A[4], neg[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                A[e] = __builtin_amdgcn_perm(0xFFFFFFFFu, 0x01010101u, (e < 2 ? xa << (2 - e) : xa >> (e - 2)) & 0x04040404u);
                neg[e] = __builtin_amdgcn_perm(0xFFFFFFFFu, 0u, (e < 2 ? xb << (2 - e) : xb >> (e - 2)) & 0x04040404u);
            }
            sh.a[buf][ihf][ikh][iw * kWave + lane] = make_uint4(A[0], A[1], A[2], A[3]);
#pragma unroll
            for (int g = 0; g < ND; ++g) {
                sh.b[buf][g][ihf][ikh][iw * kWave + lane] = make_uint4(d[g][0] & neg[0], d[g][1] & neg[1], d[g][2] & neg[2], d[g][3] & neg[3]);
#pragma unroll
                for (int e = 0; e < 4; ++e) usum[g] = __builtin_amdgcn_sdot4((int)A[e], (int)d[g][e], usum[g], false);
            }
        };
        v4i A[2][AR], B[2][ND];
        auto load = [&](int buf, int hf) {
#pragma unroll
            for (int a = 0; a < AR; ++a) A[hf][a] = *(const v4i*)&sh.a[buf][hf][kh][(wr * AR + a) * 32 + li];
#pragma unroll
            for (int g = 0; g < ND; ++g) B[hf][g] = *(const v4i*)&sh.b[buf][g][hf][kh][wc * 32 + li];
        };
        auto multiply = [&](int hf) {
#pragma unroll
            for (int g = 0; g < ND; ++g)
#pragma unroll
                for (int a = 0; a < AR; ++a) acc[a][g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[hf][a], B[hf][g], acc[a][g], 0, 0, 0);
        };
        uint32_t next, dg[ND][4];
        {
            const uint32_t b0 = fetch(0), b1 = fetch(1), b2 = fetch(2);
            digits(0, dg);
            sh.bits[0][myh][my][lane] = transpose(b0);
            sh.bits[1][myh][my][lane] = transpose(b1);
            __syncthreads();
            build(0, 0, dg);
            digits(1, dg);
            build(1, 1, dg);
            __syncthreads();
            sh.bits[0][myh][my][lane] = transpose(b2);
            digits(2, dg);
            next = fetch(3);
            load(0, 0);
            __syncthreads();
        }
        int cur = 0, nxt = 1, bld = 2;
        for (int ch = 0; ch < chunks; ++ch) {
            load(cur, 1);
            multiply(0);
            build(ch & 1, bld, dg);  // chunk ch + 2
            digits(ch + 3, dg);
            load(nxt, 0);
            multiply(1);
            sh.bits[(ch & 1) ^ 1][myh][my][lane] = transpose(next);  // chunk ch + 3
            next = fetch(ch + 4);
            const int t = cur;
            cur = nxt;
            nxt = bld;
            bld = t;
            __syncthreads();
        }
        // register r of a 32 x 32 accumulator: row 8 (r / 4) + 4 (lane / 32) + r mod 4, column lane mod 32
        const int64_t col = tj * Tile::kN + wc * 32 + li;
        const double unit = ldexp(1.0, q);
        for (int i = tid; i < Tile::kM * kExDigits; i += Tile::kThreads) (&sh.rows[0][0])[i] = 0;
        __syncthreads();
#pragma unroll
        for (int g = 0; g < ND; ++g) atomicAdd(&sh.rows[iw * kWave + lane][g], usum[g]);  // (whole numbers: any order)
        __syncthreads();
        const int rl = wr * AR * 32 + 4 * kh;
        int64_t row_i = ti * Tile::kM + rl;
        float* po = out + row_i * n + col;
        const int(*rows)[kExDigits] = &sh.rows[rl];
        if (col < n) {
#pragma unroll
            for (int a = 0; a < AR; ++a)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int off = a * 32 + 8 * (r >> 2) + (r & 3);
                    // (one at a time: twice the sum passes 32 bits from 2^23 terms on, both differences never do)
                    double v = (double)(rows[off][ND - 1] - acc[a][ND - 1][r] - acc[a][ND - 1][r]);
#pragma unroll
                    for (int g = ND - 2; g >= 0; --g) v = v * 255.0 + (double)(rows[off][g] - acc[a][g][r] - acc[a][g][r]);
                    if (row_i + off < m) *po = (float)(v * unit);
                    po += (r & 3) == 3 ? 5 * n : n;
                    if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // (no room for more entries at a time)
                }
        }
    }
}

template <int RW, int CW>
__global__ void __launch_bounds__((ExTile<RW, CW>::kThreads), 2)
    expand_int_kernel(const uint64_t* __restrict__ S, const uint64_t* __restrict__ T, const float* __restrict__ c,
                      const ExPlan* __restrict__ plan, const uint32_t* __restrict__ dig, int64_t m, int64_t n, int64_t w, float* __restrict__ out)
{
    typedef ExTile<RW, CW> Tile;
    extern __shared__ __align__(16) unsigned char ex_lds[];
    auto& sh = *(typename Tile::Lds*)ex_lds;
    static_assert(sizeof(sh) >= sizeof(ExF64Lds) * Tile::kThreads / kExThreads, "the f64 form fits");
    if (!plan->ok) ex_f64_tiles<float, Tile::kThreads / kExThreads>(S, T, c, m, n, w, out, (ExF64Lds*)ex_lds);
    else if (plan->digits == 4) ex_int_tiles<RW, CW, 4>(S, T, dig, m, n, w, out, plan->q, sh);
    else ex_int_tiles<RW, CW, 5>(S, T, dig, m, n, w, out, plan->q, sh);
}

// f32 coefficients: most terms that go to the f64 form at once, by the number of entries, and to the int8 form in one launch.
// Us a call, f64 form / one launch: 64x64 to 48 terms 16.9 / 17.0, to 64 17.9 / 16.9; 1024x1024 to 48 18.1 / 18.2, to 64
// 19.1 / 18.2; 2048x2048 to 24 19.8 / 20.8, to 32 20.8 / 20.8, to 40 21.8 / 20.8; 4096x4096 to 20 34.0 / 34.2, to 24 34.5 / 34.1;
// 14336x4096 to 17 73.4 / 77.0, to 20 77.3 / 77.0.
// One launch / staged operands: 64x64 to 384 terms 21.2 / 21.8; 1024x1024 to 384 22.9 / 24.0, to 700 28.7 / 28.7; 2048x2048 to 33
// 20.2 / 25.4, to 384 26.9 / 29.5; 4096x4096 to 33 33.0 / 46.7, to 384 57.9 / 61.2, to 450 71.5 / 68.0; 14336x4096 to 33
// 74 / 114, to 384 164 / 164, to 450 208 / 186 (one launch takes another step at each 64 terms, the staged form at each 128).
int64_t ex_few_terms(int64_t m, int64_t n)
{
    const double entries = (double)m * (double)n;
    return entries <= (double)(1 << 20) ? 48 : (entries <= (double)(1 << 22) ? 32 : 20);
}
constexpr int64_t kExDirectTerms = 448;

unsigned ex_grid(int64_t tiles, int64_t cap) { return (unsigned)(tiles < 1 ? 1 : (tiles < cap ? tiles : cap)); }

}  // namespace

size_t expand_scratch_bytes(scd_dtype dt, int64_t w)
{
    if (dt != SCD_F32 || w <= kExDirectTerms) return 0;
    return sizeof(ExPlan) + ((size_t)((w + 127) / 128) * 2 + 1) * kExChunkDwords * 4;
}

template <int RW, int CW>
static hipError_t launch_int(const uint64_t* S, const uint64_t* T, const float* c, const ExPlan* plan, const uint32_t* dig, int64_t m, int64_t n, int64_t w,
                             float* out, hipStream_t st)
{
    typedef ExTile<RW, CW> Tile;
    const size_t lds = sizeof(typename Tile::Lds);
    const hipError_t e = hipFuncSetAttribute((const void*)expand_int_kernel<RW, CW>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int64_t tiles = ((m + Tile::kM - 1) / Tile::kM) * ((n + Tile::kN - 1) / Tile::kN);
    hipLaunchKernelGGL((expand_int_kernel<RW, CW>), dim3(ex_grid(tiles, RW == 2 ? 256 : 768)), dim3(Tile::kThreads), lds, st, S, T, c, plan, dig, m,
                       n, w, out);
    return hipGetLastError();
}

// scratch: expand_scratch_bytes, 16-byte aligned; null: everything takes the f64 form.
hipError_t launch_expand(const uint64_t* S, const uint64_t* T, const void* c, scd_dtype dt, int64_t m, int64_t n, int64_t w, void* out,
                         void* scratch, hipStream_t st)
{
    const int64_t mw = (m + 63) / 64, nw = (n + 63) / 64;
    // Measured, us a call, one launch in which every workgroup works out the digits / staged operands: 1024x4096 to 6512 terms
    // 167 / 123, 2048x2048 to 5900 180 / 136, 4096x4096 to 1500 200 / 165, 1024x1024 to 3000 80 / 63, 300x500 to 1400
    // 51 / 43, 64x64 to 700 27 / 26; with fewer terms the ends of the tiles, which a workgroup that fills its compute unit does not
    // overlap, and the second launch weigh more (see ex_few_terms).
    const unsigned gridf = ex_grid(mw * ((nw + 1) / 2), 1024);
    if (dt == SCD_F64) {
        hipLaunchKernelGGL((expand_f64_kernel<double>), dim3(gridf), dim3(kExThreads), 0, st, S, T, (const double*)c, m, n, w,
                           (double*)out);
    } else if (w > ex_few_terms(m, n) && w <= kExDirectTerms) {
        const int64_t tiles = (m + kExDirectM - 1) / kExDirectM * nw;
        hipLaunchKernelGGL(expand_direct_kernel, dim3(ex_grid(tiles, 512)), dim3(kExThreads), 0, st, S, T, (const float*)c, m, n, w,
                           (float*)out);
    } else if (w <= kExDirectTerms || !scratch || mw >= 1 << 29 || nw >= 1 << 29) {  // (rows of bits of 4 GiB and more: 32-bit strides)
        hipLaunchKernelGGL((expand_f64_kernel<float>), dim3(gridf), dim3(kExThreads), 0, st, S, T, (const float*)c, m, n, w,
                           (float*)out);
    } else {
        ExPlan* plan = (ExPlan*)scratch;
        uint32_t* dig = (uint32_t*)(plan + 1);
        hipLaunchKernelGGL(expand_digits_kernel, dim3(ex_grid((w + 1023) / 1024, 64)), dim3(kExScanThreads), 0, st, (const float*)c, w, plan, dig);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) {
            // 128 x 128 tiles read each operand byte from LDS for twice the products of 64 x 64 ones, but want some 128 of
            // them (us a call with 64 x 64 / 128 x 128: 1024x1024 to 3000 terms 64 / 75, 1920x1024 72 / 78, 1024x2048 to 4000
            // 86 / 92, 1536x1536 to 3000 97 / 79, 2048x2048 to 5900 200 / 136)
            if ((m + 127) / 128 * ((n + 127) / 128) > 128) e = launch_int<2, 2>(S, T, (const float*)c, plan, dig, m, n, w, (float*)out, st);
            else e = launch_int<1, 1>(S, T, (const float*)c, plan, dig, m, n, w, (float*)out, st);
        }
        return e;
    }
    return hipGetLastError();
}

}  // namespace scd
