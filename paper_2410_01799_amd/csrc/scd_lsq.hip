// Least squares decomposition (Algorithm 6, Section 3.3 of arXiv 2410.01799): after every greedy signed
// cut the coefficients of ALL terms are refitted, c = argmin ||A - S diag(c) T^T||_F.
//
// The remainder R_k = A - S_k diag(c_k) T_k^T is never kept: every coefficient changes with every term.  The
// register-resident engine forms it anew for each cut (scd_resident_lsq.hip).  The sweeps and the host loop below leave it
// implicit; each half step of their cut works on
//     R t   = A t   - S (c o (T^T t)),        R^T s = A^T s - T (c o (S^T s)),
// where A t and A^T s are the ordinary signed-sum passes over A, <t_j, t> = n - 2 popcount(t_j xor t)
// comes from the bitsets, and the correction is a signed sum of k scalars per entry.  The normal equations
// (Section 3.3) use the Gram matrix G_ij = <s_i,s_j><t_i,t_j>, again from popcounts, kept as a Cholesky
// factor that grows by one row per term; b_j = <s_j, A t_j> falls out of the last half step of term j, or comes from the
// cut value and the Gram row where the remainder was formed.
// Everything here is f64; the kernels are small and latency-bound.  Matrices whose f64 remainder fits the register files
// (up to 4096x2048 or 2048x4096): two launches per term, the cut on the register-resident engine (scd_resident_lsq.hip)
// and lsq_term_kernel.  Others of up to 64 words a side, and those for which the engine has no compute units or is slower: three
// launches per sweep and no host in the loop; larger ones, and tensors: about ten and a read-back.
#include "scd_device.h"
#include "scd_rng.h"

namespace scd {

namespace {

__device__ __forceinline__ double lq_wave_sum(double a)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, kWave);
    return a;
}

// out[j] = coef[j] * <x_j, vec> for sign vectors given as bitsets of `len` entries (coef null: 1);
// one wave per term.  Padding bits are zero on both sides.
__global__ void __launch_bounds__(256)
    lsq_dots_kernel(const uint64_t* __restrict__ bits, int64_t k, int64_t nw, int64_t len, const uint64_t* __restrict__ vec,
                    const double* __restrict__ coef, double* __restrict__ out)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t j = (int64_t)blockIdx.x * 4 + threadIdx.x / kWave;
    if (j >= k) return;
    int cnt = 0;
    for (int64_t p = lane; p < nw; p += kWave) cnt += __popcll(bits[j * nw + p] ^ vec[p]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, kWave);
    if (lane == 0) {
        const double d = (double)(len - 2 * (int64_t)cnt);
        out[j] = coef ? coef[j] * d : d;
    }
}

// y_i = base_i - sum_{j<k} e_j x_j[i] for the 64 entries of word p = blockIdx.x (lane = entry); the eight
// waves take the terms j = wave, wave + 8, ... and their partial sums are joined in wave order.
// Writes sgn(y) as a word of bits, optionally y, and per word sum |y_i| and sum sgn(y_i) base_i.
__global__ void __launch_bounds__(512)
    lsq_correct_kernel(const uint64_t* __restrict__ bits, int64_t k, int64_t mw, int64_t m, const double* __restrict__ e,
                       const double* __restrict__ base, uint64_t* __restrict__ out_bits, double* __restrict__ abs_parts,
                       double* __restrict__ dot_parts)
{
    __shared__ double part[8][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t p = blockIdx.x;
    double acc = 0.0;
    for (int64_t j = wv; j < k; j += 8) {
        const uint64_t word = bits[j * mw + p];  // the same for all lanes
        const double sgn = __hiloint2double(((word >> lane) & 1ull) ? (int)0xBFF00000 : (int)0x3FF00000, 0);
        acc = __builtin_fma(e[j], sgn, acc);
    }
    part[wv][lane] = acc;
    __syncthreads();
    if (wv != 0) return;
    double tot = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) tot += part[q][lane];
    const int64_t i = p * 64 + lane;
    const bool valid = i < m;
    const double b = valid ? base[i] : 0.0;
    const double y = valid ? b - tot : 0.0;
    const bool neg = y < 0.0;
    const uint64_t bal = __ballot(valid && neg);
    if (lane == 0) out_bits[p] = bal;
    if (abs_parts) {
        const double a = lq_wave_sum(fabs(y));
        const double d = lq_wave_sum(neg ? -b : b);
        if (lane == 0) {
            abs_parts[p] = a;
            dot_parts[p] = d;
        }
    }
}

// out[0] = sum a, out[1] = sum b (b may be null), n values each, in a fixed order (one workgroup)
__global__ void __launch_bounds__(256) lsq_sum2_kernel(const double* __restrict__ a, const double* __restrict__ b, int64_t n,
                                                      double* __restrict__ out)
{
    __shared__ double ra[256], rb[256];
    double sa = 0.0, sb = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        sa += a[i];
        if (b) sb += b[i];
    }
    ra[threadIdx.x] = sa;
    rb[threadIdx.x] = sb;
    __syncthreads();
    if (threadIdx.x == 0) {
        double ta = 0.0, tb = 0.0;
        for (int q = 0; q < 256; ++q) {
            ta += ra[q];
            tb += rb[q];
        }
        out[0] = ta;
        out[1] = tb;
    }
}

template <typename TE>
__global__ void __launch_bounds__(256) lsq_sumsq_kernel(const TE* __restrict__ A, int64_t total, double* __restrict__ parts)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const double v = (double)A[i];
        s += v * v;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int q = 0; q < 256; ++q) t += red[q];
        parts[blockIdx.x] = t;
    }
}

template <typename TE>
__global__ void __launch_bounds__(256) lsq_cast_kernel(const double* __restrict__ c, int64_t k, TE* __restrict__ out)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j < k) out[j] = (TE)c[j];
}

// out[j] = (coef ? coef[j] : 1) * product over the modes m != skip of D[m * ld + j]   (skip < 0: all modes)
__global__ void __launch_bounds__(256) lsq_prod_kernel(const double* __restrict__ D, int64_t ld, int order, int skip, int64_t k,
                                                      const double* __restrict__ coef, double* __restrict__ out)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= k) return;
    double p = coef ? coef[j] : 1.0;
    for (int m = 0; m < order; ++m)
        if (m != skip) p *= D[(int64_t)m * ld + j];
    out[j] = p;
}

// Sign bits of the tensor product of the sign vectors of modes first..last-1 (last mode fastest): bit q is
// the xor of the modes' bits at the multi-index of q (Algorithm 12 lines 5-7).  One lane per entry.
struct LsqKronArgs {
    const uint64_t* signs[SCD_MAX_ORDER];
    int64_t dims[SCD_MAX_ORDER];
    int first, last;
    int64_t len;
    uint64_t* out;
};

__global__ void __launch_bounds__(256) lsq_kron_kernel(LsqKronArgs a)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    unsigned bit = 0;
    if (q < a.len) {
        int64_t rest = q;
        for (int m = a.last - 1; m >= a.first; --m) {
            const int64_t i = rest % a.dims[m];
            rest /= a.dims[m];
            bit ^= (unsigned)((a.signs[m][i >> 6] >> (i & 63)) & 1ull);
        }
    }
    const uint64_t word = __ballot(q < a.len && bit);
    if ((threadIdx.x & (kWave - 1)) == 0 && (q >> 6) < (a.len + 63) / 64) a.out[q >> 6] = word;
}

// Real last mode: c[ch] = u[ch] / P, rounded to the element type (the stored value is what gets subtracted).
template <typename TE>
__global__ void __launch_bounds__(256) scalars_coef_kernel(const double* __restrict__ u, int64_t q, double P, TE* __restrict__ c)
{
    const int64_t ch = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (ch < q) c[ch] = (TE)(u[ch] / P);
}

// r[p][ch] -= sign_p * c[ch] over the whole tensor (p = index over the leading modes, sign_p = bit p of
// `lead`, a 1 bit standing for -1), and the sum of the squares of what is left, per workgroup.
template <typename TE>
__global__ void __launch_bounds__(256) scalars_update_kernel(TE* __restrict__ r, int64_t total, int64_t q,
                                                            const uint64_t* __restrict__ lead, const TE* __restrict__ c,
                                                            double* __restrict__ parts)
{
    __shared__ double red[256];
    double s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int64_t p = i / q, ch = i - p * q;
        const TE d = ((lead[p >> 6] >> (p & 63)) & 1ull) ? -c[ch] : c[ch];
        const TE v = r[i] - d;
        r[i] = v;
        s += (double)v * (double)v;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int z = 0; z < 256; ++z) t += red[z];
        parts[blockIdx.x] = t;
    }
}

constexpr int kLqThreads = 1024;

// sum over the workgroup in a fixed order; every thread gets the same bits
__device__ double lq_block_sum(double v, double* red)
{
    const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    v = lq_wave_sum(v);
    __syncthreads();  // red may still be read from the previous call
    if (lane == 0) red[wv] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < kLqThreads / kWave; ++q) t += red[q];
    return t;
}

// The new term has index k.  Appends row k to the Cholesky factor L (lower triangular, row-major, leading
// dimension ld) of the Gram matrix, whose new row is g[j] (j < k) with `diag` on the diagonal;
// extends the forward solution y of L y = b by one entry; solves L^T c = y for all k + 1 coefficients.
// False if the new term is (numerically) in the span of the old ones; else *cb = <c, b>; the same in every thread.
// One workgroup.  Both substitutions are in axpy form: a thread keeps up to four unknowns in registers, the owner of
// the next one divides and hands it on through LDS, one barrier per unknown, and the column (row) of L that the next
// step needs is loaded ahead of the barrier.  (With a sum over the workgroup per unknown, forward substitution alone
// took 0.7 us per unknown.)
__device__ bool lq_refit(double* __restrict__ L, int64_t ld, int64_t k, const double* g, double diag, const double* __restrict__ bvec,
                           double* __restrict__ yv, double* __restrict__ c, double* red, double* hand, double* cb_out)
{
    constexpr int NQ = SCD_LSQ_MAX_WIDTH / kLqThreads;
    const int tid = threadIdx.x;
    double* row = L + k * ld;
    double x[NQ], col[NQ];
    // ---- forward substitution L row = g
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int64_t q = tid + (int64_t)i * kLqThreads;
        x[i] = q < k ? g[q] : 0.0;
        col[i] = q < k ? L[q * ld] : 0.0;
    }
    for (int64_t r = 0; r < k; ++r) {
        double cur[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int64_t q = tid + (int64_t)i * kLqThreads;
            cur[i] = col[i];
            if (q == r) hand[r & 1] = x[i] = x[i] / cur[i];
            col[i] = q < k && q > r ? L[q * ld + r + 1] : 0.0;  // (q > r: column r + 1 of the rows from r + 1 on)
        }
        __syncthreads();
        const double xr = hand[r & 1];
#pragma unroll
        for (int i = 0; i < NQ; ++i)
            if (tid + (int64_t)i * kLqThreads > r) x[i] -= cur[i] * xr;
    }
    double s2 = 0.0, sy = 0.0;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int64_t q = tid + (int64_t)i * kLqThreads;
        if (q < k) {
            row[q] = x[i];
            s2 += x[i] * x[i];
            sy += x[i] * yv[q];
        }
    }
    s2 = lq_block_sum(s2, red);
    sy = lq_block_sum(sy, red);
    const double d2 = diag - s2;
    if (!(d2 > 1e-9 * diag)) return false;
    const double lkk = sqrt(d2), yk = (bvec[k] - sy) / lkk;
    if (tid == 0) {
        row[k] = lkk;
        yv[k] = yk;
    }
    // ---- back substitution L^T c = y: rows of L are contiguous.  Row k is this launch's own: from the registers.
    double cb = 0.0;
    const double ck = yk / lkk;
    double nxt[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int64_t q = tid + (int64_t)i * kLqThreads;
        const double lkq = x[i];
        x[i] = q < k ? yv[q] - lkq * ck : (q == k ? ck : 0.0);
        nxt[i] = q < k ? L[(k - 1) * ld + q] : 0.0;
        if (q == k) {
            c[q] = ck;
            cb += ck * bvec[q];
        }
    }
    __syncthreads();  // hand is free again
    for (int64_t r = k - 1; r >= 0; --r) {
        double cur[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int64_t q = tid + (int64_t)i * kLqThreads;
            cur[i] = nxt[i];
            if (q == r) {
                hand[r & 1] = x[i] = x[i] / cur[i];
                c[q] = x[i];
                cb += x[i] * bvec[q];
            }
            nxt[i] = q < r ? L[(r - 1) * ld + q] : 0.0;
        }
        __syncthreads();
        const double cr = hand[r & 1];
#pragma unroll
        for (int i = 0; i < NQ; ++i)
            if (tid + (int64_t)i * kLqThreads < r) x[i] -= cur[i] * cr;
    }
    *cb_out = lq_block_sum(cb, red);
    return true;
}

// One workgroup: refit after the new term k and record ||A - S diag(c) T^T||_F = sqrt(||A||^2 - <c, b>) (the remainder
// is orthogonal to the fit).  status: 1 if the new term is (numerically) in the span of the old ones.
__global__ void __launch_bounds__(kLqThreads)
    lsq_solve_kernel(double* __restrict__ L, int64_t ld, int64_t k, const double* __restrict__ g, double diag, const double* __restrict__ bvec, double* __restrict__ yv, double* __restrict__ c,
                     double fro0sq, double* __restrict__ trace_out, int* __restrict__ status)
{
    __shared__ double red[kLqThreads / kWave];
    __shared__ double hand[2];
    double cb = 0.0;
    const bool ok = lq_refit(L, ld, k, g, diag, bvec, yv, c, red, hand, &cb);
    if (threadIdx.x == 0) {
        const double f2 = fro0sq - cb;
        if (!ok) *status = 1;
        else trace_out[0] = sqrt(f2 > 0.0 ? f2 : 0.0);
    }
}

// =================================================================================================
// Matrices of up to kLqMaxWords words a side, where the register-resident engine does not take the cut: a sweep (both half
// steps of Algorithm 4 on the implicit remainder, the stop test and, at the end of a term, the refit) is three launches that the host enqueues blindly, many sweeps
// ahead; the position of the loop lives on the device.  A half step is one launch because a workgroup owns one word (64 rows
// or columns) from the entries of A to the sign bits: it forms the inner products with the earlier terms, the f64 sums
// over its strip of A, the correction and the signs.  Bound by the chain of memory trips, barriers and launches, not by
// bytes.  Us per sweep with ten launches and a read-back, and now: 1024x1024 f32 57 / 17.5, 64x64 57 / 15.5, 4096x4096
// 71 / 41, 2048x2048 f64 60 / 35.  (The sweep's end in the workgroup of the column step that comes last needs fences
// that write back and invalidate the caches: 20 instead of 17.5.)
constexpr int kLqMaxWords = 64;
constexpr int kLqWaves = kLqThreads / kWave;

template <typename TE>
struct LqVec;
template <>
struct LqVec<float> {
    typedef float4 type;
    static constexpr int N = 4;
};
template <>
struct LqVec<double> {
    typedef double2 type;
    static constexpr int N = 2;
};
__device__ __forceinline__ double lq_sign(uint32_t bit) { return __hiloint2double((int)(0x3FF00000u | (bit << 31)), 0); }

// The entries of one 16-byte chunk (or one entry) as doubles.
template <typename TE, bool VEC>
__device__ __forceinline__ void lq_load(const TE* __restrict__ p, double (&x)[VEC ? LqVec<TE>::N : 1])
{
    if constexpr (!VEC) {
        x[0] = (double)p[0];
    } else {
        const typename LqVec<TE>::type v = *(const typename LqVec<TE>::type*)p;
        x[0] = (double)v.x;
        x[1] = (double)v.y;
        if constexpr (LqVec<TE>::N == 4) x[2] = (double)v.z, x[3] = (double)v.w;
    }
}

struct LqShared {
    uint64_t vec[kLqMaxWords];       // the other side's sign vector
    double e[SCD_LSQ_MAX_WIDTH];     // coefficient times inner product, per earlier term
    double part[kLqWaves][kWave];
    double sums[kWave];              // the strip's entries of A t or A^T s
    double red[kLqWaves];
    int flag;
};

// out[j] = coef[j] * <x_j, vec> (coef null: 1; it may be out) for j < k: a group of 2^g >= nw lanes per term.  No barrier
// at the end.
__device__ void lq_dots(const uint64_t* __restrict__ bits, int64_t k, int nw, int64_t len, const uint64_t* vec, const double* coef,
                        double* out)
{
    int g = 1;
    while (g < nw) g <<= 1;  // at most 64
    const int p = threadIdx.x & (g - 1), per = kLqThreads / g;
    const uint64_t mine = p < nw ? vec[p] : 0;
    for (int64_t j0 = 0; j0 < k; j0 += per) {  // (whole waves stay together for the lane exchanges)
        const int64_t j = j0 + threadIdx.x / g;
        int cnt = (j < k && p < nw) ? __popcll(bits[j * nw + p] ^ mine) : 0;
        for (int off = g >> 1; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, kWave);
        if (j < k && p == 0) {
            const double d = (double)(len - 2 * (int64_t)cnt);
            out[j] = coef ? coef[j] * d : d;
        }
    }
}

// The correction, the signs and (COLS) the sums of |y| and sgn(y) base for word p of `bits` (kw words per term), the
// strip's sums in sh.sums and the weights in sh.e.
template <bool COLS>
__device__ void lq_finish(const uint64_t* __restrict__ bits, int64_t k, int64_t kw, int64_t p, int64_t len, LqShared& sh,
                          uint64_t* __restrict__ out_bits, double* __restrict__ abs_parts, double* __restrict__ dot_parts)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    double acc = 0.0;
    for (int64_t j0 = wv; j0 < k; j0 += 4 * kLqWaves) {
        uint64_t word[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) word[i] = bits[(j0 + i * kLqWaves < k ? j0 + i * kLqWaves : j0) * kw + p];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (j0 + i * kLqWaves < k) acc = __builtin_fma(sh.e[j0 + i * kLqWaves], lq_sign((uint32_t)(word[i] >> lane) & 1u), acc);
    }
    sh.part[wv][lane] = acc;
    __syncthreads();
    if (wv != 0) return;
    double q[kLqWaves], tot = 0.0;
#pragma unroll
    for (int i = 0; i < kLqWaves; ++i) q[i] = sh.part[i][lane];
#pragma unroll
    for (int i = 0; i < kLqWaves; ++i) tot += q[i];
    const bool valid = p * 64 + lane < len;
    const double b = valid ? sh.sums[lane] : 0.0;
    const double y = valid ? b - tot : 0.0;
    const bool neg = y < 0.0;
    const uint64_t bal = __ballot(valid && neg);
    if (lane == 0) out_bits[p] = bal;
    if constexpr (COLS) {
        const double a = lq_wave_sum(fabs(y));
        const double d = lq_wave_sum(neg ? -b : b);
        if (lane == 0) {
            abs_parts[p] = a;
            dot_parts[p] = d;
        }
    }
}

// s = sgn(A t - S (c o T^T t)), 64 rows per workgroup, four per wave
template <typename TE, bool VEC>
__global__ void __launch_bounds__(kLqThreads) lsq_rows_kernel(LsqMatArgs a)
{
    __shared__ LqShared sh;
    constexpr int VE = VEC ? LqVec<TE>::N : 1;
    if (a.st->done) return;
    const int64_t k = a.st->k;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int mw = (int)((a.m + 63) / 64), nw = (int)((a.n + 63) / 64);
    if (tid < nw) sh.vec[tid] = a.t[tid];
    __syncthreads();
    lq_dots(a.T, k, nw, a.n, sh.vec, a.c, sh.e);
    const TE* A = (const TE*)a.A;
    const TE* rowp[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t row = (int64_t)blockIdx.x * 64 + wv * 4 + r;
        rowp[r] = A + (row < a.m ? row : a.m - 1) * a.n;
    }
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const int nch = (int)(a.n / VE);
#pragma unroll 2
    for (int ch = lane; ch < nch; ch += kWave) {
        double x[4][VE];
#pragma unroll
        for (int r = 0; r < 4; ++r) lq_load<TE, VEC>(rowp[r] + (int64_t)ch * VE, x[r]);
        const uint32_t b = (uint32_t)(sh.vec[(ch * VE) >> 6] >> ((ch * VE) & 63));
#pragma unroll
        for (int e = 0; e < VE; ++e) {
            const double sg = lq_sign((b >> e) & 1u);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = __builtin_fma(x[r][e], sg, acc[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double u = lq_wave_sum(acc[r]);
        if (lane == 0) sh.sums[wv * 4 + r] = u;
    }
    __syncthreads();
    lq_finish<false>(a.S, k, mw, blockIdx.x, a.m, sh, a.s, nullptr, nullptr);
}

// t = sgn(A^T s - T (c o S^T s)), 64 columns per workgroup: 64 / VE lanes share a row, the waves take rows in turn
template <typename TE, bool VEC>
__global__ void __launch_bounds__(kLqThreads) lsq_cols_kernel(LsqMatArgs a)
{
    __shared__ LqShared sh;
    constexpr int VE = VEC ? LqVec<TE>::N : 1;
    constexpr int RG = VE;  // rows per load of a wave
    if (a.st->done) return;
    const int64_t k = a.st->k;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int mw = (int)((a.m + 63) / 64), nw = (int)((a.n + 63) / 64);
    if (tid < mw) sh.vec[tid] = a.s[tid];
    __syncthreads();
    lq_dots(a.S, k, mw, a.m, sh.vec, a.c, sh.e);
    const int cl = lane % (kWave / VE), rg = lane / (kWave / VE);
    const int64_t col = (int64_t)blockIdx.x * 64 + cl * VE;
    const TE* colp = (const TE*)a.A + (col < a.n ? col : 0);  // (columns past the end are dropped below)
    double acc[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) acc[e] = 0.0;
    const int m = (int)a.m;
#pragma unroll 4
    for (int row = wv * RG + rg; row < m; row += kLqWaves * RG) {
        double x[VE];
        lq_load<TE, VEC>(colp + (int64_t)row * a.n, x);
        const double sg = lq_sign((uint32_t)(sh.vec[row >> 6] >> (row & 63)) & 1u);
#pragma unroll
        for (int e = 0; e < VE; ++e) acc[e] = __builtin_fma(x[e], sg, acc[e]);
    }
#pragma unroll
    for (int e = 0; e < VE; ++e) {
        if constexpr (RG >= 4) acc[e] += __shfl_xor(acc[e], 16, kWave);
        if constexpr (RG >= 2) acc[e] += __shfl_xor(acc[e], 32, kWave);
        if (rg == 0) sh.part[wv][cl * VE + e] = acc[e];
    }
    __syncthreads();
    if (wv == 0) {
        double q[kLqWaves], v = 0.0;
#pragma unroll
        for (int i = 0; i < kLqWaves; ++i) q[i] = sh.part[i][lane];
#pragma unroll
        for (int i = 0; i < kLqWaves; ++i) v += q[i];
        sh.sums[lane] = v;
    }
    __syncthreads();
    lq_finish<true>(a.T, k, nw, blockIdx.x, a.n, sh, a.t, a.abs_parts, a.dot_parts);
}

// End of a sweep: Algorithm 4 line 8; when the term is complete, append it, refit all coefficients (Section 3.3) and draw
// the next start.  One workgroup.
__global__ void __launch_bounds__(kLqThreads) lsq_next_kernel(LsqMatArgs a)
{
    __shared__ LqShared sh;
    LsqState* st = a.st;
    if (st->done) return;
    const int64_t k = st->k;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int mw = (int)((a.m + 63) / 64), nw = (int)((a.n + 63) / 64);
    if (wv == 0) {
        const double cut = lq_wave_sum(lane < nw ? a.abs_parts[lane] : 0.0);
        const double b = lq_wave_sum(lane < nw ? a.dot_parts[lane] : 0.0);
        if (lane == 0) {
            const int j = st->j + 1;
            int conv = 0;
            if (!(fabs(cut) < INFINITY)) {
                st->status = 2;
                st->done = 1;
            } else if (cut <= st->c_prev || j >= a.max_iters) {
                if (!(cut <= st->c_prev)) st->warn = 1;
                conv = 1;
                a.bvec[k] = b;
                a.iters[k] = j;
            } else {
                st->c_prev = cut;
                st->j = j;
            }
            sh.flag = conv;
        }
    }
    if (tid < nw) sh.vec[tid] = a.t[tid];
    __syncthreads();
    if (!sh.flag) return;
    // the Gram row of the new term: products of the two sides' inner products
    lq_dots(a.T, k, nw, a.n, sh.vec, nullptr, sh.e);
    __syncthreads();
    if (tid < nw) a.T[k * nw + tid] = sh.vec[tid];
    __syncthreads();
    if (tid < mw) {
        sh.vec[tid] = a.s[tid];
        a.S[k * mw + tid] = sh.vec[tid];
    }
    __syncthreads();
    lq_dots(a.S, k, mw, a.m, sh.vec, sh.e, sh.e);  // (each element is read and written by the same lane)
    __syncthreads();
    double cb = 0.0;
    if (!lq_refit(a.L, a.w, k, sh.e, (double)a.m * (double)a.n, a.bvec, a.yv, a.c, sh.red, &sh.part[0][0], &cb)) {
        if (tid == 0) {
            st->status = 1;
            st->done = 1;
        }
        return;
    }
    if (tid == 0) {
        const double f2 = a.fro0sq - cb;
        a.trace[k + 1] = sqrt(f2 > 0.0 ? f2 : 0.0);
        st->k = k + 1;
        st->total += a.iters[k];
        st->j = 0;
        st->c_prev = -INFINITY;
        if (k + 1 >= a.w) st->done = 1;
    }
    if (tid < nw) a.t[tid] = rng_word_masked(a.seed, (uint64_t)k + 1, 1u, tid, a.n);
}

// Few terms: the refit of lq_refit by one wave that holds two unknowns a lane, with the factor in LDS: no barrier and no trip
// to memory per unknown.  Both substitutions are those of lq_refit step for step; the sums over the unknowns (the
// squares, <row, y>, <c, b>) are added in another order.
constexpr int kLqSmall = 88;  // most terms before the new one; their factor's triangle takes 31 KB
static_assert(kLqSmall <= 2 * kWave && kLqSmall <= 6 * kLqWaves, "unknowns of a lane, terms of a wave");
struct LqSmallShared {
    double e[kLqSmall];                           // Gram row of the new term
    double L[kLqSmall * (kLqSmall + 1) / 2];      // rows of the factor, packed
};
__device__ __forceinline__ double lq_lane(double v, int l)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l), hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}
// Wave 0.  yv, bvec: the lane's entries; b: of the new term.
__device__ bool lq_refit_small(const LqSmallShared& sm, double* __restrict__ L, int64_t ld, int k, double diag, double b, const double (&yl)[2],
                               const double (&bl)[2], double* __restrict__ yv, double* __restrict__ c, double* cb_out)
{
    const int lane = threadIdx.x & (kWave - 1);
    double x[2], d[2], col[2];
    int at[2];  // of the lane's rows
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int q = lane + i * kWave;
        at[i] = q * (q + 1) / 2;
        x[i] = q < k ? sm.e[q] : 0.0;
        d[i] = q < k ? sm.L[at[i] + q] : 1.0;
        col[i] = q < k ? sm.L[at[i]] : 0.0;
    }
    // ---- forward substitution L row = g
    for (int r = 0; r < k; ++r) {
        const int i0 = r >> 6;
        const double xr = lq_lane(i0 ? x[1] / d[1] : x[0] / d[0], r & 63);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = lane + i * kWave;
            const double cur = col[i];
            col[i] = q < k && q > r ? sm.L[at[i] + r + 1] : 0.0;
            x[i] = q > r ? __builtin_fma(-cur, xr, x[i]) : (q == r ? xr : x[i]);
        }
    }
    double s2 = 0.0, sy = 0.0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int q = lane + i * kWave;
        if (q < k) L[k * ld + q] = x[i];
        s2 += lq_wave_sum(q < k ? x[i] * x[i] : 0.0);
        sy += lq_wave_sum(q < k ? x[i] * yl[i] : 0.0);
    }
    const double d2 = diag - s2;
    if (!(d2 > 1e-9 * diag)) return false;
    const double lkk = sqrt(d2), yk = (b - sy) / lkk;
    // ---- back substitution L^T c = y
    const double ck = yk / lkk;
    double cb = 0.0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int q = lane + i * kWave;
        x[i] = q < k ? __builtin_fma(-x[i], ck, yl[i]) : 0.0;
        col[i] = q < k ? sm.L[(k - 1) * k / 2 + q] : 0.0;
    }
    for (int r = k - 1; r >= 0; --r) {
        const int i0 = r >> 6;
        const double xr = lq_lane(i0 ? x[1] / d[1] : x[0] / d[0], r & 63);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int q = lane + i * kWave;
            const double cur = col[i];
            col[i] = q < r ? sm.L[(r - 1) * r / 2 + q] : 0.0;
            x[i] = q < r ? __builtin_fma(-cur, xr, x[i]) : (q == r ? xr : x[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int q = lane + i * kWave;
        if (q < k) c[q] = x[i];
        cb += lq_wave_sum(q < k ? x[i] * bl[i] : 0.0);
    }
    if (lane == 0) {
        L[k * ld + k] = lkk;
        yv[k] = yk;
        c[k] = ck;
    }
    *cb_out = cb + ck * b;
    return true;
}

// End of a term whose cut the register-resident engine has found (its sign vectors are rows k of S and T, its cut value
// <s, R t> in the state): refit of all coefficients.  With the remainder R = A - sum c_j s_j t_j^T,
// <s_k, A t_k> = <s_k, R t_k> + sum_j c_j <s_j, s_k> <t_j, t_k>.  One workgroup, bound by its trips to memory and the chain
// of the two substitutions: with few terms everything is requested at once and one wave substitutes
// (1024x1024, mean over the first 32 terms: 12.6 us, with lq_dots and lq_refit 22.3).
__global__ void __launch_bounds__(kLqThreads) lsq_term_kernel(LsqMatArgs a, const ResidentResult* __restrict__ res)
{
    __shared__ union {
        LqShared sh;
        LqSmallShared sm;
    } u;
    LqShared& sh = u.sh;
    LsqState* st = a.st;
    if (st->done) return;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int64_t k = st->k;
    const double cut = st->c_prev;
    const bool gave_up = res->err != 0;
    if (gave_up || !(fabs(cut) < INFINITY)) {
        __syncthreads();  // (all waves have read the state)
        if (tid == 0) {
            st->status = gave_up ? 3 : 2;
            st->done = 1;
        }
        return;
    }
    const int mw = (int)((a.m + 63) / 64), nw = (int)((a.n + 63) / 64);
    double cb = 0.0;
    bool ok;
    if (k <= kLqSmall) {
        // a wave takes terms wv, wv + 16, .. : their inner products with the new one and their rows of the factor
        constexpr int NT = (kLqSmall + kLqWaves - 1) / kLqWaves;
        const int kk = (int)k;
        const int pt = lane < nw ? lane : 0, ps = lane < mw ? lane : 0;
        const uint64_t vt = a.T[k * nw + pt], vs = a.S[k * mw + ps];
        uint64_t tw[NT], sw[NT];
        double row[NT][2], yl[2], bl[2], cl[2];
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int j = wv + i * kLqWaves, jc = j < kk ? j : kk;  // (the new term's words stand for what is past the end)
            tw[i] = a.T[(int64_t)jc * nw + pt];
            sw[i] = a.S[(int64_t)jc * mw + ps];
#pragma unroll
            for (int h = 0; h < 2; ++h) row[i][h] = j < kk && lane + h * kWave <= j ? a.L[j * a.w + lane + h * kWave] : 0.0;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int q = lane + h * kWave;
            yl[h] = wv == 0 && q < kk ? a.yv[q] : 0.0;
            bl[h] = wv == 0 && q < kk ? a.bvec[q] : 0.0;
            cl[h] = wv == 0 && q < kk ? a.c[q] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int j = wv + i * kLqWaves;
            int ct = lane < nw ? __popcll(tw[i] ^ vt) : 0, cs = lane < mw ? __popcll(sw[i] ^ vs) : 0;
            for (int off = 32; off > 0; off >>= 1) {
                ct += __shfl_xor(ct, off, kWave);
                cs += __shfl_xor(cs, off, kWave);
            }
            if (j < kk) {
                if (lane == 0) u.sm.e[j] = (double)(a.n - 2 * (int64_t)ct) * (double)(a.m - 2 * (int64_t)cs);
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (lane + h * kWave <= j) u.sm.L[j * (j + 1) / 2 + lane + h * kWave] = row[i][h];
            }
        }
        __syncthreads();
        if (wv != 0) return;
        double b = 0.0;
#pragma unroll
        for (int h = 0; h < 2; ++h) b += lq_wave_sum(lane + h * kWave < kk ? cl[h] * u.sm.e[lane + h * kWave] : 0.0);
        b += cut;
        if (lane == 0) a.bvec[k] = b;
        ok = lq_refit_small(u.sm, a.L, a.w, kk, (double)a.m * (double)a.n, b, yl, bl, a.yv, a.c, &cb);
    } else {
        if (tid < nw) sh.vec[tid] = a.T[k * nw + tid];
        __syncthreads();
        lq_dots(a.T, k, nw, a.n, sh.vec, nullptr, sh.e);
        __syncthreads();
        if (tid < mw) sh.vec[tid] = a.S[k * mw + tid];
        __syncthreads();
        lq_dots(a.S, k, mw, a.m, sh.vec, sh.e, sh.e);  // (each element is read and written by the same lane)
        __syncthreads();
        double b = 0.0;
        for (int64_t j = tid; j < k; j += kLqThreads) b = __builtin_fma(a.c[j], sh.e[j], b);
        b = cut + lq_block_sum(b, sh.red);
        if (tid == 0) a.bvec[k] = b;
        __syncthreads();
        ok = lq_refit(a.L, a.w, k, sh.e, (double)a.m * (double)a.n, a.bvec, a.yv, a.c, sh.red, &sh.part[0][0], &cb);
    }
    if (tid == 0) {
        if (!ok) {
            st->status = 1;
            st->done = 1;
        } else {
            const double f2 = a.fro0sq - cb;
            a.trace[k + 1] = sqrt(f2 > 0.0 ? f2 : 0.0);
            st->k = k + 1;
            st->total += a.iters[k];
            if (k + 1 >= a.w) st->done = 1;
        }
    }
}

}  // namespace

hipError_t launch_lsq_dots(const uint64_t* bits, int64_t k, int64_t nw, int64_t len, const uint64_t* vec, const double* coef,
                           double* out, hipStream_t st)
{
    if (k <= 0) return hipSuccess;
    hipLaunchKernelGGL(lsq_dots_kernel, dim3((unsigned)((k + 3) / 4)), dim3(256), 0, st, bits, k, nw, len, vec, coef, out);
    return hipGetLastError();
}

hipError_t launch_lsq_correct(const uint64_t* bits, int64_t k, int64_t mw, int64_t m, const double* e, const double* base,
                              uint64_t* out_bits, double* abs_parts, double* dot_parts, hipStream_t st)
{
    hipLaunchKernelGGL(lsq_correct_kernel, dim3((unsigned)mw), dim3(512), 0, st, bits, k, mw, m, e, base, out_bits, abs_parts,
                       dot_parts);
    return hipGetLastError();
}

hipError_t launch_lsq_prod(const double* D, int64_t ld, int order, int skip, int64_t k, const double* coef, double* out,
                           hipStream_t st)
{
    if (k <= 0) return hipSuccess;
    hipLaunchKernelGGL(lsq_prod_kernel, dim3((unsigned)((k + 255) / 256)), dim3(256), 0, st, D, ld, order, skip, k, coef, out);
    return hipGetLastError();
}

hipError_t launch_lsq_kron(const uint64_t* const* signs, const int64_t* dims, int first, int last, int64_t len, uint64_t* out,
                           hipStream_t st)
{
    LsqKronArgs a;
    for (int m = 0; m < SCD_MAX_ORDER; ++m) {
        a.signs[m] = (m >= first && m < last) ? signs[m] : nullptr;
        a.dims[m] = (m >= first && m < last) ? dims[m] : 1;
    }
    a.first = first;
    a.last = last;
    a.len = len;
    a.out = out;
    const int64_t padded = ((len + 63) / 64) * 64;
    hipLaunchKernelGGL(lsq_kron_kernel, dim3((unsigned)((padded + 255) / 256)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_scalars_coef(const double* u, int64_t q, double P, scd_dtype dt, void* c, hipStream_t st)
{
    const unsigned g = (unsigned)((q + 255) / 256);
    if (dt == SCD_F32)
        hipLaunchKernelGGL((scalars_coef_kernel<float>), dim3(g), dim3(256), 0, st, u, q, P, (float*)c);
    else
        hipLaunchKernelGGL((scalars_coef_kernel<double>), dim3(g), dim3(256), 0, st, u, q, P, (double*)c);
    return hipGetLastError();
}

hipError_t launch_scalars_update(void* r, scd_dtype dt, int64_t total, int64_t q, const uint64_t* lead, const void* c,
                                 double* parts, int nparts, hipStream_t st)
{
    if (dt == SCD_F32)
        hipLaunchKernelGGL((scalars_update_kernel<float>), dim3(nparts), dim3(256), 0, st, (float*)r, total, q, lead,
                           (const float*)c, parts);
    else
        hipLaunchKernelGGL((scalars_update_kernel<double>), dim3(nparts), dim3(256), 0, st, (double*)r, total, q, lead,
                           (const double*)c, parts);
    return hipGetLastError();
}

hipError_t launch_lsq_sum2(const double* a, const double* b, int64_t n, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(lsq_sum2_kernel, dim3(1), dim3(256), 0, st, a, b, n, out);
    return hipGetLastError();
}

hipError_t launch_lsq_sumsq(const void* A, scd_dtype dt, int64_t total, double* parts, int nparts, hipStream_t st)
{
    if (dt == SCD_F32)
        hipLaunchKernelGGL((lsq_sumsq_kernel<float>), dim3(nparts), dim3(256), 0, st, (const float*)A, total, parts);
    else
        hipLaunchKernelGGL((lsq_sumsq_kernel<double>), dim3(nparts), dim3(256), 0, st, (const double*)A, total, parts);
    return hipGetLastError();
}

hipError_t launch_lsq_cast(const double* c, int64_t k, scd_dtype dt, void* out, hipStream_t st)
{
    if (k <= 0) return hipSuccess;
    const unsigned g = (unsigned)((k + 255) / 256);
    if (dt == SCD_F32)
        hipLaunchKernelGGL((lsq_cast_kernel<float>), dim3(g), dim3(256), 0, st, c, k, (float*)out);
    else
        hipLaunchKernelGGL((lsq_cast_kernel<double>), dim3(g), dim3(256), 0, st, c, k, (double*)out);
    return hipGetLastError();
}

hipError_t launch_lsq_solve(double* L, int64_t ld, int64_t k, const double* g, double diag, const double* bvec, double* yv,
                            double* c, double fro0sq, double* trace_out, int* status, hipStream_t st)
{
    hipLaunchKernelGGL(lsq_solve_kernel, dim3(1), dim3(kLqThreads), 0, st, L, ld, k, g, diag, bvec, yv, c, fro0sq,
                       trace_out, status);
    return hipGetLastError();
}

// A workgroup per word of rows or columns: up to 64 of them, each reading a strip of at most 1 MiB.
bool lsq_matrix_supported(scd_dtype dt, int64_t m, int64_t n)
{
    const int64_t es = dt == SCD_F32 ? 4 : 8;
    return m <= kLqMaxWords * 64 && n <= kLqMaxWords * 64 && 64 * m * es <= (1 << 20) && 64 * n * es <= (1 << 20);
}

template <typename TE, bool VEC>
static hipError_t lsq_sweep_t(const LsqMatArgs& a, hipStream_t st)
{
    hipLaunchKernelGGL((lsq_rows_kernel<TE, VEC>), dim3((unsigned)((a.m + 63) / 64)), dim3(kLqThreads), 0, st, a);
    hipLaunchKernelGGL((lsq_cols_kernel<TE, VEC>), dim3((unsigned)((a.n + 63) / 64)), dim3(kLqThreads), 0, st, a);
    hipLaunchKernelGGL(lsq_next_kernel, dim3(1), dim3(kLqThreads), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_lsq_sweep(const LsqMatArgs& a, scd_dtype dt, hipStream_t st)
{
    const int ve = dt == SCD_F32 ? 4 : 2;
    const bool vec = a.n % ve == 0 && ((uintptr_t)a.A & 15u) == 0;  // every row starts on a 16-byte boundary
    if (dt == SCD_F32) return vec ? lsq_sweep_t<float, true>(a, st) : lsq_sweep_t<float, false>(a, st);
    return vec ? lsq_sweep_t<double, true>(a, st) : lsq_sweep_t<double, false>(a, st);
}

hipError_t launch_lsq_term(const LsqMatArgs& a, const ResidentResult* res, hipStream_t st)
{
    hipLaunchKernelGGL(lsq_term_kernel, dim3(1), dim3(kLqThreads), 0, st, a, res);
    return hipGetLastError();
}

}  // namespace scd
