// scd_exchange.h -- what the persistent engines' exchanges share: the tag of a word, 16-byte reads of device scope, and sums
// over lanes 16 and 32 apart for two registers at once.
#ifndef SCD_EXCHANGE_H
#define SCD_EXCHANGE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace scd {

// The top bit of the exponent of a published sum (below 2 once scaled, so that the bit is free).  The tag flips each time that
// a slot is written: slots alternate by the parity of the exchange's number, so every second exchange; cleared slots
// are older than exchange 1.
constexpr uint32_t kTagBit = 0x40000000u;
__device__ __forceinline__ uint32_t exchange_tag(uint32_t seq) { return (((seq + 1u) >> 1) & 1u) ? kTagBit : 0u; }

// A word of one f64 sum that travels in accesses of 16 bytes.  Only of naturally aligned accesses of up to 64 bits does the
// memory model say that they are seen whole, and of wider ones no more than that each of their 32 bits are: so both halves of the
// word carry the tag.  The sum is scaled below 2^-511 (kF64Exp below what suffices for an f32 or an atomic word), which leaves
// two bits of its exponent clear: one for the tag, one for the lowest bit of the mantissa, whose place takes the other tag.
constexpr int kF64Exp = 512;
__device__ __forceinline__ void exchange_pack(double v, uint32_t tag, uint32_t& lo, uint32_t& hi)
{
    lo = ((uint32_t)__double2loint(v) & ~1u) | (tag >> 30);
    hi = (uint32_t)__double2hiint(v) | ((uint32_t)__double2loint(v) & 1u) << 29 | tag;
}
__device__ __forceinline__ double exchange_unpack(uint32_t lo, uint32_t hi)
{
    return __hiloint2double((int)(hi & 0x9FFFFFFFu), (int)((lo & ~1u) | ((hi >> 29) & 1u)));
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr int kDeviceScope = (int)0x80000010;  // volatile, device scope: past the caches that are not coherent
__device__ __forceinline__ u32x4 exchange_load16(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff)
{
    return __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff, (int)soff, kDeviceScope);
}

// Sum over the four 16-lane rows of a wave for two registers at once: the row-swap instructions of gfx950 exchange
// the odd rows (the upper half of the wave) of one register with the even rows (the lower half) of the other, after
// which one addition serves both.  half16(a, b): even rows hold a's pair sums, odd rows b's.  half32 of two such:
// row r of the result holds the full sum of the r-th of the four registers.
__device__ __forceinline__ float half16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float half32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ double half16(double a, double b)
{
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ double half32(double a, double b)
{
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}

}  // namespace scd

#endif
