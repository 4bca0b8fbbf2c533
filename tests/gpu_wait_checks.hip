// gpu_wait_checks.hip - device checks of the divisions of the pipelined kernel's clock
// wave and of 16-bit quotients, against the kernel's own device functions (the template
// is included as it is): bit-equal to the IEEE division over the ranges that they are
// used on.
//
//  * wait_mid: -ln(u1) / a0 for totals with a binary exponent in [-60, 60), in binary64
//    [-500, 500): a hashed sample, and both ends of every exponent;
//  * Prec16<FP16>::quotient: every pair of fp16 values.
//
// Test infrastructure: built next to the tests, loaded by them only.
#include <hip/hip_runtime.h>

#include <cstdint>

#define SSA_N_ITEMS 1
#include "../paper_2605_00479_amd/csrc/ssa_device.hip"

namespace {

__device__ __forceinline__ uint32_t mix64(uint64_t x)
{
    x ^= x >> 33;
    x *= 0xff51afd7ed558ccdull;
    x ^= x >> 33;
    x *= 0xc4ceb9fe1a85ec53ull;
    x ^= x >> 33;
    return (uint32_t)x;
}

// mantissa i of `bits`: a few at each end, then hashed
__device__ __forceinline__ uint64_t mantissa(uint64_t i, int bits)
{
    const uint64_t all = (1ull << bits) - 1;
    if (i < 8)
        return i;
    if (i < 16)
        return all - (i - 8);
    return (((uint64_t)mix64(i) << 32) | mix64(i ^ 0x9E3779B97F4A7C15ull)) & all;
}

// Per exponent of a0, n pairs: -ln(u1) is 0 or has an exponent from 2^lo on up to 2^hi.
__global__ void check_wait64(uint32_t n, unsigned long long *cnt)
{
    const uint64_t total = 1000ull * n, stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < total; i += stride) {
        const uint64_t e = 1023 - 500 + i % 1000, k = i / 1000;
        const double a0 = __longlong_as_double((i64)((e << 52) | mantissa(k % 64 < 16 ? k % 64 : i, 52)));
        const uint64_t le = 1023 - 53 + mix64(i + 0x1234567ull) % 59;   // 2^-53 .. 2^6
        const double l = k % 97 == 5 ? 0.0 : __longlong_as_double((i64)((le << 52) | mantissa(k % 61 < 16 ? k % 61 : i * 3 + 1, 52)));
        if (!total_mid<PrecF64>(a0))
            atomicAdd(&cnt[1], 1ull);
        if (__double_as_longlong(wait_mid<PrecF64>(l, a0)) != __double_as_longlong(l / a0))
            atomicAdd(&cnt[0], 1ull);
    }
}

template <class P>
__global__ void check_wait32(uint32_t n, unsigned long long *cnt)
{
    const uint64_t total = 120ull * n, stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < total; i += stride) {
        const uint32_t e = 127 - 60 + (uint32_t)(i % 120);
        const uint64_t k = i / 120;
        const float a0 = __uint_as_float((e << 23) | (uint32_t)mantissa(k % 64 < 16 ? k % 64 : i, 23));
        const uint32_t le = 127 - 24 + mix64(i + 0x1234567ull) % 29;   // 2^-24 .. 2^5
        const float l = k % 97 == 5 ? 0.0f : __uint_as_float((le << 23) | (uint32_t)mantissa(k % 61 < 16 ? k % 61 : i * 3 + 1, 23));
        if (!total_mid<P>(a0))
            atomicAdd(&cnt[1], 1ull);
        if (__float_as_uint(wait_mid<P>(l, a0)) != __float_as_uint(l / a0))
            atomicAdd(&cnt[0], 1ull);
    }
}

__device__ __forceinline__ float from_f16(uint32_t h)
{
    return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
}

// every pair of fp16 values; NaN results are compared as NaN
__global__ void check_quotient(unsigned long long *cnt)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < (1ull << 32); i += stride) {
        const float a = from_f16((uint32_t)i & 0xFFFFu), b = from_f16((uint32_t)(i >> 16));
        const float q = Prec16<FMT_FP16, 1, true, false>::quotient(a, b), r = a / b;
        const bool same = r != r ? q != q : __float_as_uint(q) == __float_as_uint(r);
        if (!same)
            atomicAdd(&cnt[0], 1ull);
    }
}

}  // namespace

// Mismatches: out[0] binary64 waiting times (1000 n pairs), out[2] and out[4] binary32
// ones of mixed bfloat16 and FP32 (120 n pairs each), out[6] fp16 quotients; out[1],
// out[3], out[5]: totals of these ranges that the kernel would send to the full division.
extern "C" int gpu_check_waits(unsigned int n, unsigned long long *out)
{
    if (n == 0 || n > (1u << 24))
        return 4;
    unsigned long long *d = nullptr;
    if (hipMalloc(&d, 7 * sizeof *d) != hipSuccess)
        return 2;
    if (hipMemset(d, 0, 7 * sizeof *d) != hipSuccess)
        return 3;
    check_wait64<<<4096, 256>>>(n, d);
    check_wait32<Prec16<FMT_BF16, 1, false, false>><<<4096, 256>>>(n, d + 2);
    check_wait32<PrecF32><<<4096, 256>>>(n, d + 4);
    check_quotient<<<4096, 256>>>(d + 6);
    if (hipDeviceSynchronize() != hipSuccess)
        return 3;
    if (hipMemcpy(out, d, 7 * sizeof *d, hipMemcpyDeviceToHost) != hipSuccess)
        return 3;
    return hipFree(d) == hipSuccess ? 0 : 3;
}
