// ssa_device.hip - device side of the ensemble direct method on gfx950.
//
// This file is compiled at run time by hipRTC together with a short,
// generated description of the reaction networks in the launch (species and
// reaction counts, the op sequence of every propensity, the net-change table)
// and one instantiation line. Everything structural is therefore a
// compile-time constant: propensity evaluation, prefix sums, selection and the
// integer update are straight-line code in registers, one trajectory per lane.
// Rate constants, initial states, horizons and snapshot grids stay runtime data.
//
// Method (Kimpson, Flegg & Flegg, Sec. 2, Direct Method steps 1-4):
//   a_j(x), a0 = sum a_j;  tau = -ln(u1)/a0;  mu = min{j : S_j > u2 a0};
//   x += nu_mu, t += tau.
// Precision partition (Sec. 3.2 and opening of Sec. 4):
//   FP64 / FP32: every op in that type.
//   mixed T16:   propensity ops in fp16/bf16, sums, tau, time in binary32.
//   uniform T16: every op in fp16/bf16, including the clock.
// Stochastic rounding (Sec. 3.3): each 16-bit op rounds its binary32 result
// up with probability (x - x-)/(x+ - x-), decided by a 16-bit halfword.
//
// Random bits: Philox4x32-10, key = seed, counter = (event lo, event hi,
// trajectory id, stream). Stream 0 gives the two uniforms (53-bit pairs in
// FP64, the high 24 bits of words 0 and 1 otherwise). In SR modes every
// rounding op of an event owns a fixed slot holding a B-bit random field
// (B = 13 for fp16, 16 for bf16: the mantissa bits a binary32 -> 16-bit
// rounding discards). Main slots are fields of the 80 spare bits of stream 0,
// then of streams 1, 2, ...; conversions of counts have their own slots in
// streams 2^31, 2^31 + 1, ..., drawn only when a count is not exactly
// representable (otherwise the conversion rounds nothing). A step's randomness
// is a function of (seed, trajectory, event) only, so results do not depend on
// lane scheduling.
#pragma clang fp contract(off)

typedef unsigned int u32;
typedef int i32;
typedef unsigned long long u64;
typedef long long i64;

#define SSA_INF_F __builtin_inff()

// --------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11).
// --------------------------------------------------------------------------
struct W4 {
    u32 w0, w1, w2, w3;
};

__device__ __forceinline__ u32 xor3(u32 a, u32 b, u32 c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);   // a ^ b ^ c in one VALU op
}

// Rounds FROM .. 9 on the counter c.
template <int FROM>
__device__ __forceinline__ W4 philox_rounds(W4 c, u32 k0, u32 k1)
{
    k0 += FROM * 0x9E3779B9u;
    k1 += FROM * 0xBB67AE85u;
#pragma unroll
    for (int r = FROM; r < 10; ++r) {
        const u64 p0 = (u64)0xD2511F53u * (u64)c.w0;
        const u64 p1 = (u64)0xCD9E8D57u * (u64)c.w2;
        c = {xor3((u32)(p1 >> 32), c.w1, k0), (u32)p1, xor3((u32)(p0 >> 32), c.w3, k1), (u32)p0};
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// The generator of one trajectory: counter (n, id, stream), key (k0, k1).
struct Philox {
    u32 id, k0, k1;
    __device__ __forceinline__ W4 operator()(u64 n, u32 stream) const
    {
        return philox_rounds<0>({(u32)n, (u32)(n >> 32), id, stream}, k0, k1);
    }
};

// The same for event indices that share their upper word: half of the first round's
// products and half of the second's depend on the trajectory and that word alone.
struct PhiloxNear {
    u32 k0, k1, lo1, hi2, lo2;
    __device__ __forceinline__ PhiloxNear(const Philox &g, u32 n_hi)
    {
        const u64 p1 = (u64)0xCD9E8D57u * (u64)g.id;
        const u64 p0 = (u64)0xD2511F53u * (u64)xor3((u32)(p1 >> 32), n_hi, g.k0);
        k0 = g.k0;
        k1 = g.k1;
        lo1 = (u32)p1;
        hi2 = (u32)(p0 >> 32) ^ (g.k1 + 0xBB67AE85u);
        lo2 = (u32)p0;
    }
    __device__ __forceinline__ W4 operator()(u64 n, u32 stream) const
    {
        const u64 p0 = (u64)0xD2511F53u * (u64)(u32)n;
        const u64 p1 = (u64)0xCD9E8D57u * (u64)((u32)(p0 >> 32) ^ (stream ^ k1));
        return philox_rounds<2>({xor3((u32)(p1 >> 32), lo1, k0 + 0x9E3779B9u), (u32)p1, hi2 ^ (u32)p0, lo2}, k0, k1);
    }
};

// Constants of the draws that are no inline operands. A kernel that keeps them in
// registers (pin) spares the copies that the two-operand multiply-add and the
// one-scalar limit of an instruction ask for.
struct DrawConst {
    double ulp53 = 0x1p-53, c19 = 0x1.af286bca1af28p-5;
    float ulp24 = 0x1p-24f;
    u32 mant64 = 0xFFFFFu, one64 = 0x3FF00000u, mant32 = 0x7FFFFFu, one32 = 0x3F800000u;
    __device__ __forceinline__ void pin()
    {
        __asm__ volatile("" : "+v"(ulp53), "+v"(c19), "+v"(ulp24), "+v"(one64), "+v"(one32));
        __asm__ volatile("" : "+s"(mant64), "+s"(mant32));
    }
};

// --------------------------------------------------------------------------
// Uniforms on (0, 1]: (m + 1) 2^-53 from 53 bits, (m + 1) 2^-24 from 24 bits.
// --------------------------------------------------------------------------
__device__ __forceinline__ double unif53(u32 a, u32 b, const DrawConst &k = DrawConst())
{
    // m = a 2^21 + (b >> 11): every product and sum below is exact (m + 1 <= 2^53)
    return __builtin_fma((double)a, 0x1p-32, __builtin_fma((double)(b >> 11), k.ulp53, k.ulp53));
}

__device__ __forceinline__ float unif24(u32 w, const DrawConst &k = DrawConst())
{
    // (m + 1) 2^-24 = m 2^-24 + 2^-24, exact in binary32 for m < 2^24
    return __builtin_fmaf((float)(w >> 8), k.ulp24, k.ulp24);
}

// --------------------------------------------------------------------------
// Correctly rounded binary32 a / b (the IEEE quotient) for operands that need
// no range scaling: a = 0 or 2^-24 <= |a| < 32, and 2^-60 <= b < 2^60. The
// hardware reciprocal is refined by one Newton-Raphson step, then the quotient
// by two remainder corrections (Markstein's fma division). On these ranges it
// equals the full division sequence, which adds operand scaling and a
// special-case fix-up (compared on the device with 2^20 pairs for each exponent of
// b, and over the fp16 ranges of b with every fourth numerator); it saves three
// instructions per use.
// --------------------------------------------------------------------------
// (f - 1) / (f + 1) for binary32 f in [1/2, 2): the hardware reciprocal, the
// product and one remainder correction already give the IEEE quotient for
// every such f (checked on the device over all of them).
__device__ __forceinline__ float div_rn_log(float a, float b)
{
    const float r = __builtin_amdgcn_rcpf(b);
    const float q = a * r;
    const float rem = __builtin_fmaf(-b, q, a);
    return __builtin_fmaf(rem, r, q);
}

// (f - 1) / (f + 1) for binary64 f in [1/2, 2): the compiler's IEEE division
// without its operand scaling and special-case fix-up, which leave these
// operands unchanged (the numerator is 0 or at least 2^-53 in magnitude, the
// denominator in [1.5, 3), the quotient normal): reciprocal, two Newton steps,
// product, and the remainder correction as a plain fma.
// The same holds for a waiting time: -ln(u1), 0 or in [2^-53, 64), by a total of exponent
// [-500, 500) (compared on the device with 2^20 pairs for each exponent).
__device__ __forceinline__ double div_rn_log64(double a, double b)
{
    const double r0 = __builtin_amdgcn_rcp(b);
    const double e0 = __builtin_fma(-b, r0, 1.0);
    const double r1 = __builtin_fma(r0, e0, r0);
    const double e1 = __builtin_fma(-b, r1, 1.0);
    const double r2 = __builtin_fma(r1, e1, r1);
    const double q = a * r2;
    const double rem = __builtin_fma(-b, q, a);
    return __builtin_fma(rem, r2, q);
}

__device__ __forceinline__ float div_rn_inrange(float a, float b)
{
    float r = __builtin_amdgcn_rcpf(b);
    float e = __builtin_fmaf(-b, r, 1.0f);
    r = __builtin_fmaf(e, r, r);
    float q = a * r;
    float rem = __builtin_fmaf(-b, q, a);
    q = __builtin_fmaf(rem, r, q);
    rem = __builtin_fmaf(-b, q, a);
    return __builtin_fmaf(rem, r, q);
}

// --------------------------------------------------------------------------
// -ln(u), u in (0, 1]: u = 2^e f with f in [1/sqrt2, sqrt2],
// ln f = 2 atanh(s) = 2s (1 + s^2/3 + s^4/5 + ...), s = (f - 1)/(f + 1),
// e ln2 with ln2 split in a short high part (exact product) and a low part.
// Only correctly rounded +, -, *, / and fused multiply-adds are used, in a
// fixed order: the quotient s, the series by Horner's rule in fmas, ln f =
// fma(2s, p z, 2s), and fma(e, ln2_hi, fma(e, ln2_lo, ln f)).
// --------------------------------------------------------------------------
__device__ __forceinline__ double neg_log64(double u, const DrawConst &k = DrawConst())
{
    const u64 bits = (u64)__double_as_longlong(u);
    const u32 hi = (u32)(bits >> 32);
    const double g = __longlong_as_double((i64)(((u64)((hi & k.mant64) | k.one64) << 32) | (bits & 0xFFFFFFFFull)));
    const bool big = g > 0x1.6a09e667f3bcdp+0;
    const int e = (int)(hi >> 20) + (big ? -1022 : -1023);
    const double h = __longlong_as_double((i64)(big ? 0x3FE0000000000000ull : 0x3FF0000000000000ull));
    double s = div_rn_log64(__builtin_fma(g, h, -1.0), __builtin_fma(g, h, 1.0));   // f = g h, exact
    double z = s * s;
    double p = 0x1.8618618618618p-5;         // 1/21
    p = __builtin_fma(p, z, k.c19);          // 1/19
    p = __builtin_fma(p, z, 0x1.e1e1e1e1e1e1ep-5); // 1/17
    p = __builtin_fma(p, z, 0x1.1111111111111p-4); // 1/15
    p = __builtin_fma(p, z, 0x1.3b13b13b13b14p-4); // 1/13
    p = __builtin_fma(p, z, 0x1.745d1745d1746p-4); // 1/11
    p = __builtin_fma(p, z, 0x1.c71c71c71c71cp-4); // 1/9
    p = __builtin_fma(p, z, 0x1.2492492492492p-3); // 1/7
    p = __builtin_fma(p, z, 0x1.999999999999ap-3); // 1/5
    p = __builtin_fma(p, z, 0x1.5555555555555p-2); // 1/3
    p = p * z;
    double s2 = s + s;
    double lnf = __builtin_fma(s2, p, s2);
    double ed = (double)e;
    return __builtin_fma(-ed, 0x1.62e42fep-1, -__builtin_fma(ed, 0x1.f473de6af278fp-30, lnf));
}

__device__ __forceinline__ float neg_log32(float u, const DrawConst &k = DrawConst())
{
    const u32 bits = __float_as_uint(u);
    const float g = __uint_as_float((bits & k.mant32) | k.one32);
    const bool big = g > 0x1.6a09e6p+0f;
    const int e = (int)(bits >> 23) + (big ? -126 : -127);
    const float h = big ? 0.5f : 1.0f;
    float s = div_rn_log(__builtin_fmaf(g, h, -1.0f), __builtin_fmaf(g, h, 1.0f));   // f = g h, exact
    float z = s * s;
    float p = 0x1.c71c72p-4f;                 // 1/9
    p = __builtin_fmaf(p, z, 0x1.24924ap-3f); // 1/7
    p = __builtin_fmaf(p, z, 0x1.99999ap-3f); // 1/5
    p = __builtin_fmaf(p, z, 0x1.555556p-2f); // 1/3
    p = p * z;
    float s2 = s + s;
    float lnf = __builtin_fmaf(s2, p, s2);
    float ed = (float)e;
    float r = __builtin_fmaf(-ed, 0x1.62e4p-1f, -__builtin_fmaf(ed, 0x1.7f7d1cp-20f, lnf));
    // rounded here: a conversion to fp16 that follows would be one instruction with the
    // multiply-add, which rounds once
    __asm__("" : "+v"(r));
    return r;
}

// --------------------------------------------------------------------------
// Rounding a binary32 value to fp16 / bf16 (result carried as binary32).
// Formats per Table tab:formats. Round-to-nearest-even uses the IEEE
// conversions (subnormals kept, overflow to infinity). Stochastic rounding
// uses gfx950's SR conversions: with f the dropped fraction of a grid step,
// the magnitude rounds up when the top B bits of the 16-bit halfword plus
// floor(f 2^B) reach 2^B (B = 16 for bf16, 13 for fp16). The instructions read
// their random bits from the upper half of the 32-bit operand and ignore the
// lower half, so `r` carries the slot's halfword in bits 31..16.
// --------------------------------------------------------------------------
typedef __bf16 ssa_v2bf16 __attribute__((ext_vector_type(2)));
typedef _Float16 ssa_v2f16 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float rne_f16(float v)
{
    return (float)(_Float16)v;
}

__device__ __forceinline__ float rne_bf16(float v)
{
    return (float)(__bf16)v;
}

// The conversions write one 16-bit half of a register and keep the other; the
// random operand serves as that other half, so no register needs clearing or copying
// where it is dead afterwards; where it is half of a word that holds two (SHARED), the
// converted value does. With the bfloat16 in the upper half and zeros
// in the lower one the register holds the value in binary32.
__device__ __forceinline__ float sr_bf16(float v, u32 r)
{
    const u32 h = r & 0xFFFF0000u;   // (no instruction where the field was shifted up)
    return __builtin_bit_cast(float, __builtin_amdgcn_cvt_sr_bf16_f32(__builtin_bit_cast(ssa_v2bf16, h), v, h, true));
}

template <bool SHARED = false>
__device__ __forceinline__ float sr_f16(float v, u32 r)
{
    const ssa_v2f16 keep = SHARED ? __builtin_bit_cast(ssa_v2f16, v) : __builtin_bit_cast(ssa_v2f16, r);
    const ssa_v2f16 o = __builtin_amdgcn_cvt_sr_f16_f32(keep, v, r, false);
    return (float)o[0];
}

// --------------------------------------------------------------------------
// Precision policies. T: propensity type; A: sum/target type; Tm: clock type.
// rnd(v, rb) is the one rounding applied after every 16-bit op.
// --------------------------------------------------------------------------
enum { FMT_FP64 = 0, FMT_FP32 = 1, FMT_FP16 = 2, FMT_BF16 = 3 };

struct PrecF64 {
    typedef PrecF64 Packed;
    typedef double T;
    typedef double A;
    typedef double Tm;
    static constexpr bool SR = false, UNI = false, NORM = false, WIDE = true, SELECTIVE = false, NATIVE16 = false, NARROW = false;
    static constexpr i32 EXACT_INT = 0;   // conversions are exact: no count test
    static constexpr int SR_B = 16;
    template <bool EXACT>
    __device__ static T cvt(i32 v, u32) { return (double)v; }
    // (x - i) converted: x converted once, then an exact binary64 subtraction
    template <bool EXACT>
    __device__ static T cvt_sub(i32 x, i32 i, u32) { return (double)x - (double)i; }
    __device__ static T mul(T a, T b, u32) { return a * b; }
    __device__ static T div(T a, T b, u32) { return a / b; }
    __device__ static T add(T a, T b, u32) { return a + b; }
    __device__ static A acc(A s, T a, u32) { return s + (A)a; }
    __device__ static A acc(A s, T a, u32 rb, float) { return acc(s, a, rb); }
    __device__ static A arnd(A v, u32) { return v; }
    __device__ static A tacc(A v, u32) { return v; }
    __device__ static A tau_div(A l, A a0) { return l / a0; }
};

struct PrecF32 {
    typedef PrecF32 Packed;
    typedef float T;
    typedef float A;
    typedef float Tm;
    static constexpr bool SR = false, UNI = false, NORM = false, WIDE = false, SELECTIVE = false, NATIVE16 = false, NARROW = false;
    static constexpr i32 EXACT_INT = 0;
    static constexpr int SR_B = 16;
    template <bool EXACT>
    __device__ static T cvt(i32 v, u32) { return (float)v; }
    template <bool EXACT>
    __device__ static T cvt_sub(i32 x, i32 i, u32 rb) { return cvt<EXACT>(x - i, rb); }
    __device__ static T mul(T a, T b, u32) { return a * b; }
    __device__ static T div(T a, T b, u32) { return a / b; }
    __device__ static T add(T a, T b, u32) { return a + b; }
    __device__ static A acc(A s, T a, u32) { return s + a; }
    __device__ static A acc(A s, T a, u32 rb, float) { return acc(s, a, rb); }
    __device__ static A arnd(A v, u32) { return v; }
    __device__ static A tacc(A v, u32) { return v; }
    __device__ static A tau_div(A l, A a0) { return l / a0; }
};

// v as computed in binary32. An operation followed by a conversion to fp16 may
// otherwise be fused into one v_fma_mixlo_f16, which rounds the exact result
// once where the op and the conversion round twice. For +, -, x, / of two fp16
// values the two agree; where an operand has more bits (u2 in the selection
// target) they can differ at a tie of the second rounding.
__device__ __forceinline__ float f32_kept(float v)
{
    __asm__ volatile("" : "+v"(v));
    return v;
}

template <int FMT, bool SRM, bool SHARED = false>
__device__ __forceinline__ float rnd16(float v, u32 rb)
{
    if constexpr (FMT == FMT_FP16)
        return SRM ? sr_f16<SHARED>(v, rb) : rne_f16(v);
    else
        return SRM ? sr_bf16(v, rb) : rne_bf16(v);
}

// RND: 0 round to nearest; 1 stochastic rounding after every 16-bit op;
// 2 stochastic rounding only where values accumulate (partial sums and the
// clock, uniform mode), round to nearest elsewhere - the selective SR the
// paper names as untested (Sec. 3.3, last paragraph).
// binary32 a * b and a + b, each rounded once. For fp16 operands they are
// written as fma(a, b, +0) and fma(a, 1, b) (equal to the product and the sum
// for the non-negative values met here), which gfx950 runs as v_fma_mix_f32
// reading the 16-bit halves directly, without a separate widening conversion.
template <int FMT>
__device__ __forceinline__ float mul32(float a, float b)
{
    if constexpr (FMT == FMT_FP16)
        return __builtin_fmaf(a, b, 0.0f);
    else
        return a * b;
}

template <int FMT>
__device__ __forceinline__ float add32(float a, float b)
{
    if constexpr (FMT == FMT_FP16)
        return __builtin_fmaf(b, 1.0f, a);
    else
        return a + b;
}

// SHARED: the event wave's fields come two to a word.
template <int FMT, int RND, bool UNIF, bool NRM, bool SHARED = false>
struct Prec16 {
    typedef Prec16<FMT, RND, UNIF, NRM, true> Packed;
    typedef float T;
    typedef float A;
    typedef float Tm;
    static constexpr bool SR = RND != 0, UNI = UNIF, NORM = NRM, WIDE = false, SELECTIVE = RND == 2;
    static constexpr bool SR_OPS = RND == 1, SR_ACC = RND != 0;
    static constexpr int SR_B = FMT == FMT_FP16 ? 13 : 16;   // random bits per SR rounding
    // counts up to EXACT_INT in magnitude are 16-bit values already: their
    // conversion rounds nothing (by either rule) and needs no random bits
    static constexpr i32 EXACT_INT = FMT == FMT_FP16 ? 2048 : 256;
    template <bool EXACT>
    __device__ static T cvt(i32 v, u32 rb)
    {
        if constexpr (EXACT)
            return (float)v;
        else
            return rnd16<FMT, SR_OPS, SHARED>((float)v, rb);
    }
    // (x - i) converted. With |x| within the exact-integer limit the binary32
    // subtraction of the converted x is exact, and x is converted once.
    template <bool EXACT>
    __device__ static T cvt_sub(i32 x, i32 i, u32 rb)
    {
        if constexpr (EXACT)
            return (float)x - (float)i;
        else
            return rnd16<FMT, SR_OPS, SHARED>((float)(x - i), rb);
    }
    // Round to nearest in fp16: the hardware's fp16 product and sum
    // (v_mul_f16, v_add_f16) are the correctly rounded results, equal to the
    // binary32 op followed by one rounding (exact product; innocuous double
    // rounding for the sum, 24 >= 2*11 + 2). Division keeps the binary32
    // quotient and one rounding (the compiler's fp16 division is not an IEEE
    // operation).
    static constexpr bool NATIVE16 = FMT == FMT_FP16 && !SR_OPS;
    static constexpr bool NARROW = FMT == FMT_FP16;   // products of counts overflow
    __device__ static T mul(T a, T b, u32 rb)
    {
        if constexpr (NATIVE16)
            return (float)((_Float16)a * (_Float16)b);
        else
            return rnd16<FMT, SR_OPS, SHARED>(mul32<FMT>(a, b), rb);
    }
    // fp16: both operands have 11 significant bits and lie in [2^-24, 2^16), or are
    // special. One remainder correction of a times the hardware reciprocal (1 ulp) is
    // within 2^-45 of the quotient, which lies at least 2^-36 from the middle of two
    // binary32 values (a 2^s = b k has no solution with k odd of 25 bits), so it is
    // the IEEE quotient; the fix-up step gives it for zeros, infinities and NaN.
    __device__ static float quotient(float a, float b)
    {
        if constexpr (FMT == FMT_FP16) {
            const float r = __builtin_amdgcn_rcpf(b);
            const float q = a * r;
            const float rem = __builtin_fmaf(-b, q, a);
            return __builtin_amdgcn_div_fixupf(__builtin_fmaf(rem, r, q), b, a);
        } else {
            return a / b;
        }
    }
    __device__ static T div(T a, T b, u32 rb) { return rnd16<FMT, SR_OPS, SHARED>(quotient(a, b), rb); }
    __device__ static T add(T a, T b, u32 rb)
    {
        if constexpr (NATIVE16)
            return (float)((_Float16)a + (_Float16)b);
        else
            return rnd16<FMT, SR_OPS, SHARED>(add32<FMT>(a, b), rb);
    }
    __device__ static A acc(A s, T a, u32 rb)
    {
        if constexpr (UNIF && FMT == FMT_FP16 && !SR_ACC)
            return (float)((_Float16)s + (_Float16)a);
        else
            return UNIF ? rnd16<FMT, SR_ACC, SHARED>(add32<FMT>(s, a), rb) : add32<FMT>(s, a);
    }
    // The same with a 1 that the compiler cannot see: s + 1 a in one rounding is the
    // sum, and the mixed multiply-add takes fp16 operands without their conversion
    // (which folds into a sum with a plain 1).
    __device__ static A acc(A s, T a, u32 rb, float one)
    {
        if constexpr (FMT == FMT_FP16 && SR_ACC) {
            const float v = __builtin_fmaf(a, one, s);
            return UNIF ? rnd16<FMT, SR_ACC, SHARED>(v, rb) : v;
        } else {
            return acc(s, a, rb);
        }
    }
    __device__ static A arnd(A v, u32 rb) { return UNIF ? rnd16<FMT, SR_OPS, SHARED>(v, rb) : v; }
    __device__ static A tacc(A v, u32 rb) { return UNIF ? rnd16<FMT, SR_ACC, SHARED>(v, rb) : v; }
    // -ln(u1) / a0. With fp16 propensities a0 lies in [2^-24, 2^22] whenever
    // the event can fire (any other value only sets a status), and
    // -ln(u1) in {0} or [2^-24, 16.7]: the short division applies.
    __device__ static A tau_div(A l, A a0)
    {
        if constexpr (FMT == FMT_FP16 && UNIF)   // both rounded to fp16
            return quotient(l, a0);
        else if constexpr (FMT == FMT_FP16)
            return div_rn_inrange(l, a0);
        else
            return l / a0;
    }
};

// --------------------------------------------------------------------------
// Random fields of one event. A string of bits is cut into B-bit fields from
// its low end (field r = bits [rB, rB + B), spanning two words when it must).
// Pool (main slots): the 80-bit string w[0..2] = (stream-0 word 2, word 3,
// low bytes of words 0 and 1) holds F0 = floor(80/B) fields; each further
// stream's 128-bit string (4 words) holds F1 = floor(128/B). ConvPool
// (conversion slots): F1 fields per stream 2^31 + q. hw(s) is the SR
// conversions' random operand for slot s: the field in bits 31..32-B (the
// instructions read only those; the bits below are don't-cares). Slot numbers
// are compile-time constants, so each hw is one shift or one funnel shift.
// --------------------------------------------------------------------------
template <int B>
__device__ __forceinline__ u32 field_operand(const u32 *w, int off)
{
    const int wi = off / 32, p = off % 32;
    if (p + B <= 32)
        return w[wi] << (32 - B - p);
    return __builtin_amdgcn_alignbit(w[wi + 1], w[wi], p + B - 32);
}

template <int NSLOT, int B>
struct Pool {
    static constexpr int F0 = 80 / B, F1 = 128 / B;
    static constexpr int NSTREAM = NSLOT <= F0 ? 1 : 1 + (NSLOT - F0 + F1 - 1) / F1;
    static constexpr int NW = NSLOT <= 0 ? 1 : 3 + 4 * (NSTREAM - 1);
    u32 w[NW];
    // slots past the pool belong to ops that do not round stochastically
    __device__ __forceinline__ u32 hw(int s) const
    {
        if (s >= NSLOT)
            return 0u;
        if (s < F0)
            return field_operand<B>(w, s * B);
        return field_operand<B>(w + 3 + 4 * ((s - F0) / F1), ((s - F0) % F1) * B);
    }
};

#define SSA_CONV_STREAM 0x80000000u

template <int NCONV, int B>
struct ConvPool {
    static constexpr int F1 = 128 / B;
    static constexpr int NSTREAM = NCONV <= 0 ? 0 : (NCONV + F1 - 1) / F1;
    u32 w[NSTREAM > 0 ? 4 * NSTREAM : 1];
    __device__ __forceinline__ u32 hw(int s) const
    {
        if (s >= NCONV)
            return 0u;
        return field_operand<B>(w + 4 * (s / F1), (s % F1) * B);
    }
};

// Conversion fields of event n (drawn only when a count is not exactly representable).
template <int NCONV, int B, class Gen>
__device__ __forceinline__ ConvPool<NCONV, B> make_conv(const Gen &gen, u64 n)
{
    ConvPool<NCONV, B> cp;
#pragma unroll
    for (int q = 0; q < ConvPool<NCONV, B>::NSTREAM; ++q) {
        W4 r = gen(n, SSA_CONV_STREAM + (u32)q);
        cp.w[4 * q + 0] = r.w0;
        cp.w[4 * q + 1] = r.w1;
        cp.w[4 * q + 2] = r.w2;
        cp.w[4 * q + 3] = r.w3;
    }
    return cp;
}

// A conversion pool for runs whose conversions need no random bits.
struct NoConv {
    __device__ __forceinline__ u32 hw(int) const { return 0u; }
};

// --------------------------------------------------------------------------
// Everything an event takes from its random numbers alone: the rounding
// halfword pool, -ln(u1) (rounded once in uniform mode) and u2. It depends on
// (seed, trajectory, event index) only, so the kernel forms event n+1's draw
// while event n's state-dependent chain runs.
// --------------------------------------------------------------------------
template <class P, int NSLOT>
struct Draw {
    Pool<NSLOT, P::SR_B> pool;
    typename P::A L;
    typename P::A u2;
};

template <class P, int NSLOT, int SLOT_LOG, class Gen>
__device__ __forceinline__ Draw<P, NSLOT> make_draw(const Gen &gen, u64 n, const DrawConst &k = DrawConst())
{
    Draw<P, NSLOT> d;
    W4 r0 = gen(n, 0u);
    if constexpr (NSLOT > 0) {
        d.pool.w[0] = r0.w2;
        d.pool.w[1] = r0.w3;
        d.pool.w[2] = (r0.w0 & 0xFFu) | ((r0.w1 & 0xFFu) << 8);
#pragma unroll
        for (int q = 1; q < Pool<NSLOT, P::SR_B>::NSTREAM; ++q) {
            W4 rq = gen(n, (u32)q);
            d.pool.w[3 + 4 * (q - 1) + 0] = rq.w0;
            d.pool.w[3 + 4 * (q - 1) + 1] = rq.w1;
            d.pool.w[3 + 4 * (q - 1) + 2] = rq.w2;
            d.pool.w[3 + 4 * (q - 1) + 3] = rq.w3;
        }
    }
    if constexpr (P::WIDE) {
        d.L = neg_log64(unif53(r0.w0, r0.w1, k), k);
        d.u2 = unif53(r0.w2, r0.w3, k);
    } else {
        d.L = P::arnd(neg_log32(unif24(r0.w0, k), k), d.pool.hw(SLOT_LOG));
        d.u2 = unif24(r0.w1, k);
    }
    return d;
}

// --------------------------------------------------------------------------
// Launch arguments.
// --------------------------------------------------------------------------
struct ItemArgs {
    const void *rates;       // [n_sets][M] constants in the mode's type (T)
    const void *hill;        // [M][2] (b_j, K_j) in T, Hill reactions only
    const i32 *x0;           // [N]
    i32 *snap;               // [k_hi - k_lo][N][E] snapshot rows of this launch
    u64 *n_events;           // [E]
    double *t_last;          // [E]
    unsigned char *status;   // [E]; 255 = suspended at a chunk boundary
    i32 *cx;                 // carry [N][E] (chunked runs)
    double *ct;              // carry clock [E]
    u64 *cn;                 // carry event index [E]
    i32 *ck;                 // carry next snapshot index [E]
    float *cm;               // carry running maximum [E]
    u32 *counter;            // work counter of this item (starts at 0)
    const u32 *order;        // claim order: trajectory of the w-th claim (NULL: w itself)
    u32 *work;               // events each trajectory fired in this launch (NULL: not recorded)
    double *rec_t;           // event record [E][rec_cap]: clock after each recorded firing
    unsigned char *rec_j;    // [E][rec_cap]: the reaction
    u32 *rec_n;              // [E]: recorded firings so far (also carried between chunks)
    u32 E;                   // trajectories
    u32 traj_per_set;        // trajectories per rate set (0: one set)
    u32 id_base;             // Philox trajectory id of trajectory 0
    u32 rec_cap;             // records kept per trajectory
    // pipelined kernels: the i-th item's turn is the item that comes i-th, and its
    // first_wg the first workgroup that starts there
    u32 turn, first_wg;
};

struct LaunchArgs {
    const double *snap_t64;  // [K]
    const float *snap_t32;   // [K]
    double t_end64;
    float t_end32;
    i32 K;
    i32 k_lo, k_hi;          // snapshot rows written by this launch
    i32 first, last;         // first / last chunk of the run
    u32 seed_lo, seed_hi;
    u32 place;               // PLACE_* bits (single-item launches of ssa_kernel)
    u32 guard;               // 1: a constant is so large that zero guards matter (pipelined kernel)
    u32 pipe_words;          // words of the pipelined kernel's ring and tables (dynamic LDS)
    u32 pipe_half;           // workgroups from this one on are the second of their CU
    u64 max_events;          // 0 = no cap
    ItemArgs item[SSA_N_ITEMS];
};

// Placement of work in a launch of ssa_kernel.
//   PLACE_WAVE_MAJOR: single-item launches take their first claims
//     statically, wave-major: claim slot r = c * gridDim.x + blockIdx.x of
//     wave c in its workgroup holds claims [64 r, 64 r + 64) of the claim
//     order (heaviest first after a reordering window), so the heaviest
//     trajectories sit on wave 0 of every workgroup; the work counter starts
//     past the static claims.
enum { PLACE_WAVE_MAJOR = 2u };

enum { ST_DONE = 0, ST_ABSORBED = 1, ST_OVERFLOW = 2, ST_CAPPED = 3, ST_SUSPENDED = 255 };

__device__ __forceinline__ u32 lane_id()
{
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

// Mask of the wave's lanes where c holds. Given one comparison, the mask is the
// comparison's own result; a conjunction is formed as the AND of its terms'
// masks (scalar ops), since a mask of a combined condition costs two dependent
// vector ops more.
__device__ __forceinline__ u64 lanes(bool c)
{
    return __builtin_amdgcn_ballot_w64(c);
}

// A wave-uniform value moved to a scalar register.
template <class V>
__device__ __forceinline__ V uniform_value(V v)
{
    if constexpr (sizeof(V) == 4) {
        return __builtin_bit_cast(V, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(u32, v)));
    } else {
        const u64 b = __builtin_bit_cast(u64, v);
        // readfirstlane returns a signed int: widen through u32, not by sign extension
        const u64 r = ((u64)(u32)__builtin_amdgcn_readfirstlane((u32)(b >> 32)) << 32) |
                      (u64)(u32)__builtin_amdgcn_readfirstlane((u32)b);
        return __builtin_bit_cast(V, r);
    }
}

__device__ __forceinline__ u32 rank_in(u64 mask)
{
    return __builtin_amdgcn_mbcnt_hi((u32)(mask >> 32), __builtin_amdgcn_mbcnt_lo((u32)mask, 0u));
}

template <class P>
__device__ __forceinline__ typename P::Tm snap_time(const LaunchArgs &L, int k)
{
    if constexpr (P::WIDE)
        return L.snap_t64[k];
    else
        return L.snap_t32[k];
}

// --------------------------------------------------------------------------
// Rounding slots of an event (Md: generated network description). With
// selective SR only the M-1 partial sums and the clock draw.
// --------------------------------------------------------------------------
template <class P, class Md>
struct Slots {
    static constexpr int M = Md::M;
    static constexpr int NSLOT = !P::SR ? 0
                                 : (P::SELECTIVE ? M : Md::NPROP + (P::UNI ? (P::NORM ? 2 * M + 4 : M + 3) : 0));
    static constexpr int NORM = Md::NPROP;
    static constexpr int SUM = P::SELECTIVE ? 0 : Md::NPROP + (P::NORM ? M : 0);
    static constexpr int LOG = SUM + M - 1;
    static constexpr int TAU = LOG + 1;
    static constexpr int TAUM = TAU + 1;
    static constexpr int TIME = P::SELECTIVE ? M - 1 : TAU + 1 + (P::NORM ? 1 : 0);
    static constexpr int TARGET = TIME + 1;
};

__device__ __forceinline__ void lgkm_wait()
{
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    __asm__ volatile("" ::: "memory");
}

__device__ __forceinline__ u32 lds_ld(const u32 *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void lds_st(u32 *p, u32 v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// --------------------------------------------------------------------------
// Propensity versions. Each computes the same values wherever it runs; a state
// needs one of them (wave-uniform, over the lanes holding a trajectory):
//   VER_EXACT    every count exactly representable in the propensity type (or
//                a binary type), none below a reactant order: no zero guard;
//   VER_GUARD    counts exact, some count below its order: zero guards;
//   VER_CONV     some count above the exact-integer limit (its conversion
//                rounds and draws conversion fields), zero guards;
//   VER_CONV_NG  the same with every count at or above its orders.
// The event loop runs one straight-line loop per version and leaves it when
// the updated state needs another, so a wave that stays in one version (a
// long trajectory far above the exact-integer limit) takes no branch but the
// loop's own each event. The loop test is one ballot for the states the
// version cannot compute; a move to a cheaper version waits for the next
// event that takes the rare path (a snapshot crossing, a fallback selection),
// which costs time, never results.
// --------------------------------------------------------------------------
enum { VER_EXACT = 0, VER_GUARD = 1, VER_CONV = 2, VER_CONV_NG = 3 };

template <int V>
struct IC {
    static constexpr int value = V;
};

template <class P, class Md>
struct Versions {
    static constexpr bool CONV = P::SR && !P::SELECTIVE && Md::NCONV > 0;
    static constexpr bool GUARD = Md::LO_MAX > 0;

    __device__ static __forceinline__ u32 max_count(const i32 (&x)[Md::N])
    {
        u32 mx = (u32)x[0];
#pragma unroll
        for (int s = 1; s < Md::N; ++s)
            mx = (u32)x[s] > mx ? (u32)x[s] : mx;
        return mx;
    }

    // as unsigned, a negative count (a network may allow one) only sends the wave
    // to a version that handles every count
    __device__ static __forceinline__ int of(const i32 (&x)[Md::N], u64 act)
    {
        if constexpr (CONV) {
            if ((act & lanes(Md::range_key(x) > (u32)(P::EXACT_INT - Md::LO_MAX))) == 0)
                return VER_EXACT;
            if ((act & lanes(max_count(x) > (u32)P::EXACT_INT)) == 0)
                return VER_GUARD;
            return (GUARD && (act & lanes(Md::below(x))) != 0) ? VER_CONV : VER_CONV_NG;
        } else if constexpr (GUARD) {
            return (act & lanes(Md::below(x))) == 0 ? VER_EXACT : VER_GUARD;
        } else {
            return VER_EXACT;
        }
    }

    // Lanes whose updated state version V cannot compute: a count above the
    // exact-integer limit where V converts without rounding, a count below a
    // reactant order where V has no zero guard. VER_CONV computes every state.
    // One ballot per version; leaving for a cheaper version (a state that no
    // longer needs V's extra work) is optional, and is tested on the rare path.
    template <int V>
    __device__ static __forceinline__ u64 must_leave(const i32 (&x)[Md::N], u64 act)
    {
        if constexpr (V == VER_EXACT) {
            if constexpr (CONV)
                return act & lanes(Md::range_key(x) > (u32)(P::EXACT_INT - Md::LO_MAX));
            else if constexpr (GUARD)
                return act & lanes(Md::below(x));
            else
                return 0;
        } else if constexpr (V == VER_GUARD) {
            if constexpr (CONV)
                return act & lanes(max_count(x) > (u32)P::EXACT_INT);
            else
                return 0;
        } else if constexpr (V == VER_CONV_NG) {
            if constexpr (GUARD)
                return act & lanes(Md::below(x));
            else
                return 0;
        } else {
            return 0;
        }
    }
};

// --------------------------------------------------------------------------
// One wave works through one item: lanes claim trajectories from the item's
// counter, run events, and claim again as they finish (ballot + prefix rank,
// one atomic per refill), until the counter passes E and every lane is idle.
// Md: generated network description; P: precision policy.
// --------------------------------------------------------------------------
template <class P, class Md, bool PER_LANE_RATES>
__device__ void run_item(const LaunchArgs &L, const ItemArgs &I, u32 slot_rank, u32 n_slots)
{
    typedef typename P::T T;
    typedef typename P::A A;
    typedef typename P::Tm Tm;
    typedef Slots<P, Md> S;
    typedef Versions<P, Md> VS;
    constexpr int N = Md::N, M = Md::M;
    constexpr int NSLOT = S::NSLOT;
    constexpr int SLOT_NORM = S::NORM;
    constexpr int SLOT_SUM = S::SUM;
    constexpr int SLOT_LOG = S::LOG;
    constexpr int SLOT_TAU = S::TAU;
    constexpr int SLOT_TAUM = S::TAUM;
    constexpr int SLOT_TIME = S::TIME;
    constexpr int SLOT_TARGET = S::TARGET;

    const T *rates = (const T *)I.rates;
    const T *hill = (const T *)I.hill;
    const Tm t_end = P::WIDE ? (Tm)L.t_end64 : (Tm)L.t_end32;
    const u32 lane = lane_id();

    // initialised: a lane without a trajectory still runs the event step on them
    i32 x[N] = {};
    T c[M] = {};
    Tm t = 0;
    u64 n = 0;
    i32 k = 0;
    Tm t_next = 0;     // time of snapshot k (infinity past the last row of this launch)
    Tm t_stop = 0;     // an event at t_new fires only if t_new <= t_stop (-infinity: suspend)
    Draw<P, NSLOT> cur = {};
    u64 n_claim = 0;   // event index when this launch claimed the trajectory
    u32 rec_cnt = 0;   // recorded firings of this trajectory (Md::REC reactions)
    const u64 n_stop = L.max_events ? L.max_events : ~0ull;
    float mrun = 0.0f;
    u32 idx = 0;
    bool active = false;
    bool open = true;

    if constexpr (!PER_LANE_RATES) {
        // one set for the item: wave-uniform, kept in scalar registers
#pragma unroll
        for (int j = 0; j < M; ++j)
            c[j] = uniform_value(rates[j]);
    }

    // wave-major static first claim (single-item launches): every lane is idle
    // at the start, so the wave's claim is its slot's 64 consecutive claims
    bool static_claim = SSA_N_ITEMS == 1 && (L.place & PLACE_WAVE_MAJOR) != 0u;
    const u32 dyn_base = static_claim ? n_slots * 64u : 0u;   // claims after the static ones
    for (;;) {
        if (open) {
            u64 need = __ballot(!active);
            if (need) {
                u32 cnt = (u32)__popcll(need);
                u32 leader = (u32)__ffsll((long long)need) - 1u;
                u32 base = 0;
                if (static_claim) {
                    base = slot_rank * 64u;
                    static_claim = false;
                } else {
                    if (lane == leader)
                        base = atomicAdd(I.counter, cnt);
                    base = __builtin_amdgcn_readlane(base, leader) + dyn_base;
                }
                if (!active) {
                    u32 w = base + rank_in(need);
                    if (w < I.E) {
                        u32 id = I.order ? I.order[w] : w;
                        idx = id;
                        active = true;
                        if constexpr (PER_LANE_RATES) {
                            u32 set = I.traj_per_set ? id / I.traj_per_set : 0u;
#pragma unroll
                            for (int j = 0; j < M; ++j)
                                c[j] = rates[(u64)set * M + j];
                        }
                        if (L.first) {
#pragma unroll
                            for (int s = 0; s < N; ++s)
                                x[s] = I.x0[s];
                            t = 0;
                            n = 0;
                            k = 0;
                            mrun = 0.0f;
                            rec_cnt = 0;
                        } else {
#pragma unroll
                            for (int s = 0; s < N; ++s)
                                x[s] = I.cx[(u64)s * I.E + id];
                            t = (Tm)I.ct[id];
                            n = I.cn[id];
                            k = I.ck[id];
                            mrun = I.cm[id];
                            if constexpr (Md::REC != 0)
                                rec_cnt = I.rec_n[id];
                            if (I.status[id] != ST_SUSPENDED) {
                                if (I.work)
                                    I.work[id] = 0u;
                                // finished in an earlier chunk: fill this chunk's rows
                                for (int kk = L.k_lo; kk < L.k_hi; ++kk)
#pragma unroll
                                    for (int s = 0; s < N; ++s)
                                        I.snap[((u64)(kk - L.k_lo) * N + s) * I.E + id] = x[s];
                                active = false;
                            }
                        }
                        t_next = k < L.k_hi ? snap_time<P>(L, k) : (Tm)SSA_INF_F;
                        t_stop = (!L.last && k >= L.k_hi) ? (Tm)(-SSA_INF_F) : t_end;
                        n_claim = n;
                        cur = make_draw<P, NSLOT, SLOT_LOG>(Philox{I.id_base + id, L.seed_lo, L.seed_hi}, n);
                    }
                }
                if (base + cnt >= I.E)
                    open = false;
            }
        }
        u64 act = lanes(active);   // the wave's lanes holding a trajectory
        if (act == 0) {
            if (!open)
                break;
            continue;
        }

        // Every lane runs the event step, also one without a trajectory: such a
        // lane never fires, stores nothing and leaves its registers unused, and
        // the step needs no exec-mask save and restore around it.
        for (;;) {
            // the last event's values, from which a stopping lane's status is read
            A a0 = 0;
            Tm t_new = 0;
            bool a_ok = false, m_ok = true, fire = false;
            u64 stop_lanes;
            // One event step in propensity version V; returns the lanes (or, for a
            // cheaper version, every lane) that make the wave choose its version again.
            auto step = [&](auto vtag) __attribute__((always_inline)) -> u64 {
                constexpr int V = decltype(vtag)::value;
                // ---- draws: cur belongs to event n; event n+1's is formed alongside
                const u32 id = I.id_base + idx;
                const Draw<P, NSLOT> nxt = make_draw<P, NSLOT, SLOT_LOG>(Philox{id, L.seed_lo, L.seed_hi}, n + 1);
                const Pool<NSLOT, P::SR_B> &pool = cur.pool;
                // ---- propensities (generated op sequence) in version V.
                // Conversions of counts draw random bits only when they round:
                // with every count exactly representable in the 16-bit type
                // no conversion stream is drawn. A mass-action propensity is
                // zero when a count is below its order; with every count at or
                // above its species' largest order no guard can apply.
                u64 cheaper = 0;
                T a[M];
                if constexpr (V == VER_EXACT) {
                    Md::template propensities<P, VS::CONV, false>(x, c, hill, a, pool, NoConv());
                } else if constexpr (V == VER_GUARD) {
                    Md::template propensities<P, VS::CONV, true>(x, c, hill, a, pool, NoConv());
                } else {
                    const ConvPool<Md::NCONV, P::SR_B> cpool =
                        make_conv<Md::NCONV, P::SR_B>(Philox{id, L.seed_lo, L.seed_hi}, n);
                    Md::template propensities<P, false, V == VER_CONV>(x, c, hill, a, pool, cpool);
                }
                // ---- optional running-max normalisation (uniform 16-bit)
                T m = (T)1;
                m_ok = true;
                if constexpr (P::NORM) {
                    float mx = 0.0f;
#pragma unroll
                    for (int j = 0; j < M; ++j)
                        mx = a[j] > mx ? a[j] : mx;
                    mrun = mx > mrun ? mx : mrun;
                    m_ok = mrun > 0.0f && mrun <= 3.40282347e38f;
                    m = mrun;
#pragma unroll
                    for (int j = 0; j < M; ++j)
                        a[j] = P::div(a[j], m, pool.hw(SLOT_NORM + j));
                }
                // ---- partial sums and total
                A S[M];
                S[0] = (A)a[0];
#pragma unroll
                for (int j = 1; j < M; ++j)
                    S[j] = P::acc(S[j - 1], a[j], pool.hw(SLOT_SUM + j - 1));
                a0 = S[M - 1];
                // a0 in (0, largest finite]: false for zero, negatives, infinity and NaN
                if constexpr (P::WIDE)   // positive finite binary64: bit patterns 1 .. 0x7FEFFFFFFFFFFFFF
                    a_ok = (u64)__double_as_longlong(a0) - 1ull < 0x7FEFFFFFFFFFFFFFull;
                else
                    a_ok = __float_as_uint(a0) - 1u < 0x7F7FFFFFu;
                a_ok = a_ok && m_ok;
                // ---- waiting time and clock (formed on every lane, used only if the event fires)
                if constexpr (P::UNI) {
                    A tau = P::arnd(P::tau_div(cur.L, a0), pool.hw(SLOT_TAU));
                    if constexpr (P::NORM)
                        tau = P::arnd(tau / m, pool.hw(SLOT_TAUM));
                    t_new = P::tacc(t + tau, pool.hw(SLOT_TIME));
                } else {
                    t_new = t + P::tau_div(cur.L, a0);
                }
                const u64 ok_lanes = act & lanes(a_ok);
                // ---- selection: mu = number of prefix sums at or below the target
                A target;
                if constexpr (P::UNI)   // binary32 product, then one rounding to the 16-bit type
                    target = P::arnd(f32_kept(cur.u2 * a0), pool.hw(SLOT_TARGET));
                else
                    target = cur.u2 * a0;
                int mu = 0;
#pragma unroll
                for (int j = 0; j < M; ++j)
                    mu += (S[j] <= target) ? 1 : 0;
                // ---- rare work behind one wave-uniform test (out of line): snapshots
                // strictly before t_new hold the current state; a target at or above
                // the total selects the last reaction with a positive propensity
                if (__builtin_expect((ok_lanes & (lanes(t_next < t_new) | lanes(mu == M))) != 0, 0)) {
                    __asm__ volatile("");
                    if (active && a_ok && t_next < t_new) {
                        do {
#pragma unroll
                            for (int s = 0; s < N; ++s)
                                I.snap[((u64)(k - L.k_lo) * N + s) * I.E + idx] = x[s];
                            ++k;
                            t_next = k < L.k_hi ? snap_time<P>(L, k) : (Tm)SSA_INF_F;
                        } while (t_next < t_new);
                        t_stop = (!L.last && k >= L.k_hi) ? (Tm)(-SSA_INF_F) : t_end;
                    }
                    if (active && a_ok && t_new <= t_stop && mu == M) {
                        int last_pos = 0;
#pragma unroll
                        for (int j = 0; j < M; ++j)
                            last_pos = (a[j] > (T)0) ? j : last_pos;
                        mu = last_pos;
                    }
                    // a cheaper version may serve the state now: leave after this event
                    // and choose again (a state V cannot compute is caught after the update)
                    if constexpr (V != VER_EXACT)
                        cheaper = lanes(VS::of(x, act) != V);
                }
                fire = active && a_ok && t_new <= t_stop;
                const u64 fire_lanes = ok_lanes & lanes(t_new <= t_stop);
                // ---- integer update (mu = M: nothing fires)
                Md::update(x, fire ? mu : M);
                t = fire ? t_new : t;
                n += 1;   // also where the event does not fire: such a lane stops, and is reset below
                if constexpr (Md::REC != 0) {
                    // event record: firings of the recorded reactions, with the clock after them
                    if (fire && ((Md::REC >> mu) & 1ull)) {
                        if (rec_cnt < I.rec_cap) {
                            I.rec_t[(u64)idx * I.rec_cap + rec_cnt] = (double)t;
                            I.rec_j[(u64)idx * I.rec_cap + rec_cnt] = (unsigned char)mu;
                        }
                        ++rec_cnt;
                    }
                }
                cur = nxt;   // a lane that stops here draws afresh when it claims again
                stop_lanes = act & (~fire_lanes | lanes(n == n_stop));
                return VS::template must_leave<V>(x, act) | cheaper;
            };
            // one straight-line loop per version; its first instruction on a
            // 64-byte boundary (where the taken back-branch lands decides how
            // many instruction-fetch lines an event spans; the same loop
            // measured up to 5% apart between offsets; the padding runs once)
            int ver = VS::of(x, act);
            for (;;) {
                u64 leave;
                if (ver == VER_EXACT) {
                    __asm__ volatile(".p2align 6");
                    do {
                        leave = step(IC<VER_EXACT>());
                    } while (__builtin_expect((stop_lanes | leave) == 0, 1));
                } else if (VS::GUARD && ver == VER_GUARD) {
                    if constexpr (VS::GUARD) {
                        __asm__ volatile(".p2align 6");
                        do {
                            leave = step(IC<VER_GUARD>());
                        } while (__builtin_expect((stop_lanes | leave) == 0, 1));
                    }
                } else if (VS::CONV && ver == VER_CONV_NG) {
                    if constexpr (VS::CONV) {
                        __asm__ volatile(".p2align 6");
                        do {
                            leave = step(IC<VER_CONV_NG>());
                        } while (__builtin_expect((stop_lanes | leave) == 0, 1));
                    }
                } else {
                    if constexpr (VS::CONV && VS::GUARD) {
                        __asm__ volatile(".p2align 6");
                        do {
                            leave = step(IC<VER_CONV>());
                        } while (__builtin_expect((stop_lanes | leave) == 0, 1));
                    }
                }
                if (stop_lanes != 0)
                    break;
                ver = VS::of(x, act);
            }
            if (active && (!fire || n == n_stop)) {
                if (!fire)
                    n -= 1;
                // ---- finish (or suspend) this trajectory, once per trajectory
                int status;
                if (!a_ok)
                    status = !m_ok ? (!(mrun <= 3.40282347e38f) ? ST_OVERFLOW : ST_ABSORBED)
                                   : (!(a0 <= (P::WIDE ? (A)1.7976931348623157e308 : (A)3.40282347e38f))
                                          ? ST_OVERFLOW
                                          : ST_ABSORBED);
                else if (!fire)
                    status = t_new > t_end ? ST_DONE : ST_SUSPENDED;
                else
                    status = ST_CAPPED;
                if (status != ST_SUSPENDED) {
                    for (; k < L.k_hi; ++k)
#pragma unroll
                        for (int s = 0; s < N; ++s)
                            I.snap[((u64)(k - L.k_lo) * N + s) * I.E + idx] = x[s];
                    I.n_events[idx] = n;
                    I.t_last[idx] = (double)t;
                }
                I.status[idx] = (unsigned char)status;
                if (I.work)
                    I.work[idx] = (u32)(n - n_claim);
                if constexpr (Md::REC != 0)
                    I.rec_n[idx] = rec_cnt;
                if (!L.last) {
#pragma unroll
                    for (int s = 0; s < N; ++s)
                        I.cx[(u64)s * I.E + idx] = x[s];
                    I.ct[idx] = (double)t;
                    I.cn[idx] = n;
                    I.ck[idx] = k;
                    I.cm[idx] = mrun;
                }
                active = false;
            }
            // leave to claim new trajectories once a lane stops (while any are
            // left), or when every lane has stopped
            act = lanes(active);
            if (open || act == 0)
                break;
        }
    }
}

// --------------------------------------------------------------------------
// Pipelined event loop (ssa_kernel_pl): one chain of events for 64
// trajectories per workgroup, its work divided among the workgroup's eight
// waves by what each part depends on.
//
//   event wave   propensities, partial sums, selection, integer update: the
//                only work whose result the next event waits for
//   clock wave   waiting times, clock, event records, the end of a trajectory and
//                the claim of the next one: it follows the event wave, which runs
//                ahead of it
//   row wave     snapshot rows: it follows the clock wave
//   draw waves   the random words, -ln(u1), u2 and conversion fields
//
// The waves pass batches of B events through an LDS ring of nb batches. Every
// lane takes one event per step, so a batch is wave-uniform: event e of batch
// b of a lane is event off + b B + e of its trajectory, and one counter per
// wave says how far it is:
//   next         batches handed to draw waves (each takes the next one)
//   ready[slot]  (batch + 1) << 2 | lanes restart << 1 | conversion fields made:
//                the batch's draws are in place
//   done_e       batches the event wave has finished: it leaves the totals a0,
//                the states or the selected reactions (and the running maximum)
//                in the slot
//   done_c       batches the clock wave has finished: it leaves the clock after
//                each event (infinity where every row left takes the state before
//                it, minus infinity past the end of a trajectory) and its lanes
//   done_s       batches the row wave has finished: batch b may be drawn once
//                b < done_s + nb, so a slot is free before it is written again
// Nothing the event wave does depends on the clock: past the end of a trajectory
// it computes events that nobody reads. The clock wave then claims the next
// trajectory for the lane, writes its id, off and state to the tables and posts
// {gen, sw}: from batch sw = done_c + nb on, the first one no draw wave can have
// started, the lane belongs to it. A draw wave takes the tables whenever gen has
// moved (what it draws for a lane between its two trajectories is not read), the
// event and row waves at batch sw, which the draw and clock waves mark. The next
// restart is posted once the row wave has finished batch sw.
// Every wait is for a counter of a wave that does not wait for the waiting one;
// `leave` ends all waits when the item has no trajectory left.
// Batch numbers have 64 bits: a lane that runs one trajectory for 2^32 batches meets
// the lower word of the last sw again. The counters carry lower words only, which is
// enough to tell batches of one ring apart. The draw and clock waves count the upper word;
// the event wave, which needs it in its careful path only, finds it in upper[the lower
// word's top bit], written by a draw wave 2^30 batches ahead (counted by the event wave in
// every batch it cost the open dimer sweep 0.6% in MIX_F16_SR).
// The tables of a lane are written while the other waves may read them (a draw wave
// whose batch lies before sw, the event wave's careful path): such a lane holds no
// trajectory in the batches that they work on, so nobody reads what they make of it,
// and a draw wave takes the tables again once it sees the new gen.
//
// With a CU to itself a workgroup is bound by the event wave's chain, whose length is
// its instructions (one wave issues one in about 5 cycles): Schloegl, 64 trajectories,
// cycles an event: 163 in FP64, 243 in MIX_F16_SR, 381 in MIX_BF16_SR, where one wave
// for all of an event took 840 in FP64 and one with its draws made elsewhere 510.
// With two workgroups to a CU the vector units are the bound: busy in 96% of the cycles
// in FP64, 87-93% in MIX_F16_SR (262k trajectories; 200 cycles a step of 64 events and
// CU on Schloegl, 161 and 180 on the dimer).
// --------------------------------------------------------------------------
typedef u32 v4u __attribute__((ext_vector_type(4)));
typedef u32 v2u __attribute__((ext_vector_type(2)));

constexpr int kPipeBatches = 16;   // most batches of a ring
constexpr int kSnapTable = 512;    // snapshot times kept in LDS

struct __attribute__((aligned(16))) PipeCtl {
    u32 ready[kPipeBatches];
    u32 lanes[4 * kPipeBatches];   // clock to row wave: {lanes, restart} of a batch
    u32 done_e, done_c, done_s, next;
    u32 gen, convw, leave, sw[2];   // sw: lower and upper word
    u32 upper[2];   // of the batches whose lower word begins with 0, with 1
    u32 rmask[2];   // lanes that start a trajectory at batch sw
    u32 live[2];    // lanes that hold one from batch sw on
};

template <bool C, class X, class Y>
struct Choose {
    typedef X type;
};
template <class X, class Y>
struct Choose<false, X, Y> {
    typedef Y type;
};

// Words that NW words of a lane take in LDS: 16-byte units [unit][lane], then the
// rest as 4- or 8-byte units (three words take a 16-byte unit).
__host__ __device__ constexpr int lds_words(int nw)
{
    return nw + (nw % 4 == 3 ? 1 : 0);
}

// words of `streams` generator calls that hold n fields of b bits at most f a call
__host__ __device__ constexpr int field_words(int n, int b, int f)
{
    return n <= 0 ? 0 : 4 * ((n - 1) / f) + (((n - 1) % f + 1) * b + 31) / 32;
}

// A slot's layout (PipeGeom::O_*, in words). First the events' pool words and u2
// (or u2 alone), read by the event wave only; its results take the same place: a0,
// the running maximum, then the states before each event (STATES) or the state
// before the batch and the selected reactions. After them L, the clock wave's
// rounding fields and the conversion words. After the ring's slots: the tables of
// a restart (T_*).
template <class P, class Md, bool HALF>
struct PipeGeom {
    typedef Slots<P, Md> S;
    static constexpr int NA = (int)(sizeof(typename P::A) / 4);
    static constexpr int NSLOT = S::NSLOT;
    static constexpr bool POOL = NSLOT > 0;
    static constexpr bool CONV = P::SR && !P::SELECTIVE && Md::NCONV > 0;
    // pool words that hold fields (80 bits of stream 0, then whole streams)
    static constexpr int F0 = 80 / P::SR_B, F1 = 128 / P::SR_B;
    // fp16 with a CU to one workgroup: the draw waves, which wait most of the time there,
    // pack the event wave's fields two to a word, which leaves it one shift for two
    static constexpr bool PACK = !HALF && POOL && P::SR_B == 13;
    static constexpr int NEF = P::UNI ? S::LOG + 1 : NSLOT;   // its fields (the last: the target's)
    static constexpr int NPW = !POOL ? 0 : PACK ? (NEF + 1) / 2 : 3 + field_words(NSLOT - F0, P::SR_B, F1);
    // the slot of packed field f
    static constexpr int field_slot(int f) { return P::UNI && f == S::LOG ? S::TARGET : f; }
    struct EventPool {
        u32 w[NPW > 0 ? NPW : 1];
        __device__ __forceinline__ u32 hw(int s) const
        {
            if constexpr (PACK) {
                const int f = P::UNI && s >= S::LOG ? S::LOG : s;
                return f >= NEF ? 0u : f % 2 ? w[f / 2] << 16 : w[f / 2];
            } else {
                Pool<NSLOT, P::SR_B> p;
#pragma unroll
                for (int k = 0; k < NPW; ++k)
                    p.w[k] = w[k];
                return p.hw(s);
            }
        }
    };
    static constexpr int EW = NPW + 1;                                                     // with u2 (POOL)
    static constexpr int CW = CONV ? field_words(Md::NCONV, P::SR_B, F1) : 0;
    // rounding fields of the clock: waiting time, its quotient by the maximum, the
    // clock; two to a word
    static constexpr int NF = P::UNI && POOL ? (P::SELECTIVE ? 1 : P::NORM ? 3 : 2) : 0;
    static constexpr int FW = (NF + 1) / 2;
    // few species: the event wave stores every state (one LDS instruction per four
    // events and species) and needs no reaction index; more, or an event record:
    // it stores the reactions and the clock wave replays them where it must
    static constexpr bool STATES = Md::N <= 3 && Md::REC == 0;
    static constexpr int mu_bits()
    {
        int w = 1;
        while ((1 << w) <= Md::M)
            ++w;
        return w;
    }
    static constexpr int MUB = mu_bits();
    static constexpr int MUPER = 32 / MUB;   // selected reactions per word
    static constexpr int mu_words(int b) { return (b + MUPER - 1) / MUPER; }
    static constexpr int draw_words(int b) { return POOL ? b * lds_words(EW) : lds_words(b * NA); }
    static constexpr int result_words(int b)
    {
        return lds_words(b * NA) + (P::NORM ? lds_words(b) : 0) +
               (STATES ? Md::N * lds_words(b) : Md::N + mu_words(b));
    }
    static constexpr int front_words(int b)
    {
        return draw_words(b) > result_words(b) ? draw_words(b) : result_words(b);
    }
    static constexpr int slot_words(int b)
    {
        return 64 * (front_words(b) + lds_words(b * NA) + lds_words(b * FW) + b * lds_words(CW));
    }
    static constexpr int TABLE = 64 * (6 + Md::N + Md::M * NA);
    static constexpr bool fits(int b, int n, int bytes) { return 4 * (n * slot_words(b) + TABLE) <= bytes; }
    // Batch length B: what a wave does once a batch is shared by B events, and the
    // event wave's straight-line code is that long. One workgroup to a CU (!HALF): the
    // longest that leaves a ring of five batches. Two to a CU (HALF): four at most, with
    // six, so that the draw waves keep several in hand (telegraph, 262k trajectories,
    // 101 rows: UNI_BF16_SR 3.5 ms with six of four and 3.9 with eleven of two,
    // UNI_F16_SR_NORM 4.8 with five of four and 4.5 with eleven of two).
    static constexpr int pick()
    {
        for (int b = HALF ? 4 : Md::M <= 12 ? 8 : Md::M <= 32 ? 4 : 2; b >= 2; b /= 2)
            if (fits(b, HALF ? 6 : 5, Md::pipe_lds(HALF)))
                return b;
        return fits(2, 4, Md::pipe_lds(HALF)) ? 2 : 0;
    }
    static constexpr bool OK = pick() != 0;
    static constexpr int B = OK ? pick() : 2;
    static constexpr int MUW = mu_words(B);
    static constexpr int SLOT = slot_words(B);
    static constexpr int O_EV = 0, EVS = 64 * lds_words(EW);   // one event's words to the next
    static constexpr int O_A = 0;
    static constexpr int O_M = O_A + 64 * lds_words(B * NA);
    static constexpr int O_X = O_M + (P::NORM ? 64 * lds_words(B) : 0);
    static constexpr int XS = 64 * lds_words(B);               // one species' states to the next
    static constexpr int O_MU = O_X + 64 * Md::N;              // (!STATES)
    static constexpr int O_L = 64 * front_words(B);
    static constexpr int O_F = O_L + 64 * lds_words(B * NA);
    static constexpr int O_CV = O_F + 64 * lds_words(B * FW), CVS = 64 * lds_words(CW);
    static constexpr int T_ID = 0, T_LO = 64, T_HI = 128, T_M = 192, T_K = 256, T_IDX = 320, T_X = 384;
    static constexpr int T_C = T_X + 64 * Md::N;
    __device__ static u32 batches(u32 words)   // of a ring in an LDS array of so many words
    {
        const u32 n = (words - (u32)TABLE) / (u32)SLOT;
        return n < (u32)kPipeBatches ? n : (u32)kPipeBatches;
    }
};

// what the waves of a workgroup share for one item
struct PipeWg {
    PipeCtl *ctl;
    u32 *ring;      // nb slots
    u32 *tab;       // per-lane tables
    u32 nb;         // batches of the ring
    const u32 *snap_t;   // the first kSnapTable snapshot times of this launch's rows
};

// NW words of a lane in the layout of lds_words: consecutive lanes on consecutive
// banks, one LDS instruction per four words
template <int NW>
__device__ __forceinline__ void put_words(u32 *p, u32 lane, const u32 *w)
{
#pragma unroll
    for (int q = 0; q < NW / 4; ++q)
        *(v4u *)(p + 256 * q + 4 * lane) = (v4u){w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]};
    constexpr int r = NW % 4, q = NW / 4;
    if constexpr (r == 1)
        p[256 * q + lane] = w[4 * q];
    else if constexpr (r == 2)
        *(v2u *)(p + 256 * q + 2 * lane) = (v2u){w[4 * q], w[4 * q + 1]};
    else if constexpr (r == 3)
        *(v4u *)(p + 256 * q + 4 * lane) = (v4u){w[4 * q], w[4 * q + 1], w[4 * q + 2], 0u};
}

template <int NW>
__device__ __forceinline__ void get_words(const u32 *p, u32 lane, u32 *w)
{
#pragma unroll
    for (int q = 0; q < (NW + 1) / 4; ++q) {
        const v4u v = *(const v4u *)(p + 256 * q + 4 * lane);
        w[4 * q] = v.x;
        w[4 * q + 1] = v.y;
        w[4 * q + 2] = v.z;
        if (4 * q + 3 < NW)
            w[4 * q + 3] = v.w;
    }
    constexpr int r = NW % 4, q = NW / 4;
    if constexpr (r == 1) {
        w[4 * q] = p[256 * q + lane];
    } else if constexpr (r == 2) {
        const v2u v = *(const v2u *)(p + 256 * q + 2 * lane);
        w[4 * q] = v.x;
        w[4 * q + 1] = v.y;
    }
}

template <class A>
__device__ __forceinline__ A value_at(const u32 *w, int i)
{
    if constexpr (sizeof(A) == 4)
        return __builtin_bit_cast(A, w[i]);
    else
        return __builtin_bit_cast(A, ((u64)w[2 * i + 1] << 32) | (u64)w[2 * i]);
}

template <class A>
__device__ __forceinline__ void value_to(u32 *w, int i, A v)
{
    if constexpr (sizeof(A) == 4) {
        w[i] = __builtin_bit_cast(u32, v);
    } else {
        const u64 b = __builtin_bit_cast(u64, v);
        w[2 * i] = (u32)b;
        w[2 * i + 1] = (u32)(b >> 32);
    }
}

// a0 in (0, largest finite]
template <class P>
__device__ __forceinline__ bool total_ok(typename P::A a0)
{
    if constexpr (P::WIDE)   // positive finite binary64: bit patterns 1 .. 0x7FEFFFFFFFFFFFFF
        return (u64)__double_as_longlong(a0) - 1ull < 0x7FEFFFFFFFFFFFFFull;
    else
        return __float_as_uint(a0) - 1u < 0x7F7FFFFFu;
}

// Whether the clock's short division gives the IEEE quotient for the total a0
// (and the total can fire): its exponent is in [-500, 500) (binary64), [-60, 60)
// (binary32), where the compiler's division sequence scales neither operand and
// its fix-up changes nothing. -ln(u1) is 0 or in [2^-53, 37], [2^-24, 17].
template <class P>
__device__ __forceinline__ bool total_mid(typename P::A a0)
{
    if constexpr (P::WIDE)
        return (u32)((u64)__double_as_longlong(a0) >> 32) - 0x20B00000u < 0x3E800000u;
    else
        return __float_as_uint(a0) - 0x21800000u < 0x3C000000u;
}

template <class P>
__device__ __forceinline__ typename P::A wait_mid(typename P::A l, typename P::A a0)
{
    if constexpr (P::WIDE)
        return div_rn_log64(l, a0);
    else if constexpr (P::NARROW && P::UNI)
        return P::tau_div(l, a0);
    else
        return div_rn_inrange(l, a0);
}

// every LDS access before it has completed, none after it has started
__device__ __forceinline__ void lds_fence()
{
    __asm__ volatile("" ::: "memory");
    lgkm_wait();
}

// c ? a : b as one select of its own: left to itself the compiler folds a tree of
// selects of +-1 into flags, a comparison and one more select
__device__ __forceinline__ i32 pick(bool c, i32 a, i32 b)
{
    i32 v = c ? a : b;
    __asm__("" : "+v"(v));
    return v;
}

// whether this lane is in the mask
__device__ __forceinline__ bool in_mask(u64 m)
{
    return __builtin_amdgcn_inverse_ballot_w64(m);
}

// a uniform LDS word
__device__ __forceinline__ u32 ctl_ld(const u32 *p)
{
    return (u32)__builtin_amdgcn_readfirstlane(lds_ld(p));
}

// ------------------------------------------------------------ draw waves
// Bound by vector instructions, 88 a draw in FP64 (100 before PhiloxNear, DrawConst and
// the shorter uniform and logarithm: dimer, 262k trajectories, 3.47 and 3.15 ms) and 78
// in MIX_F16_SR, of which the generator takes 37. Four draws are formed together, five
// waves share the batches: a lone event wave needs four of them in FP64.
template <class P, class Md, bool HALF>
__device__ void pipe_draw(const LaunchArgs &L, const PipeWg &W)
{
    typedef PipeGeom<P, Md, HALF> G;
    typedef Slots<P, Md> S;
    typedef typename P::A A;
    constexpr int B = G::B, NA = G::NA;
    constexpr int GR = B < 4 ? B : 4;   // draws formed together: their chains overlap
    const u32 lane = lane_id();
    PipeCtl *ctl = W.ctl;
    u32 gen = 0, id = 0, si = 0;
    u64 off = 0, b64 = 0, sw = 0;
    DrawConst con;
    con.pin();
    for (;;) {
        u32 nb = 0;
        if (lane == 0)
            nb = __hip_atomic_fetch_add(&ctl->next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const u32 b = (u32)__builtin_amdgcn_readfirstlane(nb);
        const u32 step = b - (u32)b64;
        b64 += (u64)step;
        si += step;
        while (si >= W.nb)   // b mod nb
            si -= W.nb;
        for (;;) {
            const u32 dc = lds_ld(&ctl->done_s), lv = lds_ld(&ctl->leave);
            if ((u32)__builtin_amdgcn_readfirstlane(lv) != 0u)
                return;
            if ((i32)(b - (u32)__builtin_amdgcn_readfirstlane(dc)) < (i32)W.nb)
                break;
            __builtin_amdgcn_s_sleep(1);
        }
        lds_fence();   // the restart of a batch is posted before the count that frees its slot
        const u32 g = ctl_ld(&ctl->gen);
        const bool conv = G::CONV && ctl_ld(&ctl->convw) != 0u;
        lds_fence();
        if (g != gen) {
            gen = g;
            sw = ((u64)ctl_ld(&ctl->sw[1]) << 32) | ctl_ld(&ctl->sw[0]);
            id = W.tab[G::T_ID + lane];
            off = ((u64)W.tab[G::T_HI + lane] << 32) | W.tab[G::T_LO + lane];
        }
        u32 *slot = W.ring + si * G::SLOT;
        const u64 n0 = off + b64 * B;
        const Philox any{id, L.seed_lo, L.seed_hi};
        auto draws = [&](const auto &rng) __attribute__((always_inline)) {
#pragma unroll
            for (int e0 = 0; e0 < B; e0 += GR) {
                Draw<P, S::NSLOT> d[GR];
#pragma unroll
                for (int e = 0; e < GR; ++e)
                    d[e] = make_draw<P, S::NSLOT, S::LOG>(rng, n0 + (u64)(e0 + e), con);
                u32 lw[GR * NA], uw[GR * NA];
#pragma unroll
                for (int e = 0; e < GR; ++e) {
                    value_to<A>(lw, e, d[e].L);
                    value_to<A>(uw, e, d[e].u2);
                }
                put_words<GR * NA>(slot + G::O_L + 64 * e0 * NA, lane, lw);
                if constexpr (G::POOL) {
#pragma unroll
                    for (int e = 0; e < GR; ++e) {
                        u32 w[G::EW];
#pragma unroll
                        for (int k = 0; k < G::NPW; ++k) {
                            if constexpr (G::PACK)
                                w[k] = (d[e].pool.hw(G::field_slot(2 * k)) & 0xFFFF0000u) |
                                       (2 * k + 1 < G::NEF ? d[e].pool.hw(G::field_slot(2 * k + 1)) >> 16 : 0u);
                            else
                                w[k] = d[e].pool.w[k];
                        }
                        w[G::NPW] = uw[e];
                        put_words<G::EW>(slot + G::O_EV + G::EVS * (e0 + e), lane, w);
                    }
                    if constexpr (G::NF > 0) {
                        u32 fw[GR * G::FW];
#pragma unroll
                        for (int e = 0; e < GR; ++e) {
                            const u32 time = d[e].pool.hw(S::TIME);
                            if constexpr (G::NF == 1) {
                                fw[e] = time;
                            } else {
                                fw[e * G::FW] = (time & 0xFFFF0000u) | (d[e].pool.hw(S::TAU) >> 16);
                                if constexpr (G::NF == 3)
                                    fw[e * G::FW + 1] = d[e].pool.hw(S::TAUM);
                            }
                        }
                        put_words<GR * G::FW>(slot + G::O_F + 64 * e0 * G::FW, lane, fw);
                    }
                } else {
                    put_words<GR * NA>(slot + G::O_EV + 64 * e0 * NA, lane, uw);
                }
            }
            if constexpr (G::CONV) {
                if (conv) {
#pragma unroll
                    for (int e = 0; e < B; ++e) {
                        const ConvPool<Md::NCONV, P::SR_B> cv = make_conv<Md::NCONV, P::SR_B>(rng, n0 + (u64)e);
                        put_words<G::CW>(slot + G::O_CV + G::CVS * e, lane, cv.w);
                    }
                }
            }
        };
        // no lane's event index carries into its upper word within the batch
        if (__builtin_expect(lanes((u32)n0 > 0u - (u32)B) == 0, 1))
            draws(PhiloxNear(any, (u32)(n0 >> 32)));
        else
            draws(any);
        if (__builtin_expect((b & 0x7FFFFFFFu) == 0x40000000u, 0))   // the other half is 2^30 batches off
            lds_st(&ctl->upper[(b >> 31) ^ 1u], (u32)(b64 >> 32) + (b >> 31));
        lds_fence();
        lds_st(ctl->ready + si, (b + 1u) << 2 | (b64 == sw ? 2u : 0u) | (conv ? 1u : 0u));
    }
}

// ------------------------------------------------------------ event wave
// The chain: bound by its own instructions, 32 (MIX_F16_SR Schloegl, fields packed) to
// 170 (UNI_F16_SR repressilator) an event, and about 200 cycles a batch.
template <class P, class Md, bool HALF, bool PER_LANE_RATES>
__device__ void pipe_events(const LaunchArgs &L, const ItemArgs &I, const PipeWg &W)
{
    typedef typename P::T T;
    typedef typename P::A A;
    typedef Slots<P, Md> S;
    typedef PipeGeom<P, Md, HALF> G;
    typedef typename Choose<G::PACK, typename P::Packed, P>::type PE;   // of the propensities and sums
    constexpr int N = Md::N, M = Md::M, B = G::B, NA = G::NA;
    constexpr int FW = G::POOL ? G::EW : B * NA;   // words loaded as a batch starts
    typedef ConvPool<Md::NCONV, P::SR_B> CP;
    const u32 lane = lane_id();
    PipeCtl *ctl = W.ctl;

    const T *rates = (const T *)I.rates;
    T hill[2 * M];
#pragma unroll
    for (int j = 0; j < 2 * M; ++j)
        hill[j] = uniform_value(((const T *)I.hill)[j]);
    i32 x[N] = {};
    T c[M] = {};
    if constexpr (!PER_LANE_RATES) {
#pragma unroll
        for (int j = 0; j < M; ++j)
            c[j] = uniform_value(rates[j]);
    }
    float mrun = 0.0f, one = 1.0f;
    __asm__ volatile("" : "+v"(one));
    u32 convw = 0, tag = 0;
    u64 live = 0;
    bool more = true;
    u64 over = 0;    // all lanes once the item has ended

    // Waits until batch b (slot `at`) is drawn; r: its ready word as read earlier. Once
    // the item has ended, `more` is false.
    auto acquire = [&](u32 b, u32 at, u32 r) __attribute__((always_inline)) {
        u32 v = (u32)__builtin_amdgcn_readfirstlane(r);
        if (__builtin_expect((v >> 2) != ((b + 1u) & 0x3FFFFFFFu), 0)) {
            for (;;) {
                const u32 r1 = lds_ld(ctl->ready + at), lv = lds_ld(&ctl->leave);
                v = (u32)__builtin_amdgcn_readfirstlane(r1);
                if ((v >> 2) == ((b + 1u) & 0x3FFFFFFFu))
                    break;
                if ((u32)__builtin_amdgcn_readfirstlane(lv) != 0u) {
                    more = false;   // (left by the rare branch after the batch)
                    over = ~0ull;
                    break;
                }
            }
        }
        tag = v;
        __asm__ volatile("" ::: "memory");
    };

    acquire(0u, 0u, 0u);
    if (!more)
        return;
    u32 si_next = 0;
    __asm__ volatile(".p2align 6");
    for (u32 b = 0;; ++b) {
        const u32 si = (u32)__builtin_amdgcn_readfirstlane(si_next);   // b mod nb
        u32 *slot = W.ring + si * G::SLOT;
        u32 first[FW];   // event 0's words, or every u2: in flight while the batch is looked over
        get_words<FW>(slot + G::O_EV, lane, first);
        if (__builtin_expect((tag & 2u) != 0u, 0)) {   // lanes take their next trajectory
            const u64 rm = ((u64)ctl_ld(&ctl->rmask[1]) << 32) | ctl_ld(&ctl->rmask[0]);
            live = ((u64)ctl_ld(&ctl->live[1]) << 32) | ctl_ld(&ctl->live[0]);
            if ((rm >> lane) & 1u) {
#pragma unroll
                for (int s = 0; s < N; ++s)
                    x[s] = (i32)W.tab[G::T_X + 64 * s + lane];
                mrun = __uint_as_float(W.tab[G::T_M + lane]);
                if constexpr (PER_LANE_RATES) {
#pragma unroll
                    for (int j = 0; j < M; ++j) {
                        u32 w[NA];
#pragma unroll
                        for (int k = 0; k < NA; ++k)
                            w[k] = W.tab[G::T_C + 64 * (j * NA + k) + lane];
                        c[j] = (T)value_at<A>(w, 0);
                    }
                }
            }
            lds_fence();   // waited for in here, not by every batch
        }
        i32 x0[N];
#pragma unroll
        for (int s = 0; s < N; ++s)
            x0[s] = x[s];
        const float m_start = mrun;
        const u32 si2 = si + 1u == W.nb ? 0u : si + 1u;
        const bool conv_made = (tag & 1u) != 0u;
        u64 again = L.guard != 0u ? ~0ull : 0ull;   // lanes whose batch has to be computed again with every case
        u32 aw[B * NA], mw[B], muw[G::MUW] = {}, xw[G::STATES ? N : 1][B];

        // The batch in straight line. KIND 0: every count within the exact-integer
        // limit; 1: conversions round, with the fields that came with the draws; 2:
        // every case (zero guards, conversion fields formed here, a target at or
        // above the total, partial sums that fall), from the state before the batch.
        auto batch = [&](auto kind) __attribute__((always_inline)) {
            constexpr int KIND = decltype(kind)::value;
            __asm__ volatile("; kind %0" ::"i"(KIND));   // (keeps the kinds' common loads in each)
            u32 uw[G::POOL ? 1 : B * NA];
            if constexpr (!G::POOL) {
#pragma unroll
                for (int k = 0; k < FW; ++k)
                    uw[k] = first[k];
            }
            u64 n = 0;
            u32 id = 0;
            if constexpr (KIND == 2) {
#pragma unroll
                for (int s = 0; s < N; ++s)
                    x[s] = x0[s];
                mrun = m_start;
                id = W.tab[G::T_ID + lane];
                n = (((u64)W.tab[G::T_HI + lane] << 32) | W.tab[G::T_LO + lane]) +
                    (((u64)ctl_ld(&ctl->upper[b >> 31]) << 32) | b) * B;
#pragma unroll
                for (int k = 0; k < G::MUW; ++k)
                    muw[k] = 0u;
            }
            u32 r2 = 0;
            u32 ew[G::POOL ? G::EW : 1];   // the next event's words, loaded while this one runs
            if constexpr (G::POOL) {
#pragma unroll
                for (int k = 0; k < FW; ++k)
                    ew[k] = first[k];
            }
#pragma unroll
            for (int e = 0; e < B; ++e) {
                typename G::EventPool pool;
                A u2;
                if constexpr (G::POOL) {
#pragma unroll
                    for (int k = 0; k < G::NPW; ++k)
                        pool.w[k] = ew[k];
                    u2 = value_at<A>(ew, G::NPW);
                    if (e + 1 < B)
                        get_words<G::EW>(slot + G::O_EV + G::EVS * (e + 1), lane, ew);
                } else {
                    u2 = value_at<A>(uw, e);
                }
                if ((KIND != 2 || Md::CAREFUL) && e == B / 2) {
                    // the last batch's words have long been written: publish it, and ask
                    // for the next one's state
                    __asm__ volatile("" : "+v"(x[0]));   // not before this event
                    lds_fence();
                    lds_st(&ctl->done_e, b);
                    r2 = lds_ld(ctl->ready + si2);
                }
                if ((KIND != 2 || Md::CAREFUL) && e == B - 1) {
                    __asm__ volatile("" : "+v"(r2), "+v"(x[0]));   // not before this event
                    acquire(b + 1u, si2, r2);
                }
                if constexpr (G::STATES) {
#pragma unroll
                    for (int s = 0; s < N; ++s)
                        xw[s][e] = (u32)x[s];
                }
                T a[M];
                if constexpr (G::CONV && KIND == 2) {
                    const CP cp = make_conv<Md::NCONV, P::SR_B>(Philox{id, L.seed_lo, L.seed_hi}, n + (u64)e);
                    Md::template propensities<PE, false, true>(x, c, hill, a, pool, cp);
                } else if constexpr (KIND == 2) {
                    Md::template propensities<PE, false, true>(x, c, hill, a, pool, NoConv());
                } else if constexpr (KIND == 1) {
                    CP cp;
                    get_words<G::CW>(slot + G::O_CV + G::CVS * e, lane, cp.w);
                    Md::template propensities<PE, false, Md::template needs_guard<PE>()>(x, c, hill, a, pool, cp);
                } else {
                    Md::template propensities<PE, G::CONV, Md::template needs_guard<PE>()>(x, c, hill, a, pool, NoConv());
                }
                if constexpr (P::NORM) {
                    float mx = 0.0f;
#pragma unroll
                    for (int j = 0; j < M; ++j)
                        mx = a[j] > mx ? a[j] : mx;
                    mrun = mx > mrun ? mx : mrun;
                    mw[e] = __float_as_uint(mrun);
#pragma unroll
                    for (int j = 0; j < M; ++j)
                        a[j] = PE::div(a[j], mrun, pool.hw(S::NORM + j));
                }
                A sum[M];
                sum[0] = (A)a[0];
#pragma unroll
                for (int j = 1; j < M; ++j)
                    sum[j] = PE::acc(sum[j - 1], a[j], pool.hw(S::SUM + j - 1), one);
                const A a0 = sum[M - 1];
                A target;
                if constexpr (P::UNI)
                    target = PE::arnd(f32_kept(u2 * a0), pool.hw(S::TARGET));
                else
                    target = u2 * a0;
                // past[j]: the reaction comes after j (partial sums never fall outside KIND 2,
                // so the first false one names it). A target rounded up to the total selects the
                // last reaction that can fire: the last of all, where that one can (a
                // 16-bit target is one in most bfloat16 batches and a fifth of the fp16
                // ones of 64 lanes and 8 events); else the batch is computed again.
                bool past[M];
#pragma unroll
                for (int j = 0; j < M; ++j)
                    past[j] = sum[j] <= target;
                if constexpr (KIND == 2) {
                    int mu = 0, last_pos = 0;
#pragma unroll
                    for (int j = 0; j < M; ++j) {
                        mu += past[j] ? 1 : 0;
                        last_pos = (a[j] > (T)0) ? j : last_pos;
                    }
                    mu = mu == M && total_ok<P>(a0) ? last_pos : mu;
                    Md::update(x, mu);
                    muw[e / G::MUPER] |= (u32)mu << (G::MUB * (e % G::MUPER));
                } else if constexpr (G::STATES) {
                    again |= lanes(past[M - 1]) & ~(P::UNI ? lanes(a[M - 1] > (T)0) : 0ull);
                    Md::advance(x, past);
                } else {
                    again |= lanes(past[M - 1]) & ~(P::UNI ? lanes(a[M - 1] > (T)0) : 0ull);
                    const int mu = Md::reaction(past);
                    Md::update(x, mu);
                    muw[e / G::MUPER] |= (u32)mu << (G::MUB * (e % G::MUPER));
                }
                value_to<A>(aw, e, a0);
            }
        };
        bool conv_now = false;
        if constexpr (G::CONV) {
            // counts grow by at most DMAX an event; the draw waves are asked for
            // conversion fields some batches before one reaches the limit
            constexpr int lim = P::EXACT_INT - (B - 1) * Md::DMAX, near = P::EXACT_INT - 96 * Md::DMAX;
            const u32 mx = Versions<P, Md>::max_count(x);
            const u64 close = near < 0 ? live : live & lanes(mx > (u32)near);
            if (__builtin_expect(close != 0 || convw != 0u, 0)) {
                const bool cv = lim < 0 ? live != 0 : (live & lanes(mx > (u32)lim)) != 0;
                const u32 want = close != 0 ? 1u : 0u;
                if (want != convw) {
                    convw = want;
                    lds_st(&ctl->convw, want);
                }
                if (cv && !conv_made)
                    again = ~0ull;
                conv_now = cv && conv_made;
            }
        }
        if constexpr (Md::CAREFUL) {
            batch(IC<2>());
            again = 0;
        } else if constexpr (G::CONV) {
            if (conv_now)
                batch(IC<1>());
            else
                batch(IC<0>());
        } else {
            batch(IC<0>());
        }
        if (__builtin_expect(((again & live) | over) != 0, 0)) {
            if (!more)
                return;
            if constexpr (!Md::CAREFUL)
                batch(IC<2>());
        }
        put_words<B * NA>(slot + G::O_A, lane, aw);
        if constexpr (P::NORM)
            put_words<B>(slot + G::O_M, lane, mw);
        if constexpr (G::STATES) {
#pragma unroll
            for (int s = 0; s < N; ++s)
                put_words<B>(slot + G::O_X + G::XS * s, lane, xw[s]);
        } else {
#pragma unroll
            for (int s = 0; s < N; ++s)
                slot[G::O_X + 64 * s + lane] = (u32)x0[s];
#pragma unroll
            for (int k = 0; k < G::MUW; ++k)
                slot[G::O_MU + 64 * k + lane] = muw[k];
        }
        si_next = si2;
    }
}

// ------------------------------------------------------------ clock wave
// Has slack: it waits for the event wave 10 to 60% of the time, least in FP64, where a
// division takes 8 instructions. Its rare work (ends, claims) is behind one test a batch.
template <class P, class Md, bool HALF, bool PER_LANE_RATES>
__device__ void pipe_clock(const LaunchArgs &L, const ItemArgs &I, const PipeWg &W)
{
    typedef typename P::T T;
    typedef typename P::A A;
    typedef typename P::Tm Tm;
    typedef Slots<P, Md> S;
    typedef PipeGeom<P, Md, HALF> G;
    constexpr int N = Md::N, M = Md::M, B = G::B, NA = G::NA;
    const u32 lane = lane_id();
    PipeCtl *ctl = W.ctl;
    const T *rates = (const T *)I.rates;
    const Tm t_end = P::WIDE ? (Tm)L.t_end64 : (Tm)L.t_end32;
    const u64 n_stop = L.max_events ? L.max_events : ~0ull;
    Tm t = 0, t_lim = 0;   // an event at t_new fires only if t_new <= t_lim
    Tm t_hold = 0;         // clock of a trajectory whose first batch is still to come
    u64 off = 0;           // event e of batch b is event off + b B + e
    u64 cap_b = 0;         // batches from here on hold the event cap
    u64 n_claim = 0;
    u32 idx = 0, rec_cnt = 0, gen = 0;
    u64 sw = 0;
    u64 act = 0, hold = 0;   // lanes in a trajectory, lanes waiting for batch sw
    bool open = true, pending = false, changed = false;
    // past the last row of this launch a trajectory is suspended (the last launch: ends)
    const Tm t_rows = L.last ? t_end : L.k_hi > L.k_lo ? snap_time<P>(L, L.k_hi - 1) : (Tm)(-SSA_INF_F);

    // trajectories for the lanes without one; their first batch is at_batch
    auto claim = [&](u64 at_batch) {
        u64 fresh = 0;
        while (open) {
            const u64 need = ~(act | hold);
            if (need == 0)
                break;
            const u32 cnt = (u32)__popcll(need);
            const u32 leader = (u32)__ffsll((long long)need) - 1u;
            u32 base = 0;
            if (lane == leader)
                base = atomicAdd(I.counter, cnt);
            base = __builtin_amdgcn_readlane(base, leader);
            bool run = false;
            if (in_mask(need)) {
                const u32 w = base + rank_in(need);
                if (w < I.E) {
                    const u32 id = I.order ? I.order[w] : w;
                    i32 x[N];
                    float mrun = 0.0f;
                    i32 k = 0;
                    run = true;
                    t_hold = 0;
                    n_claim = 0;
                    rec_cnt = 0;
                    if (L.first) {
#pragma unroll
                        for (int s = 0; s < N; ++s)
                            x[s] = I.x0[s];
                    } else {
#pragma unroll
                        for (int s = 0; s < N; ++s)
                            x[s] = I.cx[(u64)s * I.E + id];
                        t_hold = (Tm)I.ct[id];
                        n_claim = I.cn[id];
                        k = I.ck[id];
                        mrun = I.cm[id];
                        if constexpr (Md::REC != 0)
                            rec_cnt = I.rec_n[id];
                        if (I.status[id] != ST_SUSPENDED) {
                            if (I.work)
                                I.work[id] = 0u;
                            // finished in an earlier chunk: fill this chunk's rows
                            for (int kk = L.k_lo; kk < L.k_hi; ++kk)
#pragma unroll
                                for (int s = 0; s < N; ++s)
                                    I.snap[((u64)(kk - L.k_lo) * N + s) * I.E + id] = x[s];
                            run = false;
                        }
                    }
                    if (run) {
                        idx = id;
                        t_lim = !L.last && k >= L.k_hi ? (Tm)(-SSA_INF_F) : t_rows;
                        off = n_claim - at_batch * B;
                        cap_b = at_batch + (n_stop - n_claim) / (u64)B;
                        W.tab[G::T_K + lane] = (u32)k;
                        W.tab[G::T_IDX + lane] = id;
                        W.tab[G::T_ID + lane] = I.id_base + id;
                        W.tab[G::T_LO + lane] = (u32)off;
                        W.tab[G::T_HI + lane] = (u32)(off >> 32);
                        W.tab[G::T_M + lane] = __float_as_uint(mrun);
#pragma unroll
                        for (int s = 0; s < N; ++s)
                            W.tab[G::T_X + 64 * s + lane] = (u32)x[s];
                        if constexpr (PER_LANE_RATES) {
                            const u32 set = I.traj_per_set ? id / I.traj_per_set : 0u;
#pragma unroll
                            for (int j = 0; j < M; ++j) {
                                u32 w2[NA];
                                value_to<A>(w2, 0, (A)rates[(u64)set * M + j]);
#pragma unroll
                                for (int q = 0; q < NA; ++q)
                                    W.tab[G::T_C + 64 * (j * NA + q) + lane] = w2[q];
                            }
                        }
                    }
                }
            }
            fresh |= lanes(run);
            hold |= lanes(run);
            if (base + cnt >= I.E)
                open = false;
        }
        sw = at_batch;
        gen += 1u;
        lds_st(&ctl->rmask[0], (u32)fresh);
        lds_st(&ctl->rmask[1], (u32)(fresh >> 32));
        lds_st(&ctl->live[0], (u32)(act | hold));
        lds_st(&ctl->live[1], (u32)((act | hold) >> 32));
        lds_st(&ctl->sw[0], (u32)sw);
        lds_st(&ctl->sw[1], (u32)(sw >> 32));
        lds_fence();
        lds_st(&ctl->gen, gen);
        lds_fence();
        pending = true;
        changed = false;
    };

    claim(0);
    lds_st(&ctl->done_s, 0u);
    u32 si_next = 0, e_done = 0;
    u64 b = 0;
    // (the loop's first line decides 1 to 2% where this wave is the slower one: telegraph
    // with records, 665 trajectories, 0.642 and 0.638 ms)
    __asm__ volatile(".p2align 6");
    for (;; ++b) {
        if ((act | hold) == 0 && !open)
            break;   // the queue is empty and no lane runs
        const u32 bl = (u32)b;
        const u32 si = (u32)__builtin_amdgcn_readfirstlane(si_next);
        u32 *slot = W.ring + si * G::SLOT;
        if ((i32)(e_done - bl) <= 0) {
            // the event wave is behind: what the row wave waits for goes out first
            lds_fence();
            lds_st(&ctl->done_c, bl);
            for (;;) {
                e_done = ctl_ld(&ctl->done_e);
                if ((i32)(e_done - bl) > 0)
                    break;
                __builtin_amdgcn_s_sleep(1);
            }
            __asm__ volatile("" ::: "memory");
        }
        const bool restart = pending && bl == (u32)sw;   // (pending: at most a ring ahead)
        if (restart) {
            t = in_mask(hold) ? t_hold : t;
            act |= hold;
            hold = 0;
            pending = false;
        }
        // ---- the batch's clock values, as if every event fired
        u32 lw[B * NA], aw[B * NA], mw[P::NORM ? B : 1] = {};
        get_words<B * NA>(slot + G::O_L, lane, lw);
        get_words<B * NA>(slot + G::O_A, lane, aw);
        if constexpr (P::NORM)
            get_words<B>(slot + G::O_M, lane, mw);
        u32 fw[G::NF > 0 ? B * G::FW : 1] = {};
        if constexpr (G::NF > 0)
            get_words<B * G::FW>(slot + G::O_F, lane, fw);
        const u32 e_now = lds_ld(&ctl->done_e);
        lds_fence();   // with these words, what this wave wrote for the last batch is in place
        lds_st(&ctl->done_c, bl);
        e_done = (u32)__builtin_amdgcn_readfirstlane(e_now);
        Tm tn[B];
        u64 ok[B], mid = ~0ull;   // ok: lanes whose total (and running maximum) can fire event e
        auto clock = [&](auto full_range) __attribute__((always_inline)) {
            constexpr bool FULL = decltype(full_range)::value != 0;
#pragma unroll
            for (int e = 0; e < B; ++e) {
                const A a0 = value_at<A>(aw, e), l = value_at<A>(lw, e);
                const Tm before = e ? tn[e - 1] : t;
                const A wait = FULL ? P::tau_div(l, a0) : wait_mid<P>(l, a0);
                if constexpr (P::UNI) {
                    // fields in the upper halfword; below it are bits no conversion reads
                    const u32 f0 = G::NF > 0 ? fw[G::NF > 0 ? e * G::FW : 0] : 0u;
                    A tau = P::arnd(wait, f0 << 16);
                    if constexpr (P::NORM)
                        tau = P::arnd(P::quotient(tau, __uint_as_float(mw[e])),
                                      G::NF == 3 ? fw[G::NF == 3 ? e * G::FW + 1 : 0] : 0u);
                    tn[e] = P::tacc(before + tau, f0);
                } else {
                    tn[e] = before + wait;
                }
                if constexpr (FULL) {
                    ok[e] = lanes(total_ok<P>(a0));
                } else {
                    ok[e] = lanes(total_mid<P>(a0));
                }
                if constexpr (P::NORM)
                    ok[e] &= lanes(__uint_as_float(mw[e]) > 0.0f) & lanes(__uint_as_float(mw[e]) <= 3.40282347e38f);
                if constexpr (!FULL)
                    mid &= ok[e];
            }
        };
        clock(IC<0>());
        // no lane ends or reaches the cap: the clock moves on
        const u64 plain = mid & lanes(tn[B - 1] <= t_lim) & lanes(b < cap_b);
        const u64 was = act;
        const Tm t_before = t;
        if (Md::REC != 0 || (act & ~plain) != 0) {
            if ((act & ~mid) != 0)
                clock(IC<1>());
            t = tn[B - 1];
            u64 run = act;          // lanes still in their trajectory
            u32 stop_e = 0;         // the event a lane stops at (it does not fire)
            Tm t_at = 0, t_over = 0;
            A a_at = 0;
            float m_at = 1.0f;
            // rem: events until the cap, for lanes near it
            const u64 n0 = off + b * (u64)B;
            const u32 rem = b < cap_b ? (u32)B : (u32)(n_stop - n0);
#pragma unroll
            for (int e = 0; e < B; ++e) {
                const Tm t_new = tn[e];
                const u64 fire = run & ok[e] & lanes(t_new <= t_lim) & ~lanes(rem == (u32)e);
                const u64 stop = run & ~fire;
                if (Md::REC != 0) {
                    const int mu = (int)((slot[G::O_MU + 64 * (e / G::MUPER) + lane] >> (G::MUB * (e % G::MUPER))) &
                                         ((1u << G::MUB) - 1u));
                    if (in_mask(fire) && ((Md::REC >> mu) & 1ull)) {
                        if (rec_cnt < I.rec_cap) {
                            I.rec_t[(u64)idx * I.rec_cap + rec_cnt] = (double)t_new;
                            I.rec_j[(u64)idx * I.rec_cap + rec_cnt] = (unsigned char)mu;
                        }
                        ++rec_cnt;
                    }
                }
                if (stop) {
                    if (in_mask(stop)) {
                        stop_e = (u32)e;
                        t_at = e ? tn[e ? e - 1 : 0] : t_before;
                        t_over = t_new;
                        a_at = value_at<A>(aw, e);
                        m_at = P::NORM ? __uint_as_float(mw[P::NORM ? e : 0]) : 1.0f;
                    }
                    run = fire;
                }
            }
            const u64 ended = act & ~run;
            if (in_mask(ended)) {
                // what the row wave sees: a trajectory that stops in its state leaves it to
                // every row from here on, and nothing follows
                const bool frozen = rem == stop_e || !(t_over > t_lim) || !total_ok<P>(a_at) ||
                                    (P::NORM && !(m_at > 0.0f && m_at <= 3.40282347e38f));
#pragma unroll
                for (int e = 0; e < B; ++e)
                    tn[e] = (u32)e > stop_e ? (Tm)(-SSA_INF_F) : (u32)e == stop_e && frozen ? (Tm)SSA_INF_F : tn[e];
                i32 x[N];
                if constexpr (G::STATES) {
#pragma unroll
                    for (int s = 0; s < N; ++s)
                        x[s] = (i32)slot[G::O_X + G::XS * s +
                                         (B >= 4 ? 256 * (stop_e / 4u) + 4 * lane + stop_e % 4u : B * lane + stop_e)];
                } else {
#pragma unroll
                    for (int s = 0; s < N; ++s)
                        x[s] = (i32)slot[G::O_X + 64 * s + lane];
#pragma unroll
                    for (int e = 0; e < B; ++e) {
                        const u32 mu = (slot[G::O_MU + 64 * (e / G::MUPER) + lane] >> (G::MUB * (e % G::MUPER))) &
                                       ((1u << G::MUB) - 1u);
                        Md::update(x, (u32)e < stop_e ? (int)mu : M);
                    }
                }
                // ---- finish (or suspend) this trajectory, once per trajectory
                const u64 n = n0 + (u64)stop_e;
                const bool m_ok = !P::NORM || (m_at > 0.0f && m_at <= 3.40282347e38f);
                int status;
                if (rem == stop_e)
                    status = ST_CAPPED;
                else if (!m_ok)
                    status = !(m_at <= 3.40282347e38f) ? ST_OVERFLOW : ST_ABSORBED;
                else if (!total_ok<P>(a_at))
                    status = !(a_at <= (P::WIDE ? (A)1.7976931348623157e308 : (A)3.40282347e38f)) ? ST_OVERFLOW
                                                                                                  : ST_ABSORBED;
                else
                    status = t_over > t_end ? ST_DONE : ST_SUSPENDED;
                if (status != ST_SUSPENDED) {
                    I.n_events[idx] = n;
                    I.t_last[idx] = (double)t_at;
                }
                I.status[idx] = (unsigned char)status;
                if (I.work)
                    I.work[idx] = (u32)(n - n_claim);
                if constexpr (Md::REC != 0)
                    I.rec_n[idx] = rec_cnt;
                if (!L.last) {
#pragma unroll
                    for (int s = 0; s < N; ++s)
                        I.cx[(u64)s * I.E + idx] = x[s];
                    I.ct[idx] = (double)t_at;
                    I.cn[idx] = n;
                    I.ck[idx] = L.k_hi;
                    I.cm[idx] = P::NORM ? m_at : 0.0f;
                }
            }
            act = run;
            changed = changed || ended != 0;
        } else {
            t = tn[B - 1];
        }
        // for the row wave, in the place of L
        u32 tw[B * NA];
#pragma unroll
        for (int e = 0; e < B; ++e)
            value_to<A>(tw, e, (A)tn[e]);
        put_words<B * NA>(slot + G::O_L, lane, tw);
        *(v4u *)(ctl->lanes + 4 * si) = (v4u){(u32)was, (u32)(was >> 32), restart ? 1u : 0u, 0u};
        if (__builtin_expect(!pending && changed, 0)) {
            // the row wave's number: at most a ring behind this one
            if (b - (u64)(bl - ctl_ld(&ctl->done_s)) > sw)
                claim(b + W.nb);
        }
        si_next = si + 1u == W.nb ? 0u : si + 1u;
    }
    lds_fence();
    lds_st(&ctl->done_c, (u32)b);
    lds_fence();
    lds_st(&ctl->leave, 1u);
    lds_fence();
}

// ------------------------------------------------------------ row wave
// Mostly LDS latency: everything a batch may need is read in one go, and a batch without a
// row is one comparison. It holds the ring where rows are dense (telegraph in FP64, a row
// per 13 events and trajectory: 262k trajectories 1.2 ms with rows, 0.85 without).
template <class P, class Md, bool HALF>
__device__ void pipe_rows(const LaunchArgs &L, const ItemArgs &I, const PipeWg &W)
{
    typedef typename P::A A;
    typedef typename P::Tm Tm;
    typedef PipeGeom<P, Md, HALF> G;
    constexpr int N = Md::N, B = G::B, NA = G::NA;
    const u32 lane = lane_id();
    PipeCtl *ctl = W.ctl;
    Tm t_next = (Tm)SSA_INF_F, t_after = (Tm)SSA_INF_F;   // times of the lane's next two rows
    i32 *row = nullptr;                                   // where the next one goes
    i32 k = 0;
    // time of row r: from the LDS table, which ends with two infinities; past a table
    // that does not hold all of this launch's rows, from memory
    const bool all_rows = L.k_hi - L.k_lo <= kSnapTable;
    auto row_time = [&](i32 r) __attribute__((always_inline)) -> Tm {
        const i32 i = r - L.k_lo;
        Tm v = ((const Tm *)W.snap_t)[i <= kSnapTable ? i : kSnapTable + 1];
        if (__builtin_expect(!all_rows, 0)) {
            if (i >= kSnapTable)
                v = r < L.k_hi ? snap_time<P>(L, r) : (Tm)SSA_INF_F;
            // the wait for this load stays in here: where the paths join it would hold
            // for every row stored before
            __asm__ volatile("" : "+v"(v));
        }
        return v;
    };
    u32 si_next = 0, c_done = 0;
    for (u32 b = 0;; ++b) {
        const u32 si = (u32)__builtin_amdgcn_readfirstlane(si_next);
        while ((i32)(c_done - b) <= 0) {
            const u32 lv = lds_ld(&ctl->leave);
            __asm__ volatile("" ::: "memory");
            const u32 dc = lds_ld(&ctl->done_c);
            c_done = (u32)__builtin_amdgcn_readfirstlane(dc);
            if ((i32)(c_done - b) > 0)
                break;
            if ((u32)__builtin_amdgcn_readfirstlane(lv) != 0u)
                return;
            __builtin_amdgcn_s_sleep(1);
        }
        __asm__ volatile("" ::: "memory");
        const u32 *slot = W.ring + si * G::SLOT;
        // everything the batch may need in one go: most of its time is LDS latency
        u32 tw[B * NA], sw[G::STATES ? N : 1][B], x0[N], muw[G::MUW];
        get_words<B * NA>(slot + G::O_L, lane, tw);
        const v4u on = *(const v4u *)(ctl->lanes + 4 * si);
        if constexpr (G::STATES) {
#pragma unroll
            for (int s = 0; s < N; ++s)
                get_words<B>(slot + G::O_X + G::XS * s, lane, sw[s]);
        } else {
#pragma unroll
            for (int s = 0; s < N; ++s)
                x0[s] = slot[G::O_X + 64 * s + lane];
#pragma unroll
            for (int q = 0; q < G::MUW; ++q)
                muw[q] = slot[G::O_MU + 64 * q + lane];
        }
        const u64 act = ((u64)(u32)__builtin_amdgcn_readfirstlane(on.y) << 32) |
                        (u64)(u32)__builtin_amdgcn_readfirstlane(on.x);
        if (__builtin_expect(__builtin_amdgcn_readfirstlane(on.z) != 0, 0)) {
            const u64 rm = ((u64)ctl_ld(&ctl->rmask[1]) << 32) | ctl_ld(&ctl->rmask[0]);
            if (in_mask(rm)) {
                k = (i32)W.tab[G::T_K + lane];
                row = I.snap + (u64)(k - L.k_lo) * N * I.E + W.tab[G::T_IDX + lane];
                t_next = k < L.k_hi ? row_time(k) : (Tm)SSA_INF_F;
                t_after = k + 1 < L.k_hi ? row_time(k + 1) : (Tm)SSA_INF_F;
            }
            lds_fence();
        }
        Tm tn[B], t_max = (Tm)(-SSA_INF_F);
#pragma unroll
        for (int e = 0; e < B; ++e) {
            tn[e] = (Tm)value_at<A>(tw, e);
            t_max = tn[e] > t_max ? tn[e] : t_max;
        }
        if ((act & lanes(t_next < t_max)) != 0) {
            u32 xw[N][B];   // states before each event
            if constexpr (G::STATES) {
#pragma unroll
                for (int s = 0; s < N; ++s)
#pragma unroll
                    for (int e = 0; e < B; ++e)
                        xw[s][e] = sw[s][e];
            } else {
                i32 x[N];
#pragma unroll
                for (int s = 0; s < N; ++s)
                    x[s] = (i32)x0[s];
#pragma unroll
                for (int e = 0; e < B; ++e) {
#pragma unroll
                    for (int s = 0; s < N; ++s)
                        xw[s][e] = (u32)x[s];
                    if (e + 1 < B)
                        Md::update(x, (int)((muw[e / G::MUPER] >> (G::MUB * (e % G::MUPER))) & ((1u << G::MUB) - 1u)));
                }
            }
            // One row a lane and turn, every lane at its own event. Where only a lane or
            // two are left, each with a wait that spans many rows (a promoter that is off
            // for twenty of them), the whole wave writes that lane's rows, one a lane.
            for (;;) {
                const u64 cross = act & lanes(t_next < t_max);
                if (cross == 0)
                    break;
                i32 xs[N];   // the state before the first event after t_next, and its time
                Tm at = tn[B - 1];
#pragma unroll
                for (int s = 0; s < N; ++s)
                    xs[s] = (i32)xw[s][B - 1];
#pragma unroll
                for (int e = B - 2; e >= 0; --e) {
                    const bool here = t_next < tn[e];
                    at = here ? tn[e] : at;
#pragma unroll
                    for (int s = 0; s < N; ++s)
                        xs[s] = here ? (i32)xw[s][e] : xs[s];
                }
                const u64 more = cross & lanes(t_after < at);   // a second row at the same event
                if (more != 0 && __popcll(cross) <= 2) {
                    const u32 j = (u32)__ffsll((long long)cross) - 1u;
                    const i32 kj = __builtin_amdgcn_readlane(k, j);
                    const u64 rj = ((u64)(u32)__builtin_amdgcn_readlane((u32)((u64)row >> 32), j) << 32) |
                                   (u64)(u32)__builtin_amdgcn_readlane((u32)(u64)row, j);
                    Tm aj;
                    if constexpr (sizeof(Tm) == 8) {
                        const u64 ab = __builtin_bit_cast(u64, at);
                        aj = __builtin_bit_cast(Tm, ((u64)(u32)__builtin_amdgcn_readlane((u32)(ab >> 32), j) << 32) |
                                                        (u64)(u32)__builtin_amdgcn_readlane((u32)ab, j));
                    } else {
                        aj = __builtin_bit_cast(Tm, __builtin_amdgcn_readlane(__builtin_bit_cast(u32, at), j));
                    }
                    const u64 stored = lanes(row_time(kj + (i32)lane) < aj);   // times ascend: its first lanes
                    i32 *const to = (i32 *)rj + (u64)lane * ((u64)N * I.E);
#pragma unroll
                    for (int s = 0; s < N; ++s) {
                        const i32 xj = __builtin_amdgcn_readlane(xs[s], j);
                        if (in_mask(stored))
                            to[(u64)s * I.E] = xj;
                    }
                    if (lane == j) {
                        const u32 cnt = (u32)__popcll(stored);
                        row += (u64)cnt * N * I.E;
                        k += (i32)cnt;
                        t_next = row_time(k);
                        t_after = row_time(k + 1);
                    }
                } else if (in_mask(cross)) {
#pragma unroll
                    for (int s = 0; s < N; ++s)
                        row[(u64)s * I.E] = xs[s];
                    row += (u64)N * I.E;
                    ++k;
                    t_next = t_after;
                    t_after = row_time(k + 1);
                }
            }
        }
        lds_fence();
        lds_st(&ctl->done_s, b + 1u);
        si_next = si + 1u == W.nb ? 0u : si + 1u;
    }
}

template <class P, class Md, bool HALF, bool PER_LANE_RATES>
__device__ __forceinline__ void pipe_item(const LaunchArgs &L, const ItemArgs &I, const PipeWg &W0, u32 words, u32 role)
{
    typedef PipeGeom<P, Md, HALF> G;
    PipeWg W = W0;
    W.nb = G::batches(words);
    W.tab = W.ring + W.nb * (u32)G::SLOT;
    if (role == 0u) {
        __builtin_amdgcn_s_setprio(3);
        pipe_events<P, Md, HALF, PER_LANE_RATES>(L, I, W);
    } else if (role == 1u) {
        __builtin_amdgcn_s_setprio(2);
        pipe_clock<P, Md, HALF, PER_LANE_RATES>(L, I, W);
    } else if (role == 3u) {
        __builtin_amdgcn_s_setprio(2);
        pipe_rows<P, Md, HALF>(L, I, W);
    } else {
        pipe_draw<P, Md, HALF>(L, W);
    }
}

// --------------------------------------------------------------------------
// Claim order for the next snapshot chunk: trajectories sorted by the events
// they fired in the last chunk, heaviest first, in 256 log-spaced classes
// (8 per octave). Waves then hold trajectories of similar length, and the
// longest start first. Only the lane a trajectory runs on changes; its draws
// are keyed by its id, so results are unchanged.
// --------------------------------------------------------------------------
__device__ __forceinline__ u32 work_class(u32 w)
{
    u32 v = w + 1u;
    u32 lz = 31u - (u32)__builtin_clz(v);                 // floor(log2 v)
    u32 frac = lz >= 3u ? (v >> (lz - 3u)) & 7u : (v << (3u - lz)) & 7u;
    u32 key = lz * 8u + frac;
    return 255u - (key > 255u ? 255u : key);               // heaviest first
}

extern "C" __global__ void ssa_regroup_hist(const u32 *work, u32 E, u32 *hist)
{
    __shared__ u32 h[256];
    h[threadIdx.x] = 0u;
    __syncthreads();
    for (u32 i = blockIdx.x * blockDim.x + threadIdx.x; i < E; i += gridDim.x * blockDim.x)
        atomicAdd(&h[work_class(work[i])], 1u);
    __syncthreads();
    if (h[threadIdx.x])
        atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}

extern "C" __global__ void ssa_regroup_scan(u32 *hist)
{
    // one workgroup of 256 threads: exclusive prefix sum in place
    __shared__ u32 v[256];
    const u32 t = threadIdx.x;
    v[t] = hist[t];
    __syncthreads();
    for (u32 off = 1; off < 256u; off <<= 1) {
        u32 add = t >= off ? v[t - off] : 0u;
        __syncthreads();
        v[t] += add;
        __syncthreads();
    }
    hist[t] = t ? v[t - 1] : 0u;
}

// Workgroups of 256 threads take tiles of 256 trajectories: ranks within a
// class come from an LDS histogram of the tile and each (tile, class) reserves
// its range with one global atomic. The order inside a class is arbitrary.
extern "C" __global__ void __launch_bounds__(256) ssa_regroup_scatter(const u32 *work, u32 E, u32 *offs, u32 *order)
{
    __shared__ u32 cnt[256];
    __shared__ u32 base[256];
    const u32 t = threadIdx.x;
    // the tile loop condition is the same for every thread of the workgroup
    for (u32 tile = blockIdx.x * 256u; tile < E; tile += gridDim.x * 256u) {
        cnt[t] = 0u;
        __syncthreads();
        const u32 i = tile + t;
        u32 cls = 0u, rank = 0u;
        if (i < E) {
            cls = work_class(work[i]);
            rank = atomicAdd(&cnt[cls], 1u);
        }
        __syncthreads();
        if (cnt[t])
            base[t] = atomicAdd(&offs[t], cnt[t]);
        __syncthreads();
        if (i < E)
            order[base[cls] + rank] = i;
        __syncthreads();
    }
}
