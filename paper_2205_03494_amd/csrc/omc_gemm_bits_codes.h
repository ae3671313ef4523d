// What the kernels of the products on codes of any width share: their arguments, and a thread's run of consecutive codes from the packed stream to bfloat16.
#pragma once
#include "omc_mma.h"

#pragma clang fp contract(off)

namespace omc {

struct BitsArgs {
    const uint16_t *A;
    const uint32_t *codes;
    const float *sb;
    float *C;
    uint32_t N, K, tiles_m, tiles_n;
    FmtParams fp;
};

// U consecutive codes (U = 32 or 16) as dwords.  Sixteen codes of an odd width start in the middle of a dword every other time;
// their dwords never reach past those of the 32 codes they belong to.
template <int B, int U>
struct Unit {
    static constexpr int kDwords = (U * B + 31) / 32;
    static constexpr bool kShifted = (U * B) % 32 != 0;
    uint32_t w[kDwords];
};
template <int B, int U>
__device__ __forceinline__ void load_unit(const uint32_t *__restrict__ from, Unit<B, U> &u) {
    typedef uint32_t x4 __attribute__((ext_vector_type(4), aligned(4)));
    typedef uint32_t x2 __attribute__((ext_vector_type(2), aligned(4)));
    constexpr int n = Unit<B, U>::kDwords;
    int i = 0;
#pragma unroll
    for (; i + 4 <= n; i += 4) {
        const x4 t = *reinterpret_cast<const x4 *>(from + i);
        u.w[i] = t[0]; u.w[i + 1] = t[1]; u.w[i + 2] = t[2]; u.w[i + 3] = t[3];
    }
    if constexpr ((n & 2) != 0) {
        const x2 t = *reinterpret_cast<const x2 *>(from + (n & ~3));
        u.w[n & ~3] = t[0];
        u.w[(n & ~3) + 1] = t[1];
    }
    if constexpr ((n & 1) != 0) u.w[n - 1] = from[n - 1];
}
// moves the codes of a unit that starts `shift` bits into its first dword to bit 0
template <int B, int U>
__device__ __forceinline__ void align_unit(Unit<B, U> &u, uint32_t shift) {
    if constexpr (Unit<B, U>::kShifted) {
#pragma unroll
        for (int i = 0; i < Unit<B, U>::kDwords; ++i)
            u.w[i] = __builtin_amdgcn_alignbit(i + 1 < Unit<B, U>::kDwords ? u.w[i + 1] : 0u, u.w[i], shift);
    }
}
// code i with its sign bit at bit 31 (what lies below is masked by the decoder)
template <int B, int U>
__device__ __forceinline__ uint32_t unit_code(const Unit<B, U> &u, int i) {
    const int p = i * B, idx = p >> 5, off = p & 31;
    if (off + B <= 32) return u.w[idx] << (32 - B - off);
    return __builtin_amdgcn_alignbit(u.w[idx + 1], u.w[idx], off + B - 32);
}
// codes 2 i and 2 i + 1 of a unit as bfloat16 (their fp32 images have nothing in the low 16 bits)
template <int B, int U>
__device__ __forceinline__ uint32_t decode_pair(const Unit<B, U> &u, int i, const FmtParams &fp) {
    const uint32_t lo = __float_as_uint(decode_top(unit_code<B, U>(u, 2 * i), fp));
    const uint32_t hi = __float_as_uint(decode_top(unit_code<B, U>(u, 2 * i + 1), fp));
    return __builtin_amdgcn_perm(hi, lo, 0x07060302u);
}

// A unit on its way to LDS, as pairs of bfloat16.  HW: the hardware converts the format: S1E2M3 with bias 1 is the microscaling formats' 6-bit E2M3, of which one instruction converts 32 codes;
// S1E5M2 with bias 15 is OCP FP8 E5M2 but for the top exponent (Inf and NaN there), whose codes are converted with the exponent below it and get the missing one afterwards, 11
// instructions for four codes.  The bit-domain decode takes 18.
template <int B, bool HW>
constexpr bool converts_units() { return HW && B == 6; }
inline bool hardware_converts(const FmtParams &fp) {
    return (fp.exp_bits == 2 && fp.man_bits == 3 && fp.bias == 1) || (fp.exp_bits == 5 && fp.man_bits == 2 && fp.bias == 15);
}
template <int B, int U, bool HW>
struct Pairs {
    static constexpr int kWords = converts_units<B, HW>() ? U / 2 : Unit<B, U>::kDwords;
    uint32_t w[kWords];                                       // pairs already, or the codes
    __device__ __forceinline__ void take(const Unit<B, U> &from, uint32_t shift) {
        if constexpr (converts_units<B, HW>()) {
            typedef uint32_t x6 __attribute__((ext_vector_type(6)));
            typedef __bf16 bf16x32 __attribute__((ext_vector_type(32)));
            typedef uint32_t x16 __attribute__((ext_vector_type(16)));
            x6 c = {0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int i = 0; i < Unit<B, U>::kDwords; ++i) c[i] = from.w[i];
            const bf16x32 v = __builtin_amdgcn_cvt_scalef32_pk32_bf16_fp6(c, 1.0f);
            const x16 d = __builtin_bit_cast(x16, v);
#pragma unroll
            for (int i = 0; i < kWords; ++i) w[i] = d[i];
        } else {
            Unit<B, U> u = from;
            align_unit<B, U>(u, shift);
#pragma unroll
            for (int i = 0; i < kWords; ++i) w[i] = u.w[i];
        }
    }
    __device__ __forceinline__ uint32_t pair(int i, const FmtParams &fp) const {
        if constexpr (converts_units<B, HW>()) {
            return w[i];
        } else if constexpr (HW && B == 8) {
            const uint32_t codes = w[i / 2], top = ((codes & 0x7c7c7c7cu) + 0x04040404u) & 0x80808080u;   // bit 7 of the bytes with the top exponent
            const uint32_t lower = codes - (top >> 5);
            const uint32_t two = i % 2 ? __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(lower, 1.0f, true))
                                       : __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(lower, 1.0f, false));
            return two + __builtin_amdgcn_perm(0u, top, i % 2 ? 0x0c030c02u : 0x0c010c00u);               // one more in the exponent
        } else {
            Unit<B, U> u;
#pragma unroll
            for (int d = 0; d < kWords; ++d) u.w[d] = w[d];
            return decode_pair<B, U>(u, i, fp);
        }
    }
};

}  // namespace omc
