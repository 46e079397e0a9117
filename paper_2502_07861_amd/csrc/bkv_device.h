// Device-side building blocks shared by the BalanceKV kernels (gfx950 / CDNA4 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/balancekv.h"

namespace bkv {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------------
// Counter-based draws for "eta_j = +1 with probability p_j" (Alg. 2 line 9): two rounds of the
// SplitMix64 output mixer over (seed, stream, counter); the top 24 bits give u = bits * 2^-24.
// Integer-only, so host and device agree bit for bit.
// ---------------------------------------------------------------------------------------------
__host__ __device__ inline uint64_t mix64(uint64_t z) {
    z ^= z >> 30; z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27; z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}
__host__ __device__ inline uint64_t stream_key(uint64_t seed, uint64_t stream) {
    return mix64(seed + 0x9E3779B97F4A7C15ull * (stream + 1));
}
__host__ __device__ inline uint32_t draw_bits_keyed(uint64_t key, uint64_t ctr) {
    return (uint32_t)(mix64(key + 0x9E3779B97F4A7C15ull * (ctr + 1)) >> 40);
}
__host__ __device__ inline uint32_t draw_bits(uint64_t seed, uint64_t stream, uint64_t ctr) {
    return draw_bits_keyed(stream_key(seed, stream), ctr);
}

// ---------------------------------------------------------------------------------------------
// Element traits: 16-byte operand fragments and the MFMA step that consumes one pair of them.
// A fragment is what one lane contributes to a 32-row (or 32-column) operand for one "k-group"
// of 32 bytes per row: lane (n = lane%32, h = lane/32) holds bytes [32g + 16h, 32g + 16h + 16)
// of row n.  Both operands of the Gram use the same mapping, so the contraction visits every
// column of K exactly once whatever order the hardware pairs the sub-elements in.
// ---------------------------------------------------------------------------------------------
template <typename T> struct Elem;

template <> struct Elem<__bf16> {
    typedef bf16x8_t Frag;
    static constexpr int kPerFrag = 8;                 // elements in 16 bytes
    static __device__ __forceinline__ void mma(floatx16& acc, Frag a, Frag b) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
    }
    // the same product on top of c, into a result of its own (c stays intact: several accumulators can start from it)
    static __device__ __forceinline__ floatx16 mma_from(Frag a, Frag b, const floatx16& c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    // several products with one b, their accumulators in turn
    template <int N>
    static __device__ __forceinline__ void mma_turns(floatx16 (&acc)[N], const Frag (&a)[N], Frag b) {
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b, acc[i], 0, 0, 0);
    }
    static __device__ __forceinline__ void unpack(const uintx4& raw, float (&f)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(raw[i] << 16);
            f[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u);
        }
    }
    // part[e] += element e of the slice, e = 0..7: one v_dot2c_f32_bf16 per element (the pair times (1, 0) or (0, 1): the
    // product with 1 is exact, the one with 0 adds nothing for finite inputs) instead of a shift or mask and an add
    static __device__ __forceinline__ void accumulate(float (&part)[8], const uintx4& raw) {
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
        // (1, 0) and (0, 1) as bf16 pairs, kept in registers: written as literals the compiler folds them into an inline
        // operand of the packed instruction that selects the wrong half (both calls then add the high element)
        unsigned int lo_one = 0x00003f80u, hi_one = 0x3f800000u;
        asm volatile("" : "+v"(lo_one), "+v"(hi_one));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned int ri = raw[i];
            part[2 * i] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, ri), __builtin_bit_cast(bf16x2_t, lo_one), part[2 * i], false);
            part[2 * i + 1] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, ri), __builtin_bit_cast(bf16x2_t, hi_one), part[2 * i + 1], false);
        }
    }
    // dot product of two 16-byte slices (8 bf16 each), fp32 accumulation: v_dot2c_f32_bf16
    static __device__ __forceinline__ float dot(const uintx4& a, const uintx4& b) {
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const unsigned int ai = a[i], bi = b[i];      // scalars first: bit-casting a vector element directly picks element 0
            acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, ai), __builtin_bit_cast(bf16x2_t, bi), acc, false);
        }
        return acc;
    }
};

template <> struct Elem<float> {
    typedef floatx4 Frag;
    static constexpr int kPerFrag = 4;
    static __device__ __forceinline__ void mma(floatx16& acc, Frag a, Frag b) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc, 0, 0, 0);
    }
    static __device__ __forceinline__ floatx16 mma_from(Frag a, Frag b, const floatx16& c) {
        floatx16 acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0], b[0], c, 0, 0, 0);
#pragma unroll
        for (int e = 1; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], acc, 0, 0, 0);
        return acc;
    }
    template <int N>
    static __device__ __forceinline__ void mma_turns(floatx16 (&acc)[N], const Frag (&a)[N], Frag b) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[e], acc[i], 0, 0, 0);
    }
    static __device__ __forceinline__ void unpack(const uintx4& raw, float (&f)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(raw[i]);
    }
    static __device__ __forceinline__ void accumulate(float (&part)[4], const uintx4& raw) {
#pragma unroll
        for (int i = 0; i < 4; ++i) part[i] += __uint_as_float(raw[i]);
    }
    static __device__ __forceinline__ float dot(const uintx4& a, const uintx4& b) {
        float acc = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = fmaf(__uint_as_float(a[i]), __uint_as_float(b[i]), acc);
        return acc;
    }
};

// fp32 -> bf16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ unsigned int f32_to_bf16_bits(float x) {
    unsigned int u = __float_as_uint(x);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Cross-lane steps without LDS: DPP inside a row of 16 lanes, v_permlane16_swap / v_permlane32_swap between rows
// (__shfl_xor goes through LDS: about 130 clocks a step, and a reduction is a chain of six).
template <int CTRL> __device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
// acc += x[lane FIRST + e of the row of 16] * f[e], e = 0 .. N-1 in order: the broadcast is part of the multiply-add.  (A DPP operand
// may be read two wait states after a vector instruction wrote it at the earliest.)
template <int FIRST> __device__ __forceinline__ void dpp_dot(float& acc, float x, const float (&f)[4]) {
    asm("s_nop 1\n\tv_fmac_f32_dpp %0, %1, %2 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\tv_fmac_f32_dpp %0, %1, %3 row_newbcast:%7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\tv_fmac_f32_dpp %0, %1, %5 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
        : "+&v"(acc) : "v"(x), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]), "n"(FIRST), "n"(FIRST + 1), "n"(FIRST + 2), "n"(FIRST + 3));
}
template <int FIRST> __device__ __forceinline__ void dpp_dot(float& acc, float x, const float (&f)[8]) {
    asm("s_nop 1\n\tv_fmac_f32_dpp %0, %1, %2 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\tv_fmac_f32_dpp %0, %1, %3 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:%12 row_mask:0xf bank_mask:0xf\n\tv_fmac_f32_dpp %0, %1, %5 row_newbcast:%13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %6 row_newbcast:%14 row_mask:0xf bank_mask:0xf\n\tv_fmac_f32_dpp %0, %1, %7 row_newbcast:%15 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %8 row_newbcast:%16 row_mask:0xf bank_mask:0xf\n\tv_fmac_f32_dpp %0, %1, %9 row_newbcast:%17 row_mask:0xf bank_mask:0xf"
        : "+&v"(acc) : "v"(x), "v"(f[0]), "v"(f[1]), "v"(f[2]), "v"(f[3]), "v"(f[4]), "v"(f[5]), "v"(f[6]), "v"(f[7]), "n"(FIRST), "n"(FIRST + 1),
          "n"(FIRST + 2), "n"(FIRST + 3), "n"(FIRST + 4), "n"(FIRST + 5), "n"(FIRST + 6), "n"(FIRST + 7));
}
struct LanePair { float a, b; };
// the values of lanes l and l ^ O as an unordered pair, the same pair in both lanes (for commutative reductions)
template <int O> __device__ __forceinline__ LanePair lane_pair(float x) {
    if constexpr (O == 32) {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return {__uint_as_float(sw[0]), __uint_as_float(sw[1])};
    } else if constexpr (O == 16) {
        const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        return {__uint_as_float(sw[0]), __uint_as_float(sw[1])};
    } else if constexpr (O == 8) return {x, dpp<0x128>(x)};                    // row_ror:8
    else if constexpr (O == 4) return {x, dpp<0x1B>(dpp<0x141>(x))};           // row_half_mirror (^ 7), quad_perm [3,2,1,0] (^ 3)
    else if constexpr (O == 2) return {x, dpp<0x4E>(x)};                       // quad_perm [2,3,0,1]
    else return {x, dpp<0xB1>(x)};                                             // quad_perm [1,0,3,2]
}
template <int O> __device__ __forceinline__ float xor_max(float x) { const LanePair p = lane_pair<O>(x); return fmaxf(p.a, p.b); }
template <int O> __device__ __forceinline__ float xor_min(float x) { const LanePair p = lane_pair<O>(x); return fminf(p.a, p.b); }
template <int O> __device__ __forceinline__ float xor_sum(float x) { const LanePair p = lane_pair<O>(x); return p.a + p.b; }
__device__ __forceinline__ float wave_max(float v) { return xor_max<1>(xor_max<2>(xor_max<4>(xor_max<8>(xor_max<16>(xor_max<32>(v)))))); }
__device__ __forceinline__ float wave_min(float v) { return xor_min<1>(xor_min<2>(xor_min<4>(xor_min<8>(xor_min<16>(xor_min<32>(v)))))); }
__device__ __forceinline__ float wave_sum(float v) { return xor_sum<1>(xor_sum<2>(xor_sum<4>(xor_sum<8>(xor_sum<16>(xor_sum<32>(v)))))); }

// all-reduce (sum) over SL consecutive lanes, SL in {8,16,32}
template <int SL> __device__ __forceinline__ float group_sum(float x) {
    x += dpp<0xB1>(x);
    x += dpp<0x4E>(x);
    x += dpp<0x141>(x);                          // row_half_mirror
    if (SL >= 16) x += dpp<0x140>(x);            // row_mirror
    if (SL >= 32) x = xor_sum<16>(x);
    return x;
}

// Sixteen values per lane, summed over the 16 lanes of a row: lane s of the row returns the total of x[s].  Each step
// halves the values a lane carries (it keeps the half its own lane bit selects and hands the other half to its
// partner), so the sixteen sums take 15 exchanges instead of 64.  The first step takes the values two at a time, x[j]
// and x[j + 8] (where they are formed one after the other, eight sums are held instead of sixteen values).
__device__ __forceinline__ float row16_pair(float xj, float xj8, int s) {
    const bool b3 = (s & 8) != 0;
    const float mine = b3 ? xj8 : xj, send = b3 ? xj : xj8;
    return mine + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0x140, 0xF, 0xF, true));       // row_mirror
}
__device__ __forceinline__ float row16_rest(const float (&y)[8], int s) {
    const bool b2 = (s & 4) != 0, b1 = (s & 2) != 0, b0 = (s & 1) != 0;
    float z[4], u[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float mine = b2 ? y[j + 4] : y[j], send = b2 ? y[j] : y[j + 4];
        z[j] = mine + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0x141, 0xF, 0xF, true));   // row_half_mirror
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const float mine = b1 ? z[j + 2] : z[j], send = b1 ? z[j] : z[j + 2];
        u[j] = mine + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
    }
    const float mine = b0 ? u[1] : u[0], send = b0 ? u[0] : u[1];
    return mine + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0xB1, 0xF, 0xF, true));        // quad_perm [1,0,3,2]
}
__device__ __forceinline__ float row16_transpose_sum(const float (&x)[16], int s) {
    float y[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) y[j] = row16_pair(x[j], x[j + 8], s);
    return row16_rest(y, s);
}

}  // namespace bkv
