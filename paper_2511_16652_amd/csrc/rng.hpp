// Counter-based noise for EGGROLL on gfx950: Threefry-2x32-20 (Salmon et al., SC'11 -- the generator
// family the paper cites for on-demand noise reconstruction, Sec. 1 and Alg. 1) and the maps from
// 32-bit words to Gaussian / bounded-integer factor entries.
//
// Everything here is integer ALU work plus four transcendental ops per Box-Muller pair; the stream
// key is wave-uniform, so the key schedule lives in scalar registers.
#pragma once
#include <hip/hip_runtime.h>
#include <array>
#include <stdint.h>

namespace egg {

struct StreamKey {  // derived key of one (seed, step, layer, which) stream, with its parity word
    uint32_t k0, k1, k2;
};

__host__ __device__ __forceinline__ uint32_t rotl(uint32_t v, int s) { return (v << s) | (v >> (32 - s)); }

// one Threefry-2x32-20 block: (c0, c1) under key (k0, k1); k2 = k0 ^ k1 ^ 0x1BD11BDA
__host__ __device__ __forceinline__ void threefry2x32_20(uint32_t k0, uint32_t k1, uint32_t k2, uint32_t c0,
                                                         uint32_t c1, uint32_t& o0, uint32_t& o1)
{
    uint32_t x0 = c0 + k0, x1 = c1 + k1;
#define EGG_TF_MIX(R) x0 += x1; x1 = rotl(x1, R); x1 ^= x0;
    EGG_TF_MIX(13) EGG_TF_MIX(15) EGG_TF_MIX(26) EGG_TF_MIX(6)
    x0 += k1; x1 += k2 + 1u;
    EGG_TF_MIX(17) EGG_TF_MIX(29) EGG_TF_MIX(16) EGG_TF_MIX(24)
    x0 += k2; x1 += k0 + 2u;
    EGG_TF_MIX(13) EGG_TF_MIX(15) EGG_TF_MIX(26) EGG_TF_MIX(6)
    x0 += k0; x1 += k1 + 3u;
    EGG_TF_MIX(17) EGG_TF_MIX(29) EGG_TF_MIX(16) EGG_TF_MIX(24)
    x0 += k1; x1 += k2 + 4u;
    EGG_TF_MIX(13) EGG_TF_MIX(15) EGG_TF_MIX(26) EGG_TF_MIX(6)
    x0 += k2; x1 += k0 + 5u;
#undef EGG_TF_MIX
    o0 = x0;
    o1 = x1;
}

// host side: key of the stream named by (seed, step, layer, which)
inline StreamKey make_stream_key(uint64_t seed, uint32_t step, uint32_t layer, int which)
{
    const uint32_t s0 = (uint32_t)seed, s1 = (uint32_t)(seed >> 32);
    StreamKey k;
    threefry2x32_20(s0, s1, s0 ^ s1 ^ 0x1BD11BDAu, step, (layer & 0x7FFFFFFFu) | ((uint32_t)(which & 1) << 31),
                    k.k0, k.k1);
    k.k2 = k.k0 ^ k.k1 ^ 0x1BD11BDAu;
    return k;
}

// words 2*block, 2*block+1 of member's vector
__device__ __forceinline__ void noise_words(const StreamKey& k, uint32_t member, uint32_t block, uint32_t& w0,
                                            uint32_t& w1)
{
    threefry2x32_20(k.k0, k.k1, k.k2, block, member, w0, w1);
}

// u = ((w >> 9) + 1/2) * 2^-23, exact in fp32 (24 significant bits).  The 23 bits become the mantissa of a number in
// [1, 2) with one alignbit (the word 0x7F : w shifted right by 9 is 0x3F800000 | w >> 9); subtracting 1 - 2^-24 leaves
// (2k + 1) 2^-24, which fp32 holds, so the subtraction is exact.  Two instructions; shift, or, convert and multiply
// (the integer (w >> 9) * 2 + 1 scaled by 2^-24) were four, of about 88 per pair of normals.
__device__ __forceinline__ float word_to_unit(uint32_t w)
{
    return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, w, 9)) - 0.999999940395355224609375f;
}

// Box-Muller pair from one block.  PRECISE: library log/sincospi (few-ulp), used where the factors
// stay fp32; otherwise the hardware log2/sin/cos/sqrt approximations, whose error is far below the
// bf16 rounding applied to the result.
template <bool PRECISE>
__device__ __forceinline__ void normal_pair(uint32_t w0, uint32_t w1, float& z0, float& z1)
{
    const float u1 = word_to_unit(w0);
    const float u2 = word_to_unit(w1);
    if constexpr (PRECISE) {
        const float rho = sqrtf(-2.0f * logf(u1));
        float s, c;
        sincospif(2.0f * u2, &s, &c);
        z0 = rho * c;
        z1 = rho * s;
    } else {
        // -2 ln u = -2 ln2 * log2 u ; v_sin/v_cos take their argument in revolutions
        const float rho = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1));
        z0 = rho * __builtin_amdgcn_cosf(u2);
        z1 = rho * __builtin_amdgcn_sinf(u2);
    }
}

// Exact division of x < 2^31 by a divisor chosen on the host: x / d = mulhi(x, mul) >> shift (d > 1; mul = 0 stands for
// d = 1).  With s = ceil(log2 d) and mul = ceil(2^(31+s) / d) the excess mul d - 2^(31+s) is below d <= 2^s, so x times it
// stays below 2^(31+s) and the quotient is exact.
struct FastDiv {
    uint32_t d, mul, shift;
};

inline FastDiv make_fast_div(uint32_t d)
{
    FastDiv f{d, 0u, 0u};
    if (d > 1) {
        uint32_t s = 1;
        while (s < 31 && (uint64_t(1) << s) < d) ++s;
        f.mul = (uint32_t)(((uint64_t(1) << (31 + s)) + d - 1) / d);
        f.shift = s - 1;
    }
    return f;
}

__host__ __device__ __forceinline__ uint32_t fast_div(const FastDiv& f, uint32_t x)
{
    return f.mul ? (uint32_t)(((uint64_t)x * f.mul) >> 32) >> f.shift : x;
}

// byte -> integer on {-b..b}: m = 2b+1, q = 256/m; byte < q*m ? byte/q - b : 0.
// In 16 bits, in both halves of a word: (byte * mul2 + add2) >> shift2 is byte / q below q m and more than 2 b from there on.
struct IntMap {
    uint32_t mul2, add2, shift2, bound2;
};

// (bound <= 127; the search takes about a microsecond, which every launch of the generator paid: all of them once in a process)
inline IntMap make_int_map(int bound)
{
    static const std::array<IntMap, 128> maps = [] {
        std::array<IntMap, 128> all{};
        for (uint32_t b = 0; b < 128; ++b) {
            const uint32_t m = 2u * b + 1u, q = 256u / m;
            IntMap& map = all[b];
            map.bound2 = b * 0x10001u;
            // 2^s / q rounded up, or rounded down and applied to byte + 1: one of them does for every bound up to 127
            for (uint32_t s = 0; s < 16 && !map.mul2; ++s)
                for (uint32_t up = 0; up < 2 && !map.mul2; ++up) {
                    const uint32_t mul = up ? (1u << s) / q : ((1u << s) + q - 1u) / q, add = up ? mul : 0u;
                    bool exact = mul && mul * 255u + add <= 65535u;
                    for (uint32_t x = 0; x < 256 && exact; ++x) {
                        const uint32_t v = (x * mul + add) >> s;
                        exact = x < q * m ? v == x / q : v > 2u * b;
                    }
                    if (exact) map.mul2 = mul * 0x10001u, map.add2 = add * 0x10001u, map.shift2 = s * 0x10001u;
                }
        }
        return all;
    }();
    return maps[bound];
}

// four packed int8 values from one word, two bytes at a time in 16 bits: a byte at or past q m has a quotient above 2 bound.  About
// 15 instructions; byte by byte it was 32, beside the 67 of the generator for two words.
__device__ __forceinline__ uint32_t int4_from_word(const IntMap& m, uint32_t w)
{
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    typedef short i16x2 __attribute__((ext_vector_type(2)));
    auto pair = [&](u16x2 x) __attribute__((always_inline)) {
        const i16x2 bound = __builtin_bit_cast(i16x2, m.bound2);
        const i16x2 v = __builtin_bit_cast(i16x2, (u16x2)((u16x2)(x * __builtin_bit_cast(u16x2, m.mul2) + __builtin_bit_cast(u16x2, m.add2)) >> __builtin_bit_cast(u16x2, m.shift2))) - bound;
        return __builtin_bit_cast(uint32_t, v) & ~__builtin_bit_cast(uint32_t, (i16x2)((i16x2)(bound - v) >> (short)15));
    };
    const u16x2 even = __builtin_bit_cast(u16x2, w & 0x00FF00FFu), odd = __builtin_bit_cast(u16x2, w) >> (uint16_t)8;
    return __builtin_amdgcn_perm(pair(odd), pair(even), 0x06020400u);
}

// fp32 -> bf16, round to nearest even, through the gfx950 packed conversion instruction
typedef __bf16 egg_bf16x2 __attribute__((ext_vector_type(2)));
typedef float egg_f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    const egg_f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, egg_bf16x2));
}

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) { return (uint16_t)(pack_bf16x2(f, 0.f) & 0xFFFFu); }

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xFFFF0000u); }

// round an fp32 value to the nearest bf16 and return it as fp32
__device__ __forceinline__ float round_bf16(float f) { return bf16_lo(pack_bf16x2(f, 0.f)); }

typedef uint32_t noise_x4 __attribute__((ext_vector_type(4)));

// 16 bytes of a factor vector: 8 normals in bf16 from the four blocks at blk, or 4 in fp32 from two
template <bool BF16>
__device__ __forceinline__ noise_x4 normal_piece(const StreamKey& k, uint32_t member, uint32_t blk)
{
    constexpr int BPP = BF16 ? 4 : 2;
    uint32_t w[2 * BPP];
#pragma unroll
    for (int b = 0; b < BPP; ++b) noise_words(k, member, blk + b, w[2 * b], w[2 * b + 1]);
    noise_x4 o;
#pragma unroll
    for (int b = 0; b < BPP; ++b) {
        float z0, z1;
        normal_pair<!BF16>(w[2 * b], w[2 * b + 1], z0, z1);
        if constexpr (BF16) {
            o[b] = pack_bf16x2(z0, z1);
        } else {
            o[2 * b] = __float_as_uint(z0);
            o[2 * b + 1] = __float_as_uint(z1);
        }
    }
    return o;
}

// vectors of one length, one per member and back to back, as 16-byte pieces: workgroup first_wg + g draws pieces 256 g .. 256 g + 255
struct NoisePiece {
    StreamKey key;
    FastDiv per_member;   // pieces per member
    uint32_t total;       // pieces
    uint32_t first_wg;
    noise_x4* out;
};

}  // namespace egg
