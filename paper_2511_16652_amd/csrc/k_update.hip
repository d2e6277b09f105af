// EGGROLL update direction (EGGROLL UPDATE box; Sec. 4.2):
//   G = scale * sum_i f_i A_i B_i^T = scale * (diag(f~) A~)^T B~,  A~ in R^{K x d_out}, B~ in R^{K x d_in},
//   K = N*r, row kappa = i*r + l holds A_i[:, l] (resp. B_i[:, l]), f~ repeats f r times.
// Two steps: (1) a pack pass turns the [member][d][r] factors (the forward's caches, or freshly
// regenerated ones) into K-packed panels -- 16-byte chunks of consecutive kappa for one column --
// with the fitness folded into the A panel; (2) the MFMA NT core contracts the panels over K.
// Small populations do both in one kernel (upd_draw_kernel).
// bf16 factors are packed as fp16 (11 significant bits instead of 8 for f_i*a): a bf16 value of magnitude
// >= 2^-14 is exact in fp16; below that it lands on fp16's subnormal grid (absolute error <= 2^-25) and below
// 2^-25 it becomes zero -- about 5e-5 of N(0,1) draws, each contributing an absolute error <= 2^-25 to a product
// of typical size 1.  The A panel holds (f_i / fnorm) a with |f_i / fnorm| <= 1 (below 2 beyond 2^127), so members whose |f_i| is far
// below max|f| lose relative precision the same way: the error per term is bounded by 2^-25 max|f|, i.e. it is
// relative to the largest fitness, not to f_i.  fp32 factors stay fp32, or (MmaF32Split) are three bf16
// parts each, which hold all their 24 bits.  No atomics: each G entry has one owner
// and a fixed summation order, so the result is run-to-run identical.
#include "common.hpp"
#include "gemm_core.hpp"
#include "gemm_small.hpp"

namespace egg {

// 2^ceil(log2(max|f|)) of the maximum, 2^127 at most (2^128 is infinite), 1 where the maximum is zero or infinite
__device__ __forceinline__ float fitness_pow2(float mx)
{
    float p = 1.f;
    if (mx > 0.f && !__builtin_isinf(mx)) {
        int e;
        (void)frexpf(mx, &e);  // mx = frac * 2^e, frac in [0.5, 1)
        p = ldexpf(1.f, min(e, 127));
    }
    return p;
}

// fnorm[0] = 2^ceil(log2(max|f|)) (fitness_pow2), fnorm[1] = 1/fnorm[0].  Folding f/fnorm[0] into the
// fp16 panel and fnorm[0] into the epilogue scale is exact (a power of two) and keeps f_i*a inside
// the fp16 range whatever the magnitude of the fitness values.
__global__ __launch_bounds__(1024) void fitness_norm_kernel(const float* __restrict__ f, int64_t n, float* __restrict__ fnorm)
{
    __shared__ float red[16];
    float m = 0.f;
    // eight loads in flight per thread (clamped: a value counted twice changes no maximum), so that 8192 members cost one
    // memory round trip; one load per iteration made the pass 9 us at 16384 members
    for (int64_t i = threadIdx.x; i < n; i += 8 * 1024) {
        float v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = f[min(i + k * 1024, n - 1)];
#pragma unroll
        for (int k = 0; k < 8; ++k) m = fmaxf(m, fabsf(v[k]));
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        float mx = red[0];
#pragma unroll
        for (int w = 1; w < 16; ++w) mx = fmaxf(mx, red[w]);
        const float p = fitness_pow2(mx);
        fnorm[0] = p;
        fnorm[1] = 1.f / p;
    }
}

// x f as an entry of an fp16 panel, rounded once (v_fma_mixlo_f16; the statement keeps it from being turned into a product in fp32 and
// a packed conversion, two roundings).  Rank 2, 4 and 8; the passes of rank 1 and 16 round the fp32 product.
__device__ __forceinline__ _Float16 f16_product(float x, float f)
{
    _Float16 p = (_Float16)(x * f);
    asm volatile("" : "+v"(p));
    return p;
}

// out chunk (kg, col) at (kg*d + col)*16 bytes holds kappa = kg*EPC .. +EPC-1 of column `col`.
template <bool BF16>
__global__ __launch_bounds__(256) void pack_kernel(const void* __restrict__ src, const float* __restrict__ fitness,
                                                   const float* __restrict__ fnorm, int64_t members, int d, int rank, int64_t kgroups,
                                                   void* __restrict__ out)
{
    constexpr int EPC = BF16 ? 8 : 4;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= kgroups * d) return;
    const int64_t kg = gid / d;
    const int col = (int)(gid - kg * d);
    const int64_t K = members * rank;
    const float finv = fitness ? fnorm[1] : 1.f;
    float v[EPC];
    if constexpr (BF16) {
        // rank 2, 4 or 8: the 8 values are 8 / rank members x rank contiguous bf16; one load per member, issued
        // unconditionally from clamped addresses (members past the end count with factor 0)
        if (rank == 2 || rank == 4 || rank == 8) {
            uint32_t w[4];
            float fs[4];
            bool in[4];  // the member of word h exists
            if (rank == 8) {
                const int64_t i = kg, ic = min(i, members - 1);
                const u32x4 t = *(const u32x4*)((const uint16_t*)src + (ic * d + col) * 8);
                w[0] = t[0]; w[1] = t[1]; w[2] = t[2]; w[3] = t[3];
                fs[0] = fs[1] = fs[2] = fs[3] = fitness ? fitness[ic] * finv : 1.f;
                in[0] = in[1] = in[2] = in[3] = i < members;
            } else if (rank == 4) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int64_t i = kg * 2 + h, ic = min(i, members - 1);
                    const uint2 t = *(const uint2*)((const uint16_t*)src + (ic * d + col) * 4);
                    w[2 * h] = t.x; w[2 * h + 1] = t.y;
                    fs[2 * h] = fs[2 * h + 1] = fitness ? fitness[ic] * finv : 1.f;
                    in[2 * h] = in[2 * h + 1] = i < members;
                }
            } else {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const int64_t i = kg * 4 + h, ic = min(i, members - 1);
                    w[h] = *(const uint32_t*)((const uint16_t*)src + (ic * d + col) * 2);
                    fs[h] = fitness ? fitness[ic] * finv : 1.f;
                    in[h] = i < members;
                }
            }
            typedef _Float16 h2 __attribute__((ext_vector_type(2)));
            u32x4 o;
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                h2 p;
                const _Float16 zero = 0;  // past the last member: +0
                p[0] = in[h] ? f16_product(bf16_lo(w[h]), fs[h]) : zero;
                p[1] = in[h] ? f16_product(bf16_hi(w[h]), fs[h]) : zero;
                o[h] = __builtin_bit_cast(uint32_t, p);
            }
            ((u32x4*)out)[gid] = o;
            return;
        }
    }
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int64_t kappa = kg * EPC + e;
        float x = 0.f;
        if (kappa < K) {
            const int64_t i = kappa / rank;
            const int l = (int)(kappa - i * rank);
            const int64_t off = (i * d + col) * rank + l;
            if constexpr (BF16) x = __uint_as_float((uint32_t)((const uint16_t*)src)[off] << 16);
            else x = ((const float*)src)[off];
            if (fitness) x *= fitness[i] * finv;
        }
        v[e] = x;
    }
    if constexpr (BF16) {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            h2 p;
            p[0] = (_Float16)v[2 * e];  // round to nearest even
            p[1] = (_Float16)v[2 * e + 1];
            o[e] = __builtin_bit_cast(uint32_t, p);
        }
        ((u32x4*)out)[gid] = o;
    } else {
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = __float_as_uint(v[e]);
        ((u32x4*)out)[gid] = o;
    }
}

// Rank-1 fast path of the pack pass: a thread turns an EPC x EPC block (EPC members x EPC columns,
// one 16-byte load per member) into EPC output chunks that are contiguous in the panel, so both the
// reads and the writes of a wave are fully coalesced.  Needs d % EPC == 0.
template <bool BF16>
__global__ __launch_bounds__(256) void pack_r1_kernel(const void* __restrict__ src, const float* __restrict__ fitness,
                                                      const float* __restrict__ fnorm, int64_t members, int d,
                                                      int64_t kgroups, void* __restrict__ out)
{
    constexpr int EPC = BF16 ? 8 : 4;
    const int cgroups = d / EPC;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= kgroups * cgroups) return;
    const int64_t kg = gid / cgroups;
    const int col0 = (int)(gid - kg * cgroups) * EPC;
    const float finv = fitness ? fnorm[1] : 1.f;
    float x[EPC][EPC];  // [member][column]
    // every load of the thread goes out before the first use (unconditional, from clamped member numbers; members past
    // the end count with factor 0, written as +0)
    u32x4 raw[EPC];
    float fsv[EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const int64_t ic = min(kg * EPC + e, members - 1);
        raw[e] = *(const u32x4*)((const char*)src + (ic * d + col0) * (BF16 ? 2 : 4));
        fsv[e] = fitness ? fitness[ic] * finv : 1.f;
    }
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
        const bool in = kg * EPC + e < members;
        const u32x4 v = in ? raw[e] : u32x4{0u, 0u, 0u, 0u};
        const float fs = in ? fsv[e] : 0.f;
        if constexpr (BF16) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                x[e][2 * w] = bf16_lo(v[w]) * fs;
                x[e][2 * w + 1] = bf16_hi(v[w]) * fs;
            }
        } else {
#pragma unroll
            for (int w = 0; w < 4; ++w) x[e][w] = __uint_as_float(v[w]) * fs;
        }
    }
    u32x4* o = (u32x4*)out + kg * d + col0;
#pragma unroll
    for (int cc = 0; cc < EPC; ++cc) {
        u32x4 r;
        if constexpr (BF16) {
            typedef _Float16 h2 __attribute__((ext_vector_type(2)));
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                h2 p;
                p[0] = (_Float16)x[2 * w][cc];  // round to nearest even
                p[1] = (_Float16)x[2 * w + 1][cc];
                r[w] = __builtin_bit_cast(uint32_t, p);
            }
        } else {
#pragma unroll
            for (int w = 0; w < 4; ++w) r[w] = __float_as_uint(x[w][cc]);
        }
        o[cc] = r;
    }
}

// Factors without caches: regenerated straight into the K-packed panels, A (with the fitness) and B in one launch; no
// [member][d][rank] intermediate is written or re-read.  The (member, block) addressing and the roundings are those of every
// other kernel: bf16 factors times f_i / fnorm as the pack pass rounds them to fp16; fp32 factors stay fp32.
//   rank 1:  a thread owns one column pair of EPC consecutive members -- one Threefry block per member -- and writes the two
//            finished 16-byte chunks, which are neighbours in the panel;
//   (parts: 8 kappa, a chunk of hi, mid and lo parts each for each column)
//   rank >= 2: a thread owns one chunk, EPC consecutive kappa = i r + l of one column: EPC / 2 blocks.
// The blocks of a thread are independent chains.  Vector-ALU bound: about 87 issue slots per block and the conversion.
// Measured at 16384 members x (8192 + 2048) x rank 4 (bf16): 906 us (744 are the generator's issue slots); noise kernel
// 2 x 640 us + pack pass 2 x 240 us before.
struct GenPackJob {
    StreamKey key;
    FastDiv div;          // work items per K group: d / 2 at rank 1, d otherwise
    uint32_t total;       // work items
    uint32_t first_wg;
    int64_t kg0;          // first K group
    int d;
    const float* fitness; // NULL: the B panel
    u32x4* out;
};
struct GenPackArgs {
    GenPackJob job[2];
    uint32_t member_begin;
    int64_t members;
    const float* fnorm;   // NULL: every workgroup of the A panel finds the norm itself (few members) ...
    float* fnorm_out;     // ... and the first one leaves it for the contraction's epilogue
};
constexpr int INLINE_NORM_MEMBERS = 1024;  // up to here the maximum over the fitness costs a workgroup less than a launch does

// how a panel holds its values: fp16 of bf16 factors; fp32; or (fp32 factors) three bf16 parts a value, the hi parts of 32 kappa in four chunks, then their
// mid parts in four, then lo
enum PanelForm { PANEL_F16, PANEL_F32, PANEL_SPLIT };

// parts of one value beyond the largest bf16 one (an infinite fitness, or one of that size beside it).  An infinite one goes into lo, whose
// products are those with the other panel's hi parts alone and keep their signs (hi times a mid part would not).
__device__ __forceinline__ void split_large(float v, float (&part)[3])
{
#pragma clang fp contract(off)
    constexpr float MOST = 3.3895313892515355e38f;  // 2^127 (2 - 2^-7)
    part[0] = part[1] = 0.f;
    part[2] = v;
    if (!__builtin_isinf(v)) {
        part[0] = fabsf(v) > MOST ? __builtin_copysignf(MOST, v) : round_bf16(v);
        part[1] = round_bf16(v - part[0]);
        part[2] = v - part[0] - part[1];
    }
}
// the parts of a + ea and b + eb, a word each; ea, eb: what rounding a and b to 24 bits left (0 for values that are fp32).  Without contraction: a is a
// product, of the generator or with the fitness, and a - hi would be formed from it unrounded, the parts of another factor than the fp32 one.
__device__ __forceinline__ void split_bf16(float a, float b, float ea, float eb, uint32_t& hi, uint32_t& mid, uint32_t& lo)
{
#pragma clang fp contract(off)
    hi = pack_bf16x2(a, b);
    const float a1 = a - bf16_lo(hi), b1 = b - bf16_hi(hi);
    mid = pack_bf16x2(a1, b1);
    lo = pack_bf16x2(a1 - bf16_lo(mid) + ea, b1 - bf16_hi(mid) + eb);
    if (fmaxf(fabsf(a), fabsf(b)) > 3.38e38f) {
        float p[3], q[3];
        split_large(a, p);
        split_large(b, q);
        hi = pack_bf16x2(p[0], q[0]);
        mid = pack_bf16x2(p[1], q[1]);
        lo = pack_bf16x2(p[2], q[2]);
    }
}

// 2^ceil(log2(max|f|)) over at most INLINE_NORM_MEMBERS members, found by the 256 threads of a workgroup
__device__ __forceinline__ float workgroup_norm(const float* __restrict__ fitness, int64_t members)
{
    __shared__ float red[4];
    float m = 0.f;
#pragma unroll
    for (int k = 0; k < INLINE_NORM_MEMBERS / 256; ++k) m = fmaxf(m, fabsf(fitness[min((int64_t)(k * 256 + threadIdx.x), members - 1)]));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    return fitness_pow2(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])));
}

// what a thread draws: EPC kappa of one column, of the pair 2u and 2u + 1 at rank 1, and their mid and lo parts
template <PanelForm FORM, int RANK>
struct PanelChunks {
    static constexpr int COLS = RANK == 1 ? 2 : 1;
    static constexpr int PARTS = FORM == PANEL_SPLIT ? 3 : 1;
    u32x4 c[PARTS][COLS];
};
// (FIT, the A panel: times the fitness; fixed at compile time, as a branch in the code of both panels the pass of 16384 members x (8192 + 2048) x rank 4 took 923 us, 906 so)
template <PanelForm FORM, int RANK, bool FIT>
__device__ __forceinline__ PanelChunks<FORM, RANK> draw_chunks(const StreamKey& key, uint32_t member_begin, int64_t members,
                                                               const float* __restrict__ fitness, float finv, int64_t kg, int u)
{
    constexpr bool BF16 = FORM == PANEL_F16;
    constexpr int EPC = FORM == PANEL_F32 ? 4 : 8;
    PanelChunks<FORM, RANK> out;
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    // fitness of a member of this K group (members past the end count with 0: their entries of the A panel are zero)
    auto fs_of = [&](int64_t m) __attribute__((always_inline)) {
        if constexpr (!FIT) return 1.f;
        const float v = fitness[min(m, members - 1)];  // unconditional, from a clamped index
        return m < members ? v * finv : 0.f;
    };
    if constexpr (RANK == 1) {
        float lo[EPC], hi[EPC];  // columns 2u and 2u + 1 of the members
        float elo[EPC], ehi[EPC];  // (parts: what rounding f a left of it)
        float fs[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) fs[e] = fs_of(kg * EPC + e);
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
            uint32_t w0, w1;
            noise_words(key, member_begin + (uint32_t)(kg * EPC + e), (uint32_t)u, w0, w1);
            normal_pair<!BF16>(w0, w1, lo[e], hi[e]);
            if constexpr (BF16) {
                const uint32_t pk = pack_bf16x2(lo[e], hi[e]);  // the factors are bf16 values
                lo[e] = bf16_lo(pk);
                hi[e] = bf16_hi(pk);
            }
            elo[e] = ehi[e] = 0.f;
            if constexpr (FIT) {
                const float z0 = lo[e], z1 = hi[e];
                lo[e] *= fs[e];
                hi[e] *= fs[e];
                if constexpr (FORM == PANEL_SPLIT) {
                    elo[e] = fmaf(z0, fs[e], -lo[e]);
                    ehi[e] = fmaf(z1, fs[e], -hi[e]);
                }
            }
        }
        u32x4 c0, c1;
        if constexpr (BF16) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                h2 a, b;
                a[0] = (_Float16)lo[2 * w]; a[1] = (_Float16)lo[2 * w + 1];  // round to nearest even
                b[0] = (_Float16)hi[2 * w]; b[1] = (_Float16)hi[2 * w + 1];
                c0[w] = __builtin_bit_cast(uint32_t, a);
                c1[w] = __builtin_bit_cast(uint32_t, b);
            }
        } else if constexpr (FORM == PANEL_F32) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                c0[w] = __float_as_uint(lo[w]);
                c1[w] = __float_as_uint(hi[w]);
            }
        }
        if constexpr (FORM == PANEL_SPLIT) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                uint32_t p[3];
                split_bf16(lo[2 * w], lo[2 * w + 1], elo[2 * w], elo[2 * w + 1], p[0], p[1], p[2]);
#pragma unroll
                for (int q = 0; q < 3; ++q) out.c[q][0][w] = p[q];
                split_bf16(hi[2 * w], hi[2 * w + 1], ehi[2 * w], ehi[2 * w + 1], p[0], p[1], p[2]);
#pragma unroll
                for (int q = 0; q < 3; ++q) out.c[q][1][w] = p[q];
            }
        } else {
            out.c[0][0] = c0;
            out.c[0][1] = c1;
        }
    } else {
        constexpr int NB = EPC / 2;
        float fs[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) fs[b] = fs_of((kg * EPC + 2 * b) / RANK);
        u32x4 o;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int64_t kappa = kg * EPC + 2 * b;
            const int64_t m = kappa / RANK;
            const int l = (int)(kappa - m * RANK);
            uint32_t w0, w1;
            noise_words(key, member_begin + (uint32_t)m, ((uint32_t)u * RANK + l) >> 1, w0, w1);
            float z0, z1;
            normal_pair<!BF16>(w0, w1, z0, z1);
            if constexpr (BF16) {
                const uint32_t pk = pack_bf16x2(z0, z1);
                z0 = bf16_lo(pk);
                z1 = bf16_hi(pk);
            }
            if constexpr (BF16 && RANK < 16) {
                if constexpr (FIT) {
                    h2 p;
                    p[0] = f16_product(z0, fs[b]);
                    p[1] = f16_product(z1, fs[b]);
                    o[b] = __builtin_bit_cast(uint32_t, p);
                    continue;
                }
            }
            float e0 = 0.f, e1 = 0.f;
            if constexpr (FIT && !(BF16 && RANK < 16)) {
                const float p0 = z0 * fs[b], p1 = z1 * fs[b];
                if constexpr (FORM == PANEL_SPLIT) {
                    e0 = fmaf(z0, fs[b], -p0);
                    e1 = fmaf(z1, fs[b], -p1);
                }
                z0 = p0;
                z1 = p1;
            }
            if constexpr (BF16) {
                h2 p;
                p[0] = (_Float16)z0;
                p[1] = (_Float16)z1;
                o[b] = __builtin_bit_cast(uint32_t, p);
            } else if constexpr (FORM == PANEL_SPLIT) {
                uint32_t p[3];
                split_bf16(z0, z1, e0, e1, p[0], p[1], p[2]);
#pragma unroll
                for (int q = 0; q < 3; ++q) out.c[q][0][b] = p[q];
            } else {
                o[2 * b] = __float_as_uint(z0);
                o[2 * b + 1] = __float_as_uint(z1);
            }
        }
        if constexpr (FORM != PANEL_SPLIT) out.c[0][0] = o;
    }
    return out;
}

template <PanelForm FORM, int RANK>
__global__ __launch_bounds__(256) void gen_pack_kernel(GenPackArgs g)
{
    const GenPackJob& J = g.job[blockIdx.x >= g.job[1].first_wg ? 1 : 0];
    float finv = 1.f;
    if (J.fitness) {
        if (g.fnorm) {
            finv = g.fnorm[1];
        } else {
            const float p = workgroup_norm(J.fitness, g.members);
            finv = 1.f / p;
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                g.fnorm_out[0] = p;
                g.fnorm_out[1] = finv;
            }
        }
    }
    const uint32_t i = (blockIdx.x - J.first_wg) * 256u + threadIdx.x;
    if (i >= J.total) return;
    const uint32_t q = fast_div(J.div, i);
    const int u = (int)(i - q * J.div.d);
    const int64_t kg = J.kg0 + q;
    typedef PanelChunks<FORM, RANK> Chunks;
    const Chunks ch = J.fitness ? draw_chunks<FORM, RANK, true>(J.key, g.member_begin, g.members, J.fitness, finv, kg, u)
                                : draw_chunks<FORM, RANK, false>(J.key, g.member_begin, g.members, nullptr, 1.f, kg, u);
    u32x4* const o = J.out + (FORM == PANEL_SPLIT ? (kg >> 2) * SPLIT_CHUNKS + (kg & 3) : kg) * J.d + Chunks::COLS * u;
#pragma unroll
    for (int q = 0; q < Chunks::PARTS; ++q)
#pragma unroll
        for (int c = 0; c < Chunks::COLS; ++c) o[(int64_t)4 * q * J.d + c] = ch.c[q][c];
}

// panels of the A and (out_b != NULL) the B factors
static egg_status launch_gen_pack(eggroll_ctx* c, PanelForm form, const StreamKey& ka, const StreamKey& kb, const egg_shape& s, const float* fitness,
                                  float* fnorm, bool inline_norm, int64_t kgroups, void* out_a, void* out_b)
{
    const int ua = s.rank == 1 ? s.d_out / 2 : s.d_out, ub = s.rank == 1 ? s.d_in / 2 : s.d_in;
    // work items are numbered in 31 bits: a launch takes as many K groups as fit
    const int64_t slab = std::max<int64_t>(1, ((int64_t(1) << 30) - 256) / std::max(ua, ub));
    for (int64_t kg0 = 0; kg0 < kgroups; kg0 += slab) {
        const int64_t nkg = std::min(slab, kgroups - kg0);
        GenPackArgs g{};
        g.member_begin = (uint32_t)s.member_begin;
        g.members = s.member_count;
        g.fnorm = inline_norm ? nullptr : fnorm;
        g.fnorm_out = fnorm;
        const uint32_t ta = (uint32_t)(nkg * ua), tb = out_b ? (uint32_t)(nkg * ub) : 0u;
        const uint32_t wa = (ta + 255u) / 256u, wb = (tb + 255u) / 256u;
        g.job[0] = GenPackJob{ka, make_fast_div((uint32_t)ua), ta, 0u, kg0, s.d_out, fitness, (u32x4*)out_a};
        g.job[1] = GenPackJob{kb, make_fast_div((uint32_t)ub), tb, wa, kg0, s.d_in, nullptr, (u32x4*)out_b};
        KernelScope ks(c, "update_pack");
#define EGG_GEN_PACK(B, R) hipLaunchKernelGGL((gen_pack_kernel<B, R>), dim3(wa + wb), dim3(256), 0, c->stream, g); break
#define EGG_GEN_PACK_RANKS(B)         \
    switch (s.rank) {                 \
        case 1: EGG_GEN_PACK(B, 1);   \
        case 2: EGG_GEN_PACK(B, 2);   \
        case 4: EGG_GEN_PACK(B, 4);   \
        case 8: EGG_GEN_PACK(B, 8);   \
        default: EGG_GEN_PACK(B, 16); \
    }
        if (form == PANEL_F16) EGG_GEN_PACK_RANKS(PANEL_F16)
        else if (form == PANEL_F32) EGG_GEN_PACK_RANKS(PANEL_F32)
        else EGG_GEN_PACK_RANKS(PANEL_SPLIT)
#undef EGG_GEN_PACK_RANKS
#undef EGG_GEN_PACK
        const egg_status st = check_hip(c, hipGetLastError(), "update_pack launch");
        if (st != EGG_OK) return st;
    }
    return EGG_OK;
}

struct UpdArgs {
    float* G;
    void* W;
    const float* fnorm;
    int d_out, d_in;
    float scale, lr;
    int accumulate, w_bf16;
};

// MBLK: row blocks (of 32) per wave tile.  G is row-major [d_out][d_in] and a column n is one k: the 32 lanes of a
// half-wave already write 32 consecutive floats of one G row, so no staging is needed.
template <int MBLK>
struct UpdEpiT {
    typedef float value_t;
    typedef UpdArgs Args;
    const Args a;
    float scale;
    // W += lr G: the lane's MBLK x 16 elements of W in the current column block, read in one batch when the block begins
    // (unconditional loads from clamped addresses; one load and one full wait per element otherwise)
    float wv[MBLK * 16];
    int row0 = 0;  // the lane's first row of the wave tile
    static constexpr __host__ __device__ int lds_per_wave(int) { return 0; }
    __device__ __forceinline__ UpdEpiT(const Args& a_, char*, int) : a(a_) { scale = a.scale * a.fnorm[0]; }
    __device__ __forceinline__ void column(int, bool) {}
    template <int J>
    __device__ __forceinline__ void column_at(int n, bool)
    {
        if (!a.W) return;
        const int64_t nc = min(n, a.d_in - 1);
        if (a.w_bf16) {
            const uint16_t* w = (const uint16_t*)a.W + nc;
#pragma unroll
            for (int k = 0; k < MBLK * 16; ++k) wv[k] = bf16_bits_to_f32(w[(int64_t)min(row0 + (k >> 4) * 32 + ((k >> 2) & 3) * 8 + (k & 3), a.d_out - 1) * a.d_in]);
        } else {
            const float* w = (const float*)a.W + nc;
#pragma unroll
            for (int k = 0; k < MBLK * 16; ++k) wv[k] = w[(int64_t)min(row0 + (k >> 4) * 32 + ((k >> 2) & 3) * 8 + (k & 3), a.d_out - 1) * a.d_in];
        }
    }
    template <int WTM>
    __device__ __forceinline__ void flush(int, int, int) {}
    template <class MT, int MB, int NB>
    __device__ __forceinline__ void extra_mma(typename MT::acc_t (&)[MB][NB], int, int, int, int) {}
    template <int MB, int NB>
    __device__ __forceinline__ void prefetch(int mw0, int, int lane, int)
    {
        static_assert(MB == MBLK, "row blocks per wave tile");
        row0 = mw0 + (lane >> 5) * 4;
    }
    // rows m .. m + 3 (row block I, group Q of the block) of column n
    template <int I, int Q>
    __device__ __forceinline__ void store4_blk(int m, int n, const float (&v)[4], bool valid, int)
    {
        if (!valid || m >= a.d_out) return;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t idx = (int64_t)(m + e) * a.d_in + n;
            float g = scale * v[e];
            if (a.accumulate) g += a.G[idx];
            a.G[idx] = g;
            if (a.W) {
                const float w_new = fmaf(a.lr, g, wv[(I * 4 + Q) * 4 + e]);
                if (a.w_bf16) ((uint16_t*)a.W)[idx] = f32_to_bf16_bits(w_new);
                else ((float*)a.W)[idx] = w_new;
            }
        }
    }
};

// Epilogue of the f16 contraction.  Rows of the product are the columns k of G (P = B panel), its columns the rows j (Q = A
// panel): a lane of a 16 x 16 block owns 4 consecutive k of one j.  A block of 16 rows of G is parked in the wave's LDS slice and
// read back so that the wave writes whole runs of WTM floats of a row in 16-byte pieces (and reads W and, when accumulating, G the
// same way, in one batch per block, unconditionally from clamped addresses).
template <int WTM>
struct UpdEpi16 {
    typedef float value_t;
    typedef UpdArgs Args;
    const Args a;
    char* const stage;
    const int lane;
    static constexpr int P = WTM * 4 + 16, CPR = WTM / 4, PASSES = 16 * CPR / 64;
    static constexpr __host__ __device__ int lds_per_wave(int) { return 16 * P; }
    __device__ __forceinline__ UpdEpi16(const Args& a_, char* slice, int lane_) : a(a_), stage(slice), lane(lane_) {}
    __device__ __forceinline__ void column(int, bool) {}
    template <int J>
    __device__ __forceinline__ void column_at(int, bool) {}
    template <class MT, int MB, int NB>
    __device__ __forceinline__ void extra_mma(typename MT::acc_t (&)[MB][NB], int, int, int, int) {}
    template <int MB, int NB>
    __device__ __forceinline__ void prefetch(int, int, int, int) {}
    template <int I, int J>
    __device__ __forceinline__ void store4_at(int m, int n, const float (&v)[4], bool valid, int ml) { store4(m, n, v, valid, ml); }
    __device__ __forceinline__ void store4(int, int, const float (&v)[4], bool, int ml)
    {
        *(float4*)(stage + (lane & 15) * P + ml * 4) = make_float4(v[0], v[1], v[2], v[3]);
    }
    template <int W_>
    __device__ __forceinline__ void flush(int mw0, int nb0, int n_rows)
    {
        static_assert(W_ == WTM, "wave tile of the launched kernel");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the wave's own LDS writes have landed
        __builtin_amdgcn_wave_barrier();
        const float scale = a.scale * a.fnorm[0];
        if (a.d_in % 4 == 0) {
            float4 g[PASSES], old[PASSES], wf[PASSES];
            uint2 wb[PASSES];
            auto at = [&](int it, bool& in) __attribute__((always_inline)) {
                const int c = it * 64 + lane, j = nb0 + c / CPR, k = mw0 + (c % CPR) * 4;
                in = j < n_rows && k < a.d_in;
                return (int64_t)min(j, n_rows - 1) * a.d_in + min(k, a.d_in - 4);
            };
            bool in;
#pragma unroll
            for (int it = 0; it < PASSES; ++it) {
                const int c = it * 64 + lane;
                g[it] = *(const float4*)(stage + (c / CPR) * P + (c % CPR) * 16);
                if (a.accumulate) old[it] = *(const float4*)(a.G + at(it, in));
                if (a.W && a.w_bf16) wb[it] = *(const uint2*)((const uint16_t*)a.W + at(it, in));
                else if (a.W) wf[it] = *(const float4*)((const float*)a.W + at(it, in));
            }
#pragma unroll
            for (int it = 0; it < PASSES; ++it) {
                const int64_t idx = at(it, in);
                float v[4] = {scale * g[it].x, scale * g[it].y, scale * g[it].z, scale * g[it].w};
                if (a.accumulate) { v[0] += old[it].x; v[1] += old[it].y; v[2] += old[it].z; v[3] += old[it].w; }
                if (!in) continue;
                *(float4*)(a.G + idx) = make_float4(v[0], v[1], v[2], v[3]);
                if (a.W && a.w_bf16)
                    *(uint2*)((uint16_t*)a.W + idx) = make_uint2(pack_bf16x2(fmaf(a.lr, v[0], bf16_lo(wb[it].x)), fmaf(a.lr, v[1], bf16_hi(wb[it].x))),
                                                                 pack_bf16x2(fmaf(a.lr, v[2], bf16_lo(wb[it].y)), fmaf(a.lr, v[3], bf16_hi(wb[it].y))));
                else if (a.W)
                    *(float4*)((float*)a.W + idx) = make_float4(fmaf(a.lr, v[0], wf[it].x), fmaf(a.lr, v[1], wf[it].y), fmaf(a.lr, v[2], wf[it].z), fmaf(a.lr, v[3], wf[it].w));
            }
        } else {
            // rows of G that are not made of whole 16-byte pieces: entry by entry
            for (int c = lane; c < 16 * WTM; c += 64) {
                const int j = nb0 + c / WTM, k = mw0 + c % WTM;
                if (j >= n_rows || k >= a.d_in) continue;
                const int64_t idx = (int64_t)j * a.d_in + k;
                float v = scale * *(const float*)(stage + (c / WTM) * P + (c % WTM) * 4);
                if (a.accumulate) v += a.G[idx];
                a.G[idx] = v;
                if (a.W && a.w_bf16) {
                    uint16_t* w = (uint16_t*)a.W + idx;
                    *w = f32_to_bf16_bits(fmaf(a.lr, v, bf16_bits_to_f32(*w)));
                } else if (a.W) {
                    float* w = (float*)a.W + idx;
                    *w = fmaf(a.lr, v, *w);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();  // the slice is reused by the next row block
    }
};

// Epilogue of the small kernel: rows of the product are the columns k of G (P = B panel), its columns the rows j, so that the 4
// consecutive values of a thread are neighbours in G.
struct UpdSmallEpi {
    typedef float value_t;
    typedef UpdArgs Args;
    const Args a;
    float scale;
    __device__ __forceinline__ UpdSmallEpi(const Args& a_) : a(a_) { scale = a.scale * a.fnorm[0]; }
    __device__ __forceinline__ UpdSmallEpi(const Args& a_, float norm) : a(a_) { scale = a.scale * norm; }
    __device__ __forceinline__ void apply4(int m, int n, const float (&v)[4])
    {
        const int64_t at = (int64_t)n * a.d_in + m;
        float g[4];
        if (a.d_in % 4 == 0) {
            if (a.accumulate) {
                const float4 o = *(const float4*)(a.G + at);
                g[0] = fmaf(scale, v[0], o.x); g[1] = fmaf(scale, v[1], o.y); g[2] = fmaf(scale, v[2], o.z); g[3] = fmaf(scale, v[3], o.w);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) g[e] = scale * v[e];
            }
            *(float4*)(a.G + at) = make_float4(g[0], g[1], g[2], g[3]);
            if (a.W && a.w_bf16) {
                uint2* w = (uint2*)((uint16_t*)a.W + at);
                const uint2 o = *w;
                *w = make_uint2(pack_bf16x2(fmaf(a.lr, g[0], bf16_lo(o.x)), fmaf(a.lr, g[1], bf16_hi(o.x))),
                                pack_bf16x2(fmaf(a.lr, g[2], bf16_lo(o.y)), fmaf(a.lr, g[3], bf16_hi(o.y))));
            } else if (a.W) {
                float4* w = (float4*)((float*)a.W + at);
                const float4 o = *w;
                *w = make_float4(fmaf(a.lr, g[0], o.x), fmaf(a.lr, g[1], o.y), fmaf(a.lr, g[2], o.z), fmaf(a.lr, g[3], o.w));
            }
            return;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (m + e >= a.d_in) break;
            g[e] = a.accumulate ? fmaf(scale, v[e], a.G[at + e]) : scale * v[e];
            a.G[at + e] = g[e];
            if (a.W && a.w_bf16) {
                uint16_t* w = (uint16_t*)a.W + at + e;
                *w = f32_to_bf16_bits(fmaf(a.lr, g[e], bf16_bits_to_f32(*w)));
            } else if (a.W) {
                float* w = (float*)a.W + at + e;
                *w = fmaf(a.lr, g[e], *w);
            }
        }
    }
};

// The whole update of a small population in one kernel: a workgroup draws the 32 columns of both panels that its 32 x 32 tile of G needs
// into LDS and multiplies them there.  Drawing a panel again for every tile beside it costs less than a second launch there (3 us; each
// thread draws K / 8 blocks).  The bits are those of the kernels that multiply packed panels of this size.
struct UpdDrawArgs {
    StreamKey ka, kb;
    uint32_t member_begin;
    int64_t members;
    const float* fitness;
    int kgroups, tiles_m;  // K groups in whole steps
};
template <PanelForm FORM, int RANK>
__global__ __launch_bounds__(256) void upd_draw_kernel(UpdDrawArgs g, UpdArgs ea)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    static_assert(FORM != PANEL_SPLIT, "few tiles are not split");
    typedef PanelChunks<FORM, RANK> Chunks;
    constexpr int PER = 32 / Chunks::COLS;
    u32x4* const panel = (u32x4*)smem;  // [B, A][kgroups][32]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = (int)(blockIdx.x % g.tiles_m) * 32, n0 = (int)(blockIdx.x / g.tiles_m) * 32;  // k, j of G
    const float norm = workgroup_norm(g.fitness, g.members);
    const float finv = 1.f / norm;
    const int items = g.kgroups * PER;
    // columns past the end are drawn as well (any entries of the stream) and not stored
    for (int i = tid; i < 2 * items; i += 256) {
        const bool a = i >= items;
        const int it = a ? i - items : i, kg = it / PER, u = it % PER;
        const Chunks ch = a ? draw_chunks<FORM, RANK, true>(g.ka, g.member_begin, g.members, g.fitness, finv, kg, n0 / Chunks::COLS + u)
                            : draw_chunks<FORM, RANK, false>(g.kb, g.member_begin, g.members, nullptr, 1.f, kg, m0 / Chunks::COLS + u);
#pragma unroll
        for (int c = 0; c < Chunks::COLS; ++c) panel[(a ? g.kgroups * 32 : 0) + kg * 32 + u * Chunks::COLS + c] = ch.c[0][c];
    }
    __syncthreads();
    UpdSmallEpi epi(ea, norm);
    const u32x4 *const P = panel, *const Q = panel + g.kgroups * 32;
    if constexpr (FORM == PANEL_F16) {
        // a wave to a quarter of the tile, K ascending: the bits of the deep kernel
        const int r = lane & 15, q = lane >> 4, mb = (wave & 1) * 16, nb = (wave >> 1) * 16;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int c = q; c < g.kgroups; c += 4) MmaF16Blk16::mma(P[c * 32 + mb + r], Q[c * 32 + nb + r], acc);
        const float v[4] = {acc[0], acc[1], acc[2], acc[3]};
        const int m = m0 + mb + 4 * q, n = n0 + nb + r;
        if (m < ea.d_in && n < ea.d_out) epi.apply4(m, n, v);
    } else {
        // a wave to a quarter of K, the partial tiles added through LDS: the bits of gemm_small_kernel
        constexpr int PITCH = 32 * 4 + 16;
        const int fr = lane & 31, fc = lane >> 5;
        const int steps = g.kgroups / 2, per = (steps + 3) / 4;
        const int s0 = min(wave * per, steps), s1 = min(s0 + per, steps);
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
        for (int s = s0; s < s1; ++s) MmaF32::mma(P[(2 * s + fc) * 32 + fr], Q[(2 * s + fc) * 32 + fr], acc);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) *(f32x4*)(smem + (wave * 32 + fr) * PITCH + (q * 8 + fc * 4) * 4) = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        __syncthreads();
        const int col = tid / 8, row = (tid % 8) * 4, m = m0 + row, n = n0 + col;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const f32x4 x = *(const f32x4*)(smem + (w * 32 + col) * PITCH + row * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += x[e];
        }
        if (m < ea.d_in && n < ea.d_out) epi.apply4(m, n, v);
    }
}

// Where: for up to two tiles of 32 x 32 a CU and populations of up to 64 kappa, 128 in bf16 where a tile is alone on its CU.  Whole updates (us,
// two kernels / this): bf16 256 x 256, K = 64 9.1 / 5.4, 128 9.1 / 6.7, 192 8.0 / 8.6; 1024 x 512 (512 tiles), K = 64 9.3 / 6.7, 128 9.3 / 9.8; fp32 256 x
// 256, K = 64 9.2 / 6.0, 128 9.1 / 8.9 (rank 16 9.1 / 9.8); 1024 x 512, K = 64 9.5 / 7.8, 128 10.2 / 12.2.
static bool draws_in_place(const egg_shape& s, bool bf, int compute_units)
{
    const int64_t tiles = ((s.d_out + 31) / 32) * (int64_t)((s.d_in + 31) / 32);
    if (tiles > 2 * (int64_t)compute_units || s.member_count > INLINE_NORM_MEMBERS) return false;
    return s.member_count * (int64_t)s.rank <= (bf && tiles <= compute_units ? 128 : 64);
}

static egg_status launch_upd_draw(eggroll_ctx* c, bool bf, const StreamKey& ka, const StreamKey& kb, const egg_shape& s, const float* fitness, const UpdArgs& ea)
{
    const int64_t K = s.member_count * (int64_t)s.rank;
    const int kgroups = bf ? (int)((K + 31) / 32) * 4 : (int)((K + 7) / 8) * 2;
    const int tm = (s.d_in + 31) / 32, tn = (s.d_out + 31) / 32;
    const UpdDrawArgs g{ka, kb, (uint32_t)s.member_begin, s.member_count, fitness, kgroups, tm};
    const size_t lds = std::max<size_t>((size_t)kgroups * 2 * 32 * 16, bf ? 0 : 4 * 32 * (32 * 4 + 16));
    KernelScope ks(c, "update_gemm_drawn");
#define EGG_UPD_DRAW(F, R) hipLaunchKernelGGL((upd_draw_kernel<F, R>), dim3((unsigned)(tm * tn)), dim3(256), lds, c->stream, g, ea); break
#define EGG_UPD_DRAW_RANKS(F)         \
    switch (s.rank) {                 \
        case 1: EGG_UPD_DRAW(F, 1);   \
        case 2: EGG_UPD_DRAW(F, 2);   \
        case 4: EGG_UPD_DRAW(F, 4);   \
        case 8: EGG_UPD_DRAW(F, 8);   \
        default: EGG_UPD_DRAW(F, 16); \
    }
    if (bf) EGG_UPD_DRAW_RANKS(PANEL_F16)
    else EGG_UPD_DRAW_RANKS(PANEL_F32)
#undef EGG_UPD_DRAW_RANKS
#undef EGG_UPD_DRAW
    return check_hip(c, hipGetLastError(), "update_gemm_drawn launch");
}

template <class MT, int T>
static egg_status launch_upd_small(eggroll_ctx* c, const char* name, const Operand& P, const Operand& Q, int kchunks, const UpdArgs& ea)
{
    const int tm = (P.rows + T - 1) / T, tn = (Q.rows + T - 1) / T;
    KernelScope ks(c, name);
    hipLaunchKernelGGL((gemm_small_kernel<MT, T, UpdSmallEpi>), dim3((unsigned)(tm * tn)), dim3(256), 0, c->stream, P, Q, kchunks, tm, ea);
    return check_hip(c, hipGetLastError(), name);
}

// DEEP: four stages in flight (parts: three), a workgroup a tile
template <class MT, int BM, int BN, int WM, int WN, bool DEEP>
static egg_status launch_upd_gemm16(eggroll_ctx* c, const char* name, const Operand& P, const Operand& Q, int kchunks, const UpdArgs& ea)
{
    typedef UpdEpi16<BM / WM> Epi;
    const int tiles_m = (P.rows + BM - 1) / BM, tiles_n = (Q.rows + BN - 1) / BN;
    const size_t stages = gemm_lds_bytes<BM, BN>(), epi = (size_t)WM * WN * Epi::lds_per_wave(BM / WM);
    constexpr int CHUNKS = is_split<MT>::value ? SPLIT_CHUNKS : 8;
    if (!operand_offsets_fit(P, BM, CHUNKS) || !operand_offsets_fit(Q, BN, CHUNKS)) return fail(c, EGG_EUNSUPPORTED, "operand strides too large for 32-bit tile offsets");
    const size_t lds = is_split<MT>::value ? (size_t)SPLIT_STAGES * SPLIT_CHUNKS * 16 * (BM + BN) : DEEP ? 2 * stages + epi : std::max(stages, epi);
    static_assert(!is_split<MT>::value || (DEEP && WM * WN * Epi::lds_per_wave(BM / WM) <= SPLIT_CHUNKS * 16 * (BM + BN)), "the slices of the epilogue over a stage");
    const dim3 g((unsigned)(tiles_m * tiles_n)), b(WM * WN * 64);
    if constexpr (DEEP) {
        auto kern = gemm_nt_deep_kernel<MT, BM, BN, WM, WN, true, Epi>;
        const egg_status st = ensure_dynamic_lds(c, (const void*)kern, lds, "gemm smem attr");
        if (st != EGG_OK) return st;
        KernelScope ks(c, name);
        hipLaunchKernelGGL(kern, g, b, lds, c->stream, P, Q, kchunks, tiles_m, tiles_n, (const char*)c->zero_page.p, c->conservative_waits ? 1 : 0, ea);
    } else {
        auto kern = gemm_nt_kernel<MT, BM, BN, WM, WN, true, Epi>;
        const egg_status st = ensure_dynamic_lds(c, (const void*)kern, lds, "gemm smem attr");
        if (st != EGG_OK) return st;
        KernelScope ks(c, name);
        hipLaunchKernelGGL(kern, g, b, lds, c->stream, P, Q, kchunks, tiles_m, tiles_n, (const char*)c->zero_page.p, ea);
    }
    return check_hip(c, hipGetLastError(), name);
}

template <class MT, int BM, int BN, int WM, int WN>
static egg_status launch_upd_gemm(eggroll_ctx* c, const char* name, const Operand& P, const Operand& Q, int kchunks,
                                  const UpdArgs& ea)
{
    const int tiles_m = (P.rows + BM - 1) / BM, tiles_n = (Q.rows + BN - 1) / BN;
    const size_t lds = gemm_lds_bytes<BM, BN>();
    if (!operand_offsets_fit(P, BM) || !operand_offsets_fit(Q, BN)) return fail(c, EGG_EUNSUPPORTED, "operand strides too large for 32-bit tile offsets");
    static_assert(MT::BLK == 32, "the epilogue indexes 32-row blocks");
    auto kern = gemm_nt_kernel<MT, BM, BN, WM, WN, true, UpdEpiT<BM / WM / 32>>;
    egg_status st = ensure_dynamic_lds(c, (const void*)kern, (size_t)lds, "gemm smem attr");
    if (st != EGG_OK) return st;
    KernelScope ks(c, name);
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(WM * WN * 64), lds, c->stream, P, Q, kchunks,
                       tiles_m, tiles_n,
                       (const char*)c->zero_page.p, ea);
    return check_hip(c, hipGetLastError(), name);
}

// fp32 factors generated for the call go into panels of three bf16 parts each (split_bf16), multiplied by bf16 MFMAs, where the tiles of 32 x 32 are more
// than two to a CU: from 192 kappa in tiles of 64 x 64, up to two of them to a CU, and beyond that from 512 in tiles of 128 x 128.  A fp32 MFMA takes 256
// cycles for what six of those do in 96; against that stand panels half as long again, 48 KB for 32 kappa of a 128 x 128 tile, and, of so large tiles, a
// nearly empty last wave.  Whole updates, us, fp32 MFMAs / parts: 64 x 64: 1024 x 736, K = 192 15.6 / 13.6, 1400 x 1400, K = 192 22.7 / 17.7, 1000 59.4 /
// 40.8; 1024 x 1024, K = 1024 40 / 31, 8000 216 / 144.  128 x 128: 2048 x 2048, K = 192 26.5 / 28.6, 384 41.0 / 38.0, 2048 161 / 108, 8000 568 / 366; 2100 x
// 2100, K = 192 32.6 / 42.5, 384 54.2 / 57.6; 4096 x 4096, K = 512 152 / 122, 1024 283 / 204, 8000 2067 / 1380.  Fewer tiles are bound by latency.
// Error against 64 bits, relative 2-norm, fp32 MFMAs / parts: all members with a fitness, 1024 x 1024, K = 192 1.32e-7 / 0.88e-7, 700 2.41e-7 / 1.69e-7, 2048 x
// 2048, K = 700 4.8e-7 / 1.7e-7, 8000 1.60e-6 / 0.57e-6; fitness over eight decades, 700 1.10e-7 / 0.49e-7; sixteen members with one 7.8e-8 / 4.2e-8, four 4.4e-8 /
// 3.0e-8, a single one 3.6e-8 / 2.6e-8 (fp32 rounds it at f a and at the end, parts hold f a to 2^-27 and round at the end).
// (A caller's caches may hold any values: their updates stay on fp32 MFMAs.)
static bool split_update(int64_t M, int64_t N, int64_t K, int compute_units)
{
    const int64_t t32 = ((M + 31) / 32) * ((N + 31) / 32), t64 = ((M + 63) / 64) * ((N + 63) / 64), two = 2 * (int64_t)compute_units;
    return t32 > two && K >= (t64 <= two ? 192 : 512) && std::max(M, N) <= 1 << 24;  // (offsets into a stage in 32 bits)
}

egg_status launch_update(eggroll_ctx* c, const StreamKey& ka, const StreamKey& kb, const egg_shape& s,
                         egg_dtype noise_dtype, const float* fitness, float scale, int accumulate, float* G, void* W,
                         egg_dtype w_dtype, float lr, const void* A_cache, const void* B_cache, bool b_panel)
{
    const bool bf = noise_dtype == EGG_BF16;
    const int esz = bf ? 2 : 4, epc = bf ? 8 : 4;
    const int64_t K = s.member_count * (int64_t)s.rank;
    // Without caches the factors are generated straight into the panels (a rank-1 work item is a column pair: an odd width goes
    // through the noise kernel and the pack pass, like the caches).
    const bool gen_packed = !A_cache && (s.rank > 1 || (s.d_out % 2 == 0 && s.d_in % 2 == 0));
    bool split = !bf && gen_packed && split_update(s.d_out, s.d_in, K, c->compute_units);
    int64_t kgroups = (K + epc - 1) / epc;  // chunks of a panel
    if (kgroups > 0x7FFFFFFF) return fail(c, EGG_EUNSUPPORTED, "population * rank too large");
    egg_status st;

    if (gen_packed && !b_panel && draws_in_place(s, bf, c->compute_units))
        return launch_upd_draw(c, bf, ka, kb, s, fitness, UpdArgs{G, W, nullptr, s.d_out, s.d_in, scale, lr, accumulate, w_dtype == EGG_BF16 ? 1 : 0});
    if ((st = reserve(c, c->fnorm, 256)) != EGG_OK) return st;
    float* fnorm = (float*)c->fnorm.p;
    if (split) {
        // three chunks for 8 kappa, whole stages of 32; where there is no memory for them, fp32 panels take two thirds of it
        const int64_t chunks = (K + 31) / 32 * SPLIT_CHUNKS;
        const eggroll_ctx::Buf held = c->pack_a;
        const size_t retired = c->retired.size();
        split = chunks <= 0x7FFFFFFF && try_reserve(c, c->pack_a, (size_t)chunks * s.d_out * 16) && try_reserve(c, c->pack_b, (size_t)chunks * s.d_in * 16);
        if (split) {
            kgroups = chunks;
        } else if (c->pack_a.p != held.p) {  // the first panel was to be had, the second not: nothing has used it yet
            (void)hipFree(c->pack_a.p);
            c->pack_a = held;
            c->retired.resize(retired);
        }
    }
    if ((st = reserve(c, c->pack_a, (size_t)kgroups * s.d_out * 16)) != EGG_OK) return st;
    // b_panel: the caller's B_cache already is the packed panel (written by the forward pass); only A is generated
    if (!b_panel && (st = reserve(c, c->pack_b, (size_t)kgroups * s.d_in * 16)) != EGG_OK) return st;
    const bool inline_norm = gen_packed && s.member_count <= INLINE_NORM_MEMBERS;
    if (!inline_norm) {
        KernelScope ks(c, "fitness_norm");
        hipLaunchKernelGGL(fitness_norm_kernel, dim3(1), dim3(1024), 0, c->stream, fitness, s.member_count, fnorm);
    }
    if (gen_packed) {
        if ((st = launch_gen_pack(c, bf ? PANEL_F16 : split ? PANEL_SPLIT : PANEL_F32, ka, kb, s, fitness, fnorm, inline_norm, split ? kgroups / 3 : kgroups, c->pack_a.p, b_panel ? nullptr : c->pack_b.p)) != EGG_OK) return st;
    } else {
        // factors in [member][d][r] layout: the caller's caches, or regenerated into scratch
        const void* A_src = A_cache;
        const void* B_src = B_cache;
        if (!A_src) {
            const size_t na = (size_t)s.member_count * s.d_out * s.rank * esz, nb = (size_t)s.member_count * s.d_in * s.rank * esz;
            if ((st = reserve(c, c->a_buf, na)) != EGG_OK) return st;
            if ((st = reserve(c, c->b_buf, nb)) != EGG_OK) return st;
            if ((st = launch_noise(c, ka, (uint32_t)s.member_begin, s.member_count, (int64_t)s.d_out * s.rank, noise_dtype, EGG_NORMAL, 0, c->a_buf.p)) != EGG_OK) return st;
            if ((st = launch_noise(c, kb, (uint32_t)s.member_begin, s.member_count, (int64_t)s.d_in * s.rank, noise_dtype, EGG_NORMAL, 0, c->b_buf.p)) != EGG_OK) return st;
            A_src = c->a_buf.p;
            B_src = c->b_buf.p;
        }
        const int64_t ta = kgroups * s.d_out, tb = kgroups * s.d_in;
        if ((ta + 255) / 256 > 0x7FFFFFFF || (tb + 255) / 256 > 0x7FFFFFFF) return fail(c, EGG_EUNSUPPORTED, "pack grid too large");
        KernelScope ks(c, "update_pack");
        auto pack = [&](const void* src, const float* fit, int d, void* dst) {
            if (s.rank == 1 && d % epc == 0) {
                const int64_t n = kgroups * (d / epc);
                const dim3 g((unsigned)((n + 255) / 256)), b(256);
                if (bf) hipLaunchKernelGGL(pack_r1_kernel<true>, g, b, 0, c->stream, src, fit, fnorm, s.member_count, d, kgroups, dst);
                else hipLaunchKernelGGL(pack_r1_kernel<false>, g, b, 0, c->stream, src, fit, fnorm, s.member_count, d, kgroups, dst);
            } else {
                const int64_t n = kgroups * d;
                const dim3 g((unsigned)((n + 255) / 256)), b(256);
                if (bf) hipLaunchKernelGGL(pack_kernel<true>, g, b, 0, c->stream, src, fit, fnorm, s.member_count, d, s.rank, kgroups, dst);
                else hipLaunchKernelGGL(pack_kernel<false>, g, b, 0, c->stream, src, fit, fnorm, s.member_count, d, s.rank, kgroups, dst);
            }
        };
        pack(A_src, fitness, s.d_out, c->pack_a.p);
        pack(B_src, nullptr, s.d_in, c->pack_b.p);
        if ((st = check_hip(c, hipGetLastError(), "pack launch")) != EGG_OK) return st;
    }

    Operand P{(const char*)c->pack_a.p, 16, (int64_t)s.d_out * 16, s.d_out};
    Operand Q{(const char*)(b_panel ? B_cache : c->pack_b.p), 16, (int64_t)s.d_in * 16, s.d_in};
    UpdArgs ea{G, W, fnorm, s.d_out, s.d_in, scale, lr, accumulate, w_dtype == EGG_BF16 ? 1 : 0};
    if (split) {
        if (((s.d_out + 63) / 64) * (int64_t)((s.d_in + 63) / 64) <= 2 * c->compute_units)
            return launch_upd_gemm16<MmaF32Split, 64, 64, 2, 2, true>(c, "update_gemm_f32", Q, P, (int)kgroups, ea);
        return launch_upd_gemm16<MmaF32Split, 128, 128, 2, 2, true>(c, "update_gemm_f32", Q, P, (int)kgroups, ea);
    }
    const int small = small_tile(s.d_in, s.d_out, c->compute_units);
    if (bf && small) {
        // four stages of K in flight through LDS (whole updates, us, K split over the waves of a tile / this): tiles of 32 256 x 256, K = 2048 17.9 / 15.3,
        // 8000 37.7 / 30.2, 1024 x 512, K = 1024 15.0 / 13.2; tiles of 64 1024 x 1024, K = 300 13.2 / 12.1, 2320 x 608, K = 300 16.2 / 14.5, 8000
        // 104 / 103.  With one tile of 64 to a CU deeper K is better split: 1024 x 1024, K = 1024 16.1 / 16.6, 8000 58 / 61.  So it is from 1.75 tiles to a CU on where the
        // tiles of a row of G are 16, 24 .. and each of the 8 XCDs, workgroups going round them, keeps to the same two or more of its columns: 512 x 4096, K = 1500
        // 30.9 / 32.4, 2000 37 / 42, 6000 75 / 79; 2048 x 1024, K = 2000 34.5 / 35.5, 4096 53.0 / 54.9; 1024 x 2048, K = 4096 50.7 / 51.5.  Otherwise: 4096 x 512 (8 tiles a
        // row), K = 2000 44.0 / 42.6, 8000 126 / 102; 1472 x 1344 (21), K = 2000 38.5 / 33.2; 1280 x 1024 (1.25 to a CU), K = 2000 31.2 / 30.6.
        if (small == 32) return launch_upd_gemm16<MmaF16Blk16, 32, 32, 2, 2, true>(c, "update_gemm_f16_small", Q, P, (int)kgroups, ea);
        const int64_t t64 = ((s.d_out + 63) / 64) * (int64_t)((s.d_in + 63) / 64);
        const int row64 = (s.d_in + 63) / 64;
        const bool split_k = t64 <= c->compute_units ? K > 512 : K > 1024 && row64 >= 16 && row64 % 8 == 0 && 4 * t64 >= 7 * (int64_t)c->compute_units;
        if (!split_k) return launch_upd_gemm16<MmaF16Blk16, 64, 64, 2, 2, true>(c, "update_gemm_f16_small", Q, P, (int)kgroups, ea);
        return launch_upd_small<MmaF16, 64>(c, "update_gemm_f16_small", Q, P, (int)kgroups, ea);
    }
    if (small == 32) return launch_upd_small<MmaF32, 32>(c, "update_gemm_f32", Q, P, (int)kgroups, ea);
    if (small) return launch_upd_small<MmaF32, 64>(c, "update_gemm_f32", Q, P, (int)kgroups, ea);
    if (bf) {
        if (big_tiles(s.d_in, s.d_out, c->compute_units)) return launch_upd_gemm16<MmaF16Blk16, 256, 256, 2, 4, false>(c, "update_gemm_f16", Q, P, (int)kgroups, ea);
        if (((s.d_out + 127) / 128) * (int64_t)((s.d_in + 127) / 128) <= c->compute_units)
            return launch_upd_gemm16<MmaF16Blk16, 128, 128, 2, 2, true>(c, "update_gemm_f16_small", Q, P, (int)kgroups, ea);
        // one to two 128 x 128 tiles per CU: 32x32 blocks, stores entry by entry.  The 16x16 form with two workgroups per CU is better
        // at middling K and worse at both ends (whole updates, us, this / that): 3072 x 2048, K = 8192 175 / 166, 32768 662 / 682;
        // 4096 x 2048, K = 256 23.7 / 26.0, 4096 114 / 107; 3000 x 2700, K = 2000 75 / 75.
        return launch_upd_gemm<MmaF16, 128, 128, 2, 2>(c, "update_gemm_f16_small", P, Q, (int)kgroups, ea);
    }
    if (narrow_f32_tiles(s.d_out, s.d_in, c->compute_units)) return launch_upd_gemm<MmaF32, 128, 64, 2, 2>(c, "update_gemm_f32", P, Q, (int)kgroups, ea);
    return launch_upd_gemm<MmaF32, 128, 128, 2, 2>(c, "update_gemm_f32", P, Q, (int)kgroups, ea);
}

}  // namespace egg
