// Projection pre-pass of the population forward:  t[q][l] = sum_k X[q][k] * B_i[k][l]
// (Sec. 4.2: for r = 1 "a batch of N vector-vector dot products of length d_in"; the B x r
// intermediate of the arithmetic-intensity appendix).  One workgroup per member: B_i is regenerated
// once into LDS (and optionally kept in the caller's cache), then the member's S rows are streamed
// against it, one wave per row (members with many rows share them among several workgroups, project_split).  HBM-bound on X for large S, integer-ALU bound (noise) for S = 1.
// With antithetic pairs a workgroup owns a pair: the factors are generated once for its 2S rows.
#include "common.hpp"
#include <algorithm>

namespace egg {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// workgroups past the members': 256 pieces each of the vectors drawn along (project_draws_along)
template <bool BF16>
__device__ __forceinline__ void draw_along(const NoisePiece& J, uint32_t member_begin)
{
    const uint32_t i = (blockIdx.x - J.first_wg) * 256u + threadIdx.x;
    if (i >= J.total) return;
    const uint32_t m = fast_div(J.per_member, i);
    J.out[i] = normal_piece<BF16>(J.key, member_begin + m, (i - m * J.per_member.d) * (BF16 ? 4 : 2));
}

// The rows of a member are shared among blockIdx.y workgroups, part_rows (a multiple of 4) to each; with READY its factors stand in B_cache.
// d_in is walked in panels of `panel` columns (a multiple of the 16-byte chunk, all of d_in when B_i fits the LDS budget):
// per panel B_i[k0 .. k0 + panel) is regenerated into LDS and the member's rows are streamed against it; with more than
// one panel the partial sums are carried in t itself (a row is always handled by the same wave).
// NR > 1, rank 8 and 16: phase 2 walks NR rows of a wave at once, so that a factor read from LDS serves them all -- a row alone reads
// 8 or 16 times its own bytes from there -- and asks for the next step's pieces of the rows before it multiplies this step's, the
// first step's before the factors are generated.  Rows past the last are repeated, not stored; the order of a row's additions
// does not depend on NR.  Whole calls of layers with 256 outputs
// (us, one row at a time / this): bf16 64 members x 128 rows of 4096, rank 16: 244 / 173; 256 x 64 of 8192, rank 8: 172 / 164; fp32
// 64 x 64 of 2048, rank 8: 143 / 109; 1024 -> 1024, 256 x 16, rank 8: 30.7 / 29.1.
// Below rank 8, and with one row to a wave, the loop over rows one at a time is as fast or faster (the registers of the deeper
// form cost more waves than its loads hide: 64 rows of 2048 at rank 4 74.6 us against 68.3).
template <bool BF16, int RANK, int NR, bool READY>
__global__ __launch_bounds__(256) void project_kernel(StreamKey kb, uint32_t member_begin, int S_all, int part_rows, int anti_rows, int d_in,
                                                      int panel, const void* __restrict__ X, float* __restrict__ t,
                                                      void* __restrict__ B_cache, NoisePiece along)
{
    if (blockIdx.x >= along.first_wg) return draw_along<BF16>(along, member_begin);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x;
    const int64_t ml = blockIdx.x;  // local member
    if (!READY && blockIdx.y) B_cache = nullptr;  // (the first part fills it)
    const int s_first = (int)blockIdx.y * part_rows, S = min(S_all, s_first + part_rows);
    const uint32_t member = member_begin + (uint32_t)ml;
    constexpr int EPC = BF16 ? 8 : 4;  // elements per 16-byte chunk of X (d_in is a multiple of it)
    // bf16 with more than one rank term: the panel sits in LDS rank-major ([l][column]), so that a 16-byte read holds the
    // same 8 columns as the chunk of the row and each pair of columns is one packed dot product (v_dot2c_f32_bf16)
    // instead of two unpacked multiply-adds: the pass was vector-ALU bound on unpacking (2.5 TB/s at rank 4).
    constexpr bool TRANSPOSED = BF16 && RANK >= 2;
    const int lane = tid & 63, wave = tid >> 6;
    constexpr int U = 2;  // chunks of a row per step (NR > 1)
    constexpr int BLOCKS_PER_PIECE = TRANSPOSED ? 8 : BF16 ? 4 : 2;
    // columns 8 c8 .. 8 c8 + 7 of rank terms l and l + 1, a word per column -> the rank-major panel of kn columns
    auto put_columns = [&](int c8, int l, int kn, const uint32_t (&pk)[8]) __attribute__((always_inline)) {
        u32x4 r0, r1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            r0[e] = (pk[2 * e] & 0xFFFFu) | (pk[2 * e + 1] << 16);
            r1[e] = (pk[2 * e] >> 16) | (pk[2 * e + 1] & 0xFFFF0000u);
        }
        *(u32x4*)((uint16_t*)smem + (int64_t)l * kn + c8 * 8) = r0;
        *(u32x4*)((uint16_t*)smem + (int64_t)(l + 1) * kn + c8 * 8) = r1;
    };

    for (int k0 = 0; k0 < d_in; k0 += panel) {
        const int kn = min(panel, d_in - k0);     // columns of this panel
        const int chunks = kn / EPC;
        const int steps = (chunks + 64 * U - 1) / (64 * U);  // per batch of rows
        // rows s0, s0 + 4, ..; pieces past the end are clamped to the last one and not multiplied
        auto load = [&](int s0, int ch0, uint4 (&x)[NR][U]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                const int64_t row = ml * S_all + min(s0 + 4 * j, S - 1);
                const uint4* xr = (const uint4*)((const char*)X + (row * (int64_t)d_in + k0) * (BF16 ? 2 : 4));
#pragma unroll
                for (int u = 0; u < U; ++u) x[j][u] = xr[min(ch0 + lane + 64 * u, chunks - 1)];
            }
        };
        uint4 xn[NR][U];
        if constexpr (NR > 1) load(s_first + wave, 0, xn);
        const int n = kn * RANK;                  // even: d_in and panel are multiples of 4
        const int first = k0 * RANK;              // flat index of the panel's first factor entry (even)
        if (k0) __syncthreads();                  // every wave is done with the previous panel
        // ---- phase 1: B_i panel -> LDS (storage dtype), optional cache ---------------------------
        if constexpr (READY) {
            if constexpr (TRANSPOSED) {
                // as below: 8 columns of two neighbouring rank terms, one word each
                constexpr int LP = RANK / 2;
                const uint32_t* const src = (const uint32_t*)B_cache + (ml * (int64_t)d_in * RANK + first) / 2;
                for (int i = tid; i < (kn >> 3) * LP; i += 256) {
                    const int c8 = i / LP, l = (i % LP) * 2;
                    uint32_t pk[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) pk[e] = src[((c8 * 8 + e) * RANK + l) >> 1];
                    put_columns(c8, l, kn, pk);
                }
            } else {
                const uint4* const src = (const uint4*)((const char*)B_cache + (ml * (int64_t)d_in * RANK + first) * (BF16 ? 2 : 4));
                for (int i = tid; i < n / EPC; i += 256) ((uint4*)smem)[i] = src[i];
            }
        } else
        // A thread expands several independent Threefry blocks and writes 16-byte pieces.
        // Where that would leave half of the threads without a piece, each expands one block at a time instead (512 columns at rank 1:
        // 64 pieces; the pass over 1618 antithetic pairs 5.7 us by pieces, 5.0 so).
        if ((n >> 1) <= 128 * BLOCKS_PER_PIECE) {
            for (int i = tid; i < (n >> 1); i += 256) {
                const int gb = (first >> 1) + i;
                uint32_t w0, w1;
                noise_words(kb, member, (uint32_t)gb, w0, w1);
                float z0, z1;
                normal_pair<!BF16>(w0, w1, z0, z1);
                if constexpr (BF16) {
                    const uint32_t pk = pack_bf16x2(z0, z1);
                    if constexpr (TRANSPOSED) {
                        const int col = 2 * i / RANK, l = 2 * i % RANK;
                        ((uint16_t*)smem)[(int64_t)l * kn + col] = (uint16_t)(pk & 0xFFFFu);
                        ((uint16_t*)smem)[(int64_t)(l + 1) * kn + col] = (uint16_t)(pk >> 16);
                    } else {
                        ((uint32_t*)smem)[i] = pk;
                    }
                    if (B_cache) ((uint32_t*)B_cache)[ml * (int64_t)((d_in * RANK) >> 1) + gb] = pk;
                } else {
                    ((float2*)smem)[i] = make_float2(z0, z1);
                    if (B_cache) ((float2*)B_cache)[ml * (int64_t)((d_in * RANK) >> 1) + gb] = make_float2(z0, z1);
                }
            }
        } else if constexpr (TRANSPOSED) {
            // one piece of two neighbouring rank terms: flat entries (column, l), (column, l + 1) are one block, so 8 columns
            // are 8 blocks and give 8 contiguous columns of rows l and l + 1 of the rank-major panel
            constexpr int LP = RANK / 2;
            for (int i = tid; i < (kn >> 3) * LP; i += 256) {
                const int c8 = i / LP, l = (i % LP) * 2;
                uint32_t pk[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int gb = (first + (c8 * 8 + e) * RANK + l) >> 1;  // Threefry block of the member's vector
                    uint32_t w0, w1;
                    noise_words(kb, member, (uint32_t)gb, w0, w1);
                    float z0, z1;
                    normal_pair<false>(w0, w1, z0, z1);
                    pk[e] = pack_bf16x2(z0, z1);
                    if (B_cache) ((uint32_t*)B_cache)[ml * (int64_t)((d_in * RANK) >> 1) + gb] = pk[e];
                }
                put_columns(c8, l, kn, pk);
            }
        } else {
            constexpr int BPP = BF16 ? 4 : 2;     // blocks per 16-byte piece of the flat vector
            for (int i = tid; i < (n >> 1) / BPP; i += 256) {
                u32x4 o;
#pragma unroll
                for (int e = 0; e < BPP; ++e) {
                    uint32_t w0, w1;
                    noise_words(kb, member, (uint32_t)((first >> 1) + i * BPP + e), w0, w1);
                    float z0, z1;
                    normal_pair<!BF16>(w0, w1, z0, z1);
                    if constexpr (BF16) {
                        o[e] = pack_bf16x2(z0, z1);
                    } else {
                        o[2 * e] = __float_as_uint(z0);
                        o[2 * e + 1] = __float_as_uint(z1);
                    }
                }
                ((u32x4*)smem)[i] = o;
                if (B_cache) *(u32x4*)((char*)B_cache + (ml * (int64_t)d_in * RANK + first) * (BF16 ? 2 : 4) + (int64_t)i * 16) = o;
            }
        }
        __syncthreads();

        // ---- phase 2: one wave per row ------------------------------------------------------------
        // the sums of a row over the wave's lanes
        auto finish = [&](int s, float (&a)[RANK]) __attribute__((always_inline)) {
            const int64_t row = ml * S_all + s;
#pragma unroll
            for (int l = 0; l < RANK; ++l) {
                const float v = wave_sum(a[l]);  // (at rank 1 the order of the normalisation pass, which forms the same projections)
                // antithetic pairs: the workgroup owns both members of a pair (2 x anti_rows rows); the second
                // member is evaluated at -sigma, which is folded into its projections
                if (lane == 0) {
                    const float sv = (anti_rows && s >= anti_rows) ? -v : v;
                    t[row * RANK + l] = k0 ? t[row * RANK + l] + sv : sv;
                }
            }
        };
      if constexpr (NR == 1) {
        for (int s = s_first + wave; s < S; s += 4) {
            const int64_t row = ml * S_all + s;
            const uint4* xr = (const uint4*)((const char*)X + (row * (int64_t)d_in + k0) * (BF16 ? 2 : 4));
            float acc[RANK];
#pragma unroll
            for (int l = 0; l < RANK; ++l) acc[l] = 0.f;
            // (four iterations at a time, so that a lane has four 16-byte loads of the row in flight: with one, the pass
            // ran at 2.5 TB/s on rows of 8192 values; the order of the additions is unchanged)
#pragma unroll 4
            for (int ch = lane; ch < chunks; ch += 64) {
                const uint4 xv = xr[ch];
                if constexpr (TRANSPOSED) {
                    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                    const uint32_t xw[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
                    for (int l = 0; l < RANK; ++l) {
                        const uint4 q = *(const uint4*)((const uint16_t*)smem + (int64_t)l * kn + (int64_t)ch * 8);
                        const uint32_t bw[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            acc[l] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, xw[e]), __builtin_bit_cast(bf16x2, bw[e]), acc[l], false);
                    }
                    continue;
                }
                float x[EPC];
                if constexpr (BF16) {
                    const uint32_t w[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        x[2 * e] = __uint_as_float(w[e] << 16);
                        x[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
                    }
                } else {
                    x[0] = __uint_as_float(xv.x); x[1] = __uint_as_float(xv.y);
                    x[2] = __uint_as_float(xv.z); x[3] = __uint_as_float(xv.w);
                }
                // B_i[k][l] for the chunk's k range: EPC*RANK consecutive elements = RANK 16-byte reads
                const uint4* bp = (const uint4*)smem + (int64_t)ch * RANK;
#pragma unroll
                for (int v = 0; v < RANK; ++v) {
                    const uint4 q = bp[v];
                    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
                    // the 16 bytes hold flat entries v*EPC .. of the chunk: entry f belongs to column f / RANK, rank term f % RANK
                    if constexpr (BF16) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int f = v * 8 + e;
                            const float bv = (e & 1) ? __uint_as_float(w[e >> 1] & 0xFFFF0000u) : __uint_as_float(w[e >> 1] << 16);
                            acc[f % RANK] = fmaf(x[f / RANK], bv, acc[f % RANK]);
                        }
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int f = v * 4 + e;
                            acc[f % RANK] = fmaf(x[f / RANK], __uint_as_float(w[e]), acc[f % RANK]);
                        }
                    }
                }
            }
            finish(s, acc);
        }
      } else {
        for (int s0 = s_first + wave; s0 < S; s0 += 4 * NR) {
            float acc[NR][RANK];
#pragma unroll
            for (int j = 0; j < NR; ++j)
#pragma unroll
                for (int l = 0; l < RANK; ++l) acc[j][l] = 0.f;
            for (int st = 0; st < steps; ++st) {
                uint4 xc[NR][U];
#pragma unroll
                for (int j = 0; j < NR; ++j)
#pragma unroll
                    for (int u = 0; u < U; ++u) xc[j][u] = xn[j][u];
                if (st + 1 < steps) load(s0, (st + 1) * 64 * U, xn);
                else if (s0 + 4 * NR < S) load(s0 + 4 * NR, 0, xn);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int ch = (st * U + u) * 64 + lane;
                    if (ch >= chunks) break;
                    if constexpr (TRANSPOSED) {
                        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
                        for (int l = 0; l < RANK; ++l) {
                            const uint4 q = *(const uint4*)((const uint16_t*)smem + (int64_t)l * kn + (int64_t)ch * 8);
                            const uint32_t bw[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                            for (int j = 0; j < NR; ++j) {
                                const uint32_t xw[4] = {xc[j][u].x, xc[j][u].y, xc[j][u].z, xc[j][u].w};
#pragma unroll
                                for (int e = 0; e < 4; ++e)
                                    acc[j][l] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, xw[e]), __builtin_bit_cast(bf16x2, bw[e]), acc[j][l], false);
                            }
                        }
                    } else {
                        static_assert(!BF16, "bf16 of rank 2 and more is rank-major");
                        float x[NR][EPC];
#pragma unroll
                        for (int j = 0; j < NR; ++j) {
                            const uint32_t w[4] = {xc[j][u].x, xc[j][u].y, xc[j][u].z, xc[j][u].w};
#pragma unroll
                            for (int e = 0; e < EPC; ++e) x[j][e] = __uint_as_float(w[e]);
                        }
                        // B_i[k][l] for the chunk's k range: EPC*RANK consecutive elements = RANK 16-byte reads
                        const uint4* bp = (const uint4*)smem + (int64_t)ch * RANK;
#pragma unroll
                        for (int v = 0; v < RANK; ++v) {
                            const uint4 q = bp[v];
                            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
                            // the 16 bytes hold flat entries v*EPC .. of the chunk: entry f belongs to column f / RANK, rank term f % RANK
#pragma unroll
                            for (int e = 0; e < EPC; ++e) {
                                const int f = v * EPC + e;
#pragma unroll
                                for (int j = 0; j < NR; ++j) acc[j][f % RANK] = fmaf(x[j][f / RANK], __uint_as_float(w[e]), acc[j][f % RANK]);
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (s0 + 4 * j < S) finish(s0 + 4 * j, acc[j]);
        }
      }
    }
}

// One row per member and rank 1: nothing is shared between rows, so B_i never needs to sit in LDS.
// Each thread multiplies the factor pairs it generates with the matching x pair on the fly; one
// shuffle reduction per wave and a 4-entry LDS reduction finish the dot product.
template <bool BF16>
__global__ __launch_bounds__(256) void project_row_kernel(StreamKey kb, uint32_t member_begin, int d_in,
                                                          const void* __restrict__ X, float* __restrict__ t,
                                                          void* __restrict__ B_cache)
{
    __shared__ float red[4];
    const int tid = threadIdx.x;
    const int64_t ml = blockIdx.x;
    const uint32_t member = member_begin + (uint32_t)ml;
    const int pairs = d_in >> 1;
    float acc = 0.f;
    // one column pair; the order of the additions is that of b
    auto pair = [&](int b, uint2 xv) __attribute__((always_inline)) {
        uint32_t w0, w1;
        noise_words(kb, member, (uint32_t)b, w0, w1);
        float z0, z1;
        normal_pair<!BF16>(w0, w1, z0, z1);
        if constexpr (BF16) {
            const uint32_t pk = pack_bf16x2(z0, z1);
            acc = fmaf(bf16_lo(xv.x), bf16_lo(pk), acc);
            acc = fmaf(bf16_hi(xv.x), bf16_hi(pk), acc);
            if (B_cache) ((uint32_t*)B_cache)[ml * pairs + b] = pk;
        } else {
            acc = fmaf(__uint_as_float(xv.x), z0, acc);
            acc = fmaf(__uint_as_float(xv.y), z1, acc);
            if (B_cache) ((float2*)B_cache)[ml * pairs + b] = make_float2(z0, z1);
        }
    };
    auto xload = [&](int b) __attribute__((always_inline)) {
        if constexpr (BF16) return make_uint2(((const uint32_t*)X)[ml * pairs + b], 0u);
        else return ((const uint2*)X)[ml * pairs + b];
    };
    int b = tid;
    // four at a time: their loads and their generator chains are independent (one at a time, 4096 members x 4096 columns took
    // 32 us, of which the generator's issue slots are 19)
    for (; b + 768 < pairs; b += 1024) {
        uint2 xv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) xv[k] = xload(b + 256 * k);
#pragma unroll
        for (int k = 0; k < 4; ++k) pair(b + 256 * k, xv[k]);
    }
    for (; b < pairs; b += 256) pair(b, xload(b));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) t[ml] = (red[0] + red[1]) + (red[2] + red[3]);
}

// One row per member (NR = 1) or a pair of them (NR = 2, antithetic: the second at -sigma), rank >= 2.  As above nothing is
// shared, so B_i does not go through LDS: a thread expands a 16-byte piece of the flat vector -- EPP consecutive entries, a few
// columns times the rank, or part of one column -- and multiplies it with the matching x at once, all 256 threads; the LDS form
// left the row to one wave of four.  Vector-ALU bound (the generator).  Measured at 1024 members x 8192 x rank 4 (bf16): 55 us,
// 64 in the LDS form.
template <bool BF16, int RANK, int NR>
__global__ __launch_bounds__(256) void project_rows_rank_kernel(StreamKey kb, uint32_t member_begin, int d_in, const void* __restrict__ X,
                                                                float* __restrict__ t, void* __restrict__ B_cache, NoisePiece along)
{
    if (blockIdx.x >= along.first_wg) return draw_along<BF16>(along, member_begin);
    constexpr int EPP = BF16 ? 8 : 4, BPP = EPP / 2;
    constexpr int NL = RANK < EPP ? RANK : EPP;         // rank terms a thread meets
    constexpr int PPC = RANK > EPP ? RANK / EPP : 1;    // pieces per column
    constexpr int CPP = RANK < EPP ? EPP / RANK : 1;    // columns per piece
    static_assert(RANK >= 2 && 256 % PPC == 0, "a thread keeps its rank terms from one piece to the next");
    __shared__ float red[4][NR][RANK];
    const int tid = threadIdx.x;
    const int64_t ml = blockIdx.x;
    const uint32_t member = member_begin + (uint32_t)ml;
    const int pieces = d_in * RANK / EPP;
    float acc[NR][NL];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int l = 0; l < NL; ++l) acc[r][l] = 0.f;
    for (int p = tid; p < pieces; p += 256) {
        const int col = PPC > 1 ? p / PPC : p * CPP;
        float x[NR][CPP];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int64_t at = (ml * NR + r) * d_in + col;
#pragma unroll
            for (int k = 0; k < CPP; ++k) {
                if constexpr (BF16) x[r][k] = bf16_bits_to_f32(((const uint16_t*)X)[at + k]);
                else x[r][k] = ((const float*)X)[at + k];
            }
        }
        float z[EPP];
        u32x4 o;
#pragma unroll
        for (int b = 0; b < BPP; ++b) {
            uint32_t w0, w1;
            noise_words(kb, member, (uint32_t)(p * BPP + b), w0, w1);
            normal_pair<!BF16>(w0, w1, z[2 * b], z[2 * b + 1]);
            if constexpr (BF16) {
                const uint32_t pk = pack_bf16x2(z[2 * b], z[2 * b + 1]);
                o[b] = pk;
                z[2 * b] = bf16_lo(pk);
                z[2 * b + 1] = bf16_hi(pk);
            } else {
                o[2 * b] = __float_as_uint(z[2 * b]);
                o[2 * b + 1] = __float_as_uint(z[2 * b + 1]);
            }
        }
        if (B_cache) ((u32x4*)B_cache)[ml * pieces + p] = o;
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int f = 0; f < EPP; ++f) acc[r][f % NL] = fmaf(x[r][PPC > 1 ? 0 : f / RANK], z[f], acc[r][f % NL]);
    }
    const int l0 = PPC > 1 ? (tid % PPC) * EPP : 0;
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            float v = acc[r][l];
#pragma unroll
            for (int off = 32; off >= PPC; off >>= 1) v += __shfl_xor(v, off, 64);  // lanes that hold the same rank terms
            if ((tid & 63) < PPC) red[tid >> 6][r][l0 + l] = v;
        }
    __syncthreads();
    if (tid < NR * RANK) {
        const int r = tid / RANK, l = tid % RANK;
        const float v = (red[0][r][l] + red[1][r][l]) + (red[2][r][l] + red[3][r][l]);
        t[(ml * NR + r) * RANK + l] = r == 1 ? -v : v;
    }
}

// The same projection for 8 consecutive members per workgroup, with B leaving the kernel as the K-packed fp16
// panel the update contracts ([member / 8][k][member % 8]).  512 threads: thread (b, half) generates the column
// pair (2b, 2b+1) of members 4 half .. 4 half + 3 and stores its 8 bytes of the two 16-byte chunks, which are
// neighbours in the panel.  The first 256 threads (half 0) and the last 256 (half 1) each hold the 256 b-lanes
// in the order of project_row_kernel, and every member's partial sums go through the same shuffle tree and the
// same final additions, so t is bit-identical to that kernel's.
__global__ __launch_bounds__(512) void project_row8_kernel(StreamKey kb, uint32_t member_begin, int64_t members, int d_in,
                                                           const void* __restrict__ X, float* __restrict__ t,
                                                           u32x4* __restrict__ panel)
{
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    __shared__ float red[4][8];
    const int tid = threadIdx.x;
    const int half = tid >> 8, bl = tid & 255;
    const int64_t g = blockIdx.x;
    const int pairs = d_in >> 1;
    float acc[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = 0.f;
    for (int b = bl; b < pairs; b += 256) {
        float lo[4], hi[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t i = g * 8 + half * 4 + e;
            lo[e] = hi[e] = 0.f;
            if (i < members) {
                uint32_t w0, w1;
                noise_words(kb, member_begin + (uint32_t)i, (uint32_t)b, w0, w1);
                float z0, z1;
                normal_pair<false>(w0, w1, z0, z1);
                const uint32_t pk = pack_bf16x2(z0, z1);
                const uint32_t xv = ((const uint32_t*)X)[i * pairs + b];
                acc[e] = fmaf(bf16_lo(xv), bf16_lo(pk), acc[e]);
                acc[e] = fmaf(bf16_hi(xv), bf16_hi(pk), acc[e]);
                lo[e] = bf16_lo(pk);
                hi[e] = bf16_hi(pk);
            }
        }
        uint2 c0, c1;
        {
            h2 p, q;
            p[0] = (_Float16)lo[0]; p[1] = (_Float16)lo[1];
            q[0] = (_Float16)lo[2]; q[1] = (_Float16)lo[3];
            c0.x = __builtin_bit_cast(uint32_t, p); c0.y = __builtin_bit_cast(uint32_t, q);
            p[0] = (_Float16)hi[0]; p[1] = (_Float16)hi[1];
            q[0] = (_Float16)hi[2]; q[1] = (_Float16)hi[3];
            c1.x = __builtin_bit_cast(uint32_t, p); c1.y = __builtin_bit_cast(uint32_t, q);
        }
        uint2* o = (uint2*)(panel + g * d_in + 2 * b) + half;   // bytes 8 half .. 8 half + 7 of chunk 2b
        o[0] = c0;
        o[2] = c1;                                              // the same bytes of chunk 2b + 1
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) acc[e] += __shfl_xor(acc[e], off, 64);
    }
    if ((tid & 63) == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) red[bl >> 6][half * 4 + e] = acc[e];
    }
    __syncthreads();
    if (tid < 8 && g * 8 + tid < members) t[g * 8 + tid] = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
}

constexpr int64_t PANEL_BYTES = 128 * 1024;  // B_i of a member in LDS, at most

template <bool BF16>
static egg_status launch_project_t(eggroll_ctx* c, const StreamKey& kb, const egg_shape& shape, const void* X, float* t,
                                   void* B_cache, bool panel, const ProjectSplit& split, const NoisePiece* with)
{
    if (panel && B_cache) {  // (bf16, rank 1, one row per member, no pairs: checked_forward)
        const int64_t groups = (shape.member_count + 7) / 8;
        if (groups > 0x7FFFFFFF) return fail(c, EGG_EUNSUPPORTED, "too many members in one call");
        KernelScope ks(c, "project");
        hipLaunchKernelGGL(project_row8_kernel, dim3((unsigned)groups), dim3(512), 0, c->stream, kb, (uint32_t)shape.member_begin,
                           shape.member_count, shape.d_in, X, t, (u32x4*)B_cache);
        return check_hip(c, hipGetLastError(), "project launch");
    }
    egg_shape s = shape;  // the noise view: pairs as members of 2S rows when antithetic
    const int anti_rows = shape.antithetic ? shape.rows_per_member : 0;
    if (shape.antithetic) {
        s.member_begin /= 2;
        s.member_count /= 2;
        s.rows_per_member *= 2;
    }
    // all of d_in when its panel fits, else the largest multiple of 64 columns
    const int esz = BF16 ? 2 : 4;
    int kpanel = s.d_in;
    if ((int64_t)s.d_in * s.rank * esz > PANEL_BYTES) kpanel = (int)(PANEL_BYTES / (s.rank * esz)) / 64 * 64;
    const size_t lds = (size_t)kpanel * s.rank * esz;
    if (s.member_count > 0x7FFFFFFF) return fail(c, EGG_EUNSUPPORTED, "too many members in one call");
    NoisePiece along{};
    if (with) along = *with;
    along.first_wg = (uint32_t)s.member_count;  // (past the grid without them)
    const dim3 g((unsigned)s.member_count + (along.total + 255u) / 256u, (unsigned)split.parts), b(256);  // (at most four parts to a CU)
    const uint32_t mb = (uint32_t)s.member_begin;
    if (s.rank == 1 && s.rows_per_member == 1) {
        KernelScope ks(c, "project");
        hipLaunchKernelGGL(project_row_kernel<BF16>, g, b, 0, c->stream, kb, mb, s.d_in, X, t, B_cache);
        return check_hip(c, hipGetLastError(), "project launch");
    }
    if (shape.rows_per_member == 1 && s.rank >= 2) {
        KernelScope ks(c, "project");
#define EGG_ROWS(R)                                                                                                                       \
    if (s.rank == R) {                                                                                                                    \
        if (shape.antithetic) hipLaunchKernelGGL((project_rows_rank_kernel<BF16, R, 2>), g, b, 0, c->stream, kb, mb, s.d_in, X, t, B_cache, along); \
        else hipLaunchKernelGGL((project_rows_rank_kernel<BF16, R, 1>), g, b, 0, c->stream, kb, mb, s.d_in, X, t, B_cache, along);               \
    }
        EGG_ROWS(2) EGG_ROWS(4) EGG_ROWS(8) EGG_ROWS(16)
#undef EGG_ROWS
        return check_hip(c, hipGetLastError(), "project launch");
    }
    // (rank 8 and 16) rows of a wave at once: four, or two, where the repeats this makes are at most an eighth of the rows (with more
    // the loop over single rows is level or faster: 5, 6, 9, 17 and 33 rows by 1 to 3 %)
    const int S = std::min(s.rows_per_member, split.rows);
    auto fits = [&](int k) { return (int64_t)(S + 4 * k - 1) / (4 * k) * (4 * k) * 8 <= (int64_t)S * 9; };
    const int nr = fits(4) ? 4 : fits(2) ? 2 : 1;
#define EGG_LAUNCH_PROJECT(R)                                                                                        \
    {                                                                                                                \
        auto kern = split.ready ? project_kernel<BF16, R, 1, true> : project_kernel<BF16, R, 1, false>;              \
        if constexpr (R >= 8) {                                                                                      \
            if (nr == 4) kern = split.ready ? project_kernel<BF16, R, 4, true> : project_kernel<BF16, R, 4, false>;  \
            if (nr == 2) kern = split.ready ? project_kernel<BF16, R, 2, true> : project_kernel<BF16, R, 2, false>;  \
        }                                                                                                            \
        if (lds > 48 * 1024) {                                                                                       \
            egg_status st = ensure_dynamic_lds(c, (const void*)kern, (size_t)lds, "project smem attr"); \
            if (st != EGG_OK) return st;                                                                             \
        }                                                                                                            \
        KernelScope ks(c, "project");                                                                                \
        hipLaunchKernelGGL(kern, g, b, lds, c->stream, kb, mb, s.rows_per_member, split.rows, anti_rows, s.d_in, kpanel, X, t, B_cache, along); \
    }
    switch (s.rank) {
        case 1: EGG_LAUNCH_PROJECT(1) break;
        case 2: EGG_LAUNCH_PROJECT(2) break;
        case 4: EGG_LAUNCH_PROJECT(4) break;
        case 8: EGG_LAUNCH_PROJECT(8) break;
        default: EGG_LAUNCH_PROJECT(16) break;
    }
#undef EGG_LAUNCH_PROJECT
    return check_hip(c, hipGetLastError(), "project launch");
}

// One workgroup per member leaves the chip idle where members are few and their rows many, so a member's rows are shared among as many
// workgroups as make four to a CU, or two where there are more than half as many members as CUs (a row still belongs to one wave, and its
// additions keep their order).  Every workgroup holds the whole panel of factors in LDS, which is drawn once by the noise kernel and
// read back (drawing it again in each cost as much as the rows: 4096 columns of rank 8 are 11 us); so that a part's rows are worth that,
// it has 8 rows or more, 16 where the panel is longer than 32 KB, 32 where it is walked in pieces or members are not that few.  Without a place for the factors they are
// drawn by every workgroup, one to a CU.  Whole calls of bf16 layers with 256 outputs, one workgroup per member / this (us): 22 x 128 rows
// of 8192, rank 1, pairs 175 / 74; 22 x 128 of 5664, rank 8 140 / 68; 25 x 178 of 400, rank 8 53 / 18; 109 x 20 of 1024, rank 16 38 / 30;
// 105 x 100 of 768, rank 1 35 / 20; 256 x 64 of 2048, rank 4 42.7 / 41.7.  Beyond: 300 x 40 of 512, rank 1 in four parts 19.9 / 17.6,
// but 400 x 64 of 2048, rank 4 56 / 63; and 256 x 16 of 1024, rank 8 in two parts of 8 23.6 / 25.4.
ProjectSplit project_split(const eggroll_ctx* c, const egg_shape& shape, egg_dtype io, bool ready)
{
    const int64_t ids = shape.antithetic ? shape.member_count / 2 : shape.member_count;
    const int S = shape.antithetic ? 2 * shape.rows_per_member : shape.rows_per_member;
    const ProjectSplit whole{1, S, false};
    const bool few = 2 * ids <= c->compute_units;
    const int64_t want = (int64_t)c->compute_units * (!ready ? 1 : few ? 4 : 2);
    if (shape.rows_per_member == 1 || ids <= 0 || 2 * ids > want) return whole;
    const int64_t panel = (int64_t)shape.d_in * shape.rank * (io == EGG_BF16 ? 2 : 4);
    const int least = few && panel <= 32 * 1024 ? 8 : few && panel <= PANEL_BYTES ? 16 : 32;
    const int64_t per = want / ids;
    const int rows = std::max((int)((S + per - 1) / per + 3) / 4 * 4, least);
    if (rows >= S) return whole;
    return ProjectSplit{(S + rows - 1) / rows, rows, ready};
}

// The factors A that the layer needs beside the projections do not depend on them: they are drawn in the same launch, by workgroups
// after the members'.  A launch of its own cost 3 us of the host's time and the chip ran empty before and after it.  Whole calls of bf16 layers
// (us, apart / along): 256 -> 256, 256 members x 4 rows, rank 4 13.0 / 9.1; 1024 -> 1024, 256 x 16, rank 8 27.6 / 24.0; 8192 -> 8192, 1024 x 1,
// rank 4 246.0 / 240.2; 1024 -> 1024, 4096 x 4, rank 16 243 / 237.  They take the LDS of the members' workgroups though, so where that leaves
// one workgroup on a CU, only up to four times the CUs of them: 8192 -> 2048, 64 x 16, rank 8 84.7 / 81.7, but 1000 x 4 267 / 272 and fp32
// 2048 -> 2048, 512 x 4, rank 16 263 / 293.  Where it leaves two of them, fp32 factors, whose normals take longer chains of instructions, only up to 80 times: 1024 -> 2048, 600 x 4,
// rank 16 (75 times) 210 / 205, 1000 x 2 (125 times) 188 / 197, 4096 x 2 676 / 727; in bf16 they are level at 256 times and gain below.  Rows in several parts have their factors, A too, from a launch before.
bool project_draws_along(const eggroll_ctx* c, const egg_shape& shape, egg_dtype io, const ProjectSplit& split, const NoisePiece& along)
{
    const int64_t ids = shape.antithetic ? shape.member_count / 2 : shape.member_count, wgs = (along.total + 255u) / 256u;
    if (split.parts > 1 || ids + wgs >= int64_t(1) << 24) return false;  // (2^32 threads to a launch)
    const int64_t lds = shape.rows_per_member == 1 && shape.rank > 1 ? 0 : (int64_t)shape.d_in * shape.rank * (io == EGG_BF16 ? 2 : 4);
    const int64_t most = lds > PANEL_BYTES / 2 ? 4 : io == EGG_F32 && 3 * lds > 160 * 1024 ? 80 : wgs;
    return wgs <= most * c->compute_units;
}

egg_status launch_project(eggroll_ctx* c, const StreamKey& kb, const egg_shape& s, egg_dtype io, const void* X,
                          float* t, void* B_cache, bool panel, const ProjectSplit& split, const NoisePiece* along)
{
    return io == EGG_BF16 ? launch_project_t<true>(c, kb, s, X, t, B_cache, panel, split, along)
                          : launch_project_t<false>(c, kb, s, X, t, B_cache, panel, split, along);
}

}  // namespace egg
