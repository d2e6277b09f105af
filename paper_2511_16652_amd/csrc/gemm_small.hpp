// NT contractions for products too small to fill the chip with the tiles of gemm_core.hpp:  C[m][n] = sum_k P[m][k] Q[n][k], in two forms: K split over the
// waves of a tile (fp32 updates of few tiles, and bf16 ones of 64 x 64 tiles with deep K), and, at the end, the tiles with four stages of K in LDS
// that keep K whole (layers; the updates that run them are chosen in k_update.hip).
//
// gemm_small_kernel: a workgroup owns a T x T tile (T = 32 or 64) and its four waves split K: each takes a quarter of it over the whole tile,
// reads its MFMA fragments straight from memory into registers (no LDS stages and no barrier in the loop: a wave alone on its
// SIMD would spend them waiting), and the four partial tiles are added through LDS, from which every thread finishes
// groups of 4 consecutive m of one n.  What bounds these calls is latency -- the length of a wave's chain of loads and MFMAs --
// and the number of workgroups: a 256 x 256 x 4096 update is 64 workgroups of a quarter of K here, 4 of all of K at 128 x 128.
// Updates only: their K is the population, so that a call's sums are those of its members anyway; a forward layer keeps K whole.
#pragma once
#include "gemm_core.hpp"

namespace egg {

// Tile of a small update of M x N, in whichever of the two forms; 0 where the tiles of 128 and more do better.  Measured over 256 .. 4096 rows and
// columns and K of 64 .. 4096 on 256 CUs (us, gemm_small_kernel in bf16 against those; the lines lie where the last listed shape still gains; the tiles with four
// stages, which bf16 takes now but for deep K, are faster than it and so gain up to the same lines at least):
//   32: up to two tiles per CU   256 x 256 x 4096: 26 / 56
//   64: up to two tiles per CU   2048 x 1024 x 4096: 57 / 68 (2048 x 2048: 86 / 78)
inline int small_tile(int64_t M, int64_t N, int compute_units)
{
    if (((M + 31) / 32) * ((N + 31) / 32) <= 2 * (int64_t)compute_units) return 32;
    return ((M + 63) / 64) * ((N + 63) / 64) <= 2 * (int64_t)compute_units ? 64 : 0;
}

// Epi requirements: struct Args; __device__ Epi(const Args&); value_t; __device__ void apply4(int m, int n, const value_t (&v)[4]),
// rows m .. m + 3 of column n, called once per in-range group (m < P.rows, n < Q.rows; P.rows may end inside the group).
template <class MT, int T, class Epi>
__global__ __launch_bounds__(256, 2) void gemm_small_kernel(Operand P, Operand Q, int kchunks, int tiles_m, typename Epi::Args ea)
{
    static_assert(MT::BLK == 32 && (T == 32 || T == 64), "32x32 MFMA blocks");
    constexpr int B = T / 32;
    constexpr int U = 4;                     // k-steps in flight: one batch is loaded while the other is multiplied
    constexpr int PITCH = T * 4 + 16;        // bytes per column of a partial tile
    __shared__ __attribute__((aligned(16))) char lds[4 * T * PITCH];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = (int)(blockIdx.x % tiles_m) * T, n0 = (int)(blockIdx.x / tiles_m) * T;
    const int fr = lane & 31, fc = lane >> 5;  // a k-step is two 16-byte chunks, one per lane half

    const char* pa[B];
    const char* qa[B];
#pragma unroll
    for (int i = 0; i < B; ++i) {
        pa[i] = P.base + (int64_t)min(m0 + i * 32 + fr, P.rows - 1) * P.row_stride;  // rows past the end re-read the last one
        qa[i] = Q.base + (int64_t)min(n0 + i * 32 + fr, Q.rows - 1) * Q.row_stride;
    }
    typename MT::acc_t acc[B][B];
#pragma unroll
    for (int i = 0; i < B; ++i)
#pragma unroll
        for (int j = 0; j < B; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;

    const int steps = (kchunks + 1) / 2, per = (steps + 3) / 4;
    const int s0 = min(wave * per, steps), s1 = min(s0 + per, steps);
    struct Batch {
        u32x4 a[U][B], b[U][B];
    };
    // k-steps s .. s + U - 1; those past the wave's range (or chunks past the end of K) count as zero
    auto load = [&](Batch& f, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t c = min((s + u) * 2 + fc, kchunks - 1);  // unconditional, from a clamped chunk
#pragma unroll
            for (int i = 0; i < B; ++i) {
                f.a[u][i] = *(const u32x4*)(pa[i] + c * P.kc_stride);
                f.b[u][i] = *(const u32x4*)(qa[i] + c * Q.kc_stride);
            }
        }
    };
    auto mul = [&](Batch& f, int s, bool tail) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (tail) {
                const bool in = s + u < s1 && (s + u) * 2 + fc < kchunks;
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    f.a[u][i] = in ? f.a[u][i] : u32x4{0u, 0u, 0u, 0u};
                    f.b[u][i] = in ? f.b[u][i] : u32x4{0u, 0u, 0u, 0u};
                }
            }
#pragma unroll
            for (int i = 0; i < B; ++i)
#pragma unroll
                for (int j = 0; j < B; ++j) MT::mma(f.a[u][i], f.b[u][j], acc[i][j]);
        }
    };
    if (s0 < s1) {
        Batch f0, f1;
        load(f0, s0);
        int s = s0;
        for (; s + 2 * U <= s1 && (s + 2 * U) * 2 <= kchunks; s += 2 * U) {  // two whole batches: nothing to mask
            load(f1, s + U);
            mul(f0, s, false);
            load(f0, s + 2 * U);  // (past the range: clamped and masked below, or never used)
            mul(f1, s + U, false);
        }
        for (; s < s1; s += U) {
            load(f1, s + U);
            mul(f0, s, true);
            f0 = f1;
        }
    }
#pragma unroll
    for (int i = 0; i < B; ++i)
#pragma unroll
        for (int j = 0; j < B; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                typedef typename Epi::value_t v4 __attribute__((ext_vector_type(4)));
                *(v4*)(lds + wave * T * PITCH + (j * 32 + fr) * PITCH + (i * 32 + q * 8 + fc * 4) * 4) =
                    v4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            }
    __syncthreads();
    Epi epi(ea);
#pragma unroll
    for (int it = 0; it < T * T / 1024; ++it) {
        const int g = it * 256 + tid, col = g / (T / 4), row = (g % (T / 4)) * 4;
        const int m = m0 + row, n = n0 + col;
        typename Epi::value_t v[4] = {0, 0, 0, 0};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            typedef typename Epi::value_t v4 __attribute__((ext_vector_type(4)));
            const v4 x = *(const v4*)(lds + w * T * PITCH + col * PITCH + row * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] += x[e];
        }
        if (m < P.rows && n < Q.rows) epi.apply4(m, n, v);
    }
}

// Products of few tiles that have to keep K whole (a layer's outputs must not depend on how many rows a call has): a workgroup of four waves
// to a tile of 32 x 32 or 64 x 64, a wave to a quarter of it, four stages of K in flight through LDS, several workgroups to a CU.  Every
// output is the one ascending chain of MFMAs that the large tiles run.  What bounds such a product is the latency of its loads and how
// many CUs share them: tiles of 128 leave most CUs empty, fragments straight from memory waited for every eighth k-step (us, whole layers
// at rank 2, before / 32 / 64: 328 outputs of 8192, 64 rows 72 / 27 / 38, 1580 rows 73 / 48 / 43, 2816 rows 75 / 57 / 58; 2048 x 2048, 512 rows
// 25.7 / 20.5 / 18.2, 1024 rows 26.3 / 30.8 / 23.4; 1696 of 5664, 512 rows 57 / 52 / 34; one row per member 1024 x 1024, 486 rows at rank 1 21.4
// / 9.4 / 11.0; 2048 of 4096, 900 rows at rank 4 65 / 61 / 46).  So: 32 up to two tiles a CU, 64 up to one, 32 again up to four
// (ragged shapes), 64 up to two where there are outputs enough that rows are not read from memory alone (256 outputs of 2048, 4800 rows
// 27.8 in tiles of 128 / 32.6; 328 of 8192, 4800 rows 81 / 104).  0: larger tiles.
inline int deep_tile(int64_t M, int64_t N, int compute_units)
{
    const int64_t t32 = ((M + 31) / 32) * ((N + 31) / 32), t64 = ((M + 63) / 64) * ((N + 63) / 64), cu = compute_units;
    if (t32 <= 2 * cu) return 32;
    if (t64 <= cu) return 64;
    if (t32 <= 4 * cu) return 32;
    return t64 <= 2 * cu && M >= 512 ? 64 : 0;
}

// An epilogue for 4 outputs of a row (extra, apply4) applied straight from the accumulators, for the kernel of one small tile per workgroup
template <class Row>
struct DirectEpi {
    typedef float value_t;
    typedef typename Row::Args Args;
    const Row row;
    static constexpr __host__ __device__ int lds_per_wave(int) { return 0; }
    __device__ __forceinline__ DirectEpi(const Args& a, char*, int) : row(a) {}
    template <int MB, int NB>
    __device__ __forceinline__ void prefetch(int, int, int, int) {}
    template <class MT, int MB, int NB>
    __device__ __forceinline__ void extra_mma(typename MT::acc_t (&acc)[MB][NB], int m0, int n0, int lane, int n_rows)
    {
        static_for<0, MB>([&](auto ic) __attribute__((always_inline)) {
            static_for<0, NB>([&](auto jc) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value, j = decltype(jc)::value;
                row.template extra<MT>(acc[i][j], m0 + i * 16, n0 + j * 16, lane, n_rows);
            });
        });
    }
    template <int J>
    __device__ __forceinline__ void column_at(int, bool) {}
    template <int I, int J>
    __device__ __forceinline__ void store4_at(int m, int n, const float (&v)[4], bool valid, int) const
    {
        if (valid && m < row.a.d_out) row.apply4(m, n, v);
    }
    template <int W>
    __device__ __forceinline__ void flush(int, int, int) {}
};

template <class MT, class Row, int T>
egg_status launch_gemm_deep(eggroll_ctx* c, const char* name, const Operand& P, const Operand& Q, int kchunks, const typename Row::Args& ea)
{
    auto kern = gemm_nt_deep_kernel<MT, T, T, 2, 2, false, DirectEpi<Row>>;
    const int tiles_m = (P.rows + T - 1) / T, tiles_n = (Q.rows + T - 1) / T;
    const size_t lds = 2 * gemm_lds_bytes<T, T>();
    // (bf16 rows of any length in tiles of 32; fp32 rows of 32 M values and more are refused in every tile)
    if (!(T == 32 && Row::IS_BF16) && (!operand_offsets_fit(P, T) || !operand_offsets_fit(Q, T))) return fail(c, EGG_EUNSUPPORTED, "operand strides too large for 32-bit tile offsets");
    const egg_status st = ensure_dynamic_lds(c, (const void*)kern, lds, "gemm smem attr");
    if (st != EGG_OK) return st;
    KernelScope ks(c, shaped_name(c, name, P.rows, kchunks * (Row::IS_BF16 ? 8 : 4)));
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(256), lds, c->stream, P, Q, kchunks, tiles_m, tiles_n,
                       (const char*)c->zero_page.p, c->conservative_waits ? 1 : 0, ea);
    return check_hip(c, hipGetLastError(), name);
}

}  // namespace egg
