// NT contraction for products too small to fill the chip with the tiles of gemm_core.hpp:  C[m][n] = sum_k P[m][k] Q[n][k].
//
// A workgroup owns a T x T tile (T = 32 or 64) and its four waves split K: each takes a quarter of it over the whole tile,
// reads its MFMA fragments straight from memory into registers (no LDS stages and no barrier in the loop: a wave alone on its
// SIMD would spend them waiting), and the four partial tiles are added through LDS, from which every thread finishes
// groups of 4 consecutive m of one n.  What bounds these calls is latency -- the length of a wave's chain of loads and MFMAs --
// and the number of workgroups: a 256 x 256 x 4096 update is 64 workgroups of a quarter of K here, 4 of all of K at 128 x 128.
// Updates only: their K is the population, so that a call's sums are those of its members anyway; a forward layer keeps K whole.
#pragma once
#include "gemm_core.hpp"

namespace egg {

// Tile of the small kernel for an M x N product, 0 where the tiles of gemm_core.hpp do better.  Measured over 256 .. 4096 rows and
// columns and K of 64 .. 4096 on 256 CUs (us, this kernel against theirs; the lines lie where the last listed shape still gains):
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

// The same for the bf16 forward layer, whose outputs must not depend on how many rows a call has (a population may be walked in
// chunks): K is not split, every output is the one ascending chain of 16x16x32 MFMAs that the large tiles run.  A workgroup owns
// 32 x 32 outputs, a wave a 16 x 16 block of them over all of K, its fragments straight from memory, two batches of eight k-steps
// in flight; the chain itself is short (16 cycles a step).
// Epi: struct Args; Epi(const Args&); extra<MT>(acc, m0, n0, lane, n_rows) adds to the block's accumulators; apply4 as above.
template <class MT, class Epi>
__global__ __launch_bounds__(256, 2) void gemm_small16_kernel(Operand P, Operand Q, int kchunks, int tiles_m, typename Epi::Args ea)
{
    static_assert(MT::BLK == 16, "16x16 MFMA blocks");
    constexpr int U = 8;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = (int)(blockIdx.x % tiles_m) * 32 + (wave & 1) * 16, n0 = (int)(blockIdx.x / tiles_m) * 32 + (wave >> 1) * 16;
    if (m0 >= P.rows || n0 >= Q.rows) return;  // (no barrier in this kernel)
    const int fr = lane & 15, fc = lane >> 4;  // a k-step is four 16-byte chunks
    const char* pa = P.base + (int64_t)min(m0 + fr, P.rows - 1) * P.row_stride;  // rows past the end re-read the last one
    const char* qa = Q.base + (int64_t)min(n0 + fr, Q.rows - 1) * Q.row_stride;
    typename MT::acc_t acc;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = 0;
    struct Batch {
        u32x4 a[U], b[U];
    };
    auto load = [&](Batch& f, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t c = min((s + u) * 4 + fc, kchunks - 1);  // unconditional, from a clamped chunk
            f.a[u] = *(const u32x4*)(pa + c * P.kc_stride);
            f.b[u] = *(const u32x4*)(qa + c * Q.kc_stride);
        }
    };
    auto mul = [&](Batch& f, int s, bool tail) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (tail) {
                const bool in = (s + u) * 4 + fc < kchunks;
                f.a[u] = in ? f.a[u] : u32x4{0u, 0u, 0u, 0u};
                f.b[u] = in ? f.b[u] : u32x4{0u, 0u, 0u, 0u};
            }
            MT::mma(f.a[u], f.b[u], acc);
        }
    };
    const int steps = (kchunks + 3) / 4;
    Batch f0, f1;
    load(f0, 0);
    int s = 0;
    for (; (s + 2 * U) * 4 <= kchunks; s += 2 * U) {  // two whole batches: nothing to mask
        load(f1, s + U);
        mul(f0, s, false);
        load(f0, s + 2 * U);  // (past the end: clamped, and masked below or never used)
        mul(f1, s + U, false);
    }
    for (; s < steps; s += U) {
        load(f1, s + U);
        mul(f0, s, true);
        f0 = f1;
    }
    Epi epi(ea);
    epi.template extra<MT>(acc, m0, n0, lane, Q.rows);
    const int m = m0 + fc * 4, n = n0 + fr;
    const float v[4] = {acc[0], acc[1], acc[2], acc[3]};
    if (m < P.rows && n < Q.rows) epi.apply4(m, n, v);
}
// Up to one tile of 32 x 32 per CU the bf16 layer takes it (us, this kernel / 128 x 128 tiles): 16 rows per member 256 x 64 x 4096
// 41 / 46, 512 x 512 x 1024 19.7 / 20.6 (1024 x 512 x 1024: 28 / 21); one row per member 512 x 256 x 1024 14 / 24.
inline bool small16(int64_t M, int64_t N, int compute_units) { return ((M + 31) / 32) * ((N + 31) / 32) <= compute_units; }

}  // namespace egg
