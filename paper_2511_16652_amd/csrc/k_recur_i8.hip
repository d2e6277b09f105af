// The integer recurrent cell over many time steps in one kernel (App. "Matrix Multiplication", "Adding EGGROLL Perturbations";
// the arithmetic of k_int8.hip, bit-exact):
//   h <- clamp((h theta^T + ((h . B_i) A_i >> corr_shift)) >> out_shift, -127, 127),  T times.
// A member's row depends on no other member, so a workgroup that owns 32 rows can walk all time steps by itself: state, factors
// and dot products stay in LDS, and no kernel boundary, no operand tile and no factor row goes through memory between steps.
// What a step costs then is reading theta: d^2 bytes per workgroup.  Its MFMA fragments are kept in registers as far as they go
// -- all of them up to d = 512, 10 of 24 k blocks at d = 768, 6 of 32 at d = 1024 -- and the rest streams from L2 in fragment order (a small kernel lays theta
// out so at the start of the call: a fragment of the row-major matrix is 32 pieces of 32 bytes, a row apart).
// Bound: the MFMAs and one barrier up to d = 512; beyond, the rate at which a CU loads.
#include "common.hpp"
#include "gemm_core.hpp"

namespace egg {

constexpr int RECUR_ROWS = 32;

// theta row-major -> [column block][k block][lane][16 bytes]: lane l of a 32x32x32 MFMA holds row (l & 31) of the block, bytes
// 16 (l >> 5) .. + 15 of the k block; zero past d
__global__ __launch_bounds__(256) void pack_theta_kernel(const int8_t* __restrict__ W, int d, int nb, u32x4* __restrict__ out)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nb * nb * 64) return;
    const int lane = i & 63, kb = (i >> 6) % nb, cb = (i >> 6) / nb;
    const int j = cb * 32 + (lane & 31), k = kb * 32 + (lane >> 5) * 16;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (j < d && k < d) v = *(const u32x4*)(W + (int64_t)j * d + k);  // d is a multiple of 16: whole pieces
    out[i] = v;
}

// CB: column blocks of 32 per wave (eight waves): d <= 256 CB.  RES: k blocks whose fragments stay in registers.
template <int CB, int RES, int PF, bool DOT24>
__global__ __launch_bounds__(512, 1) void recur_i8_kernel(const u32x4* __restrict__ Wp, const int8_t* __restrict__ A,
                                                          const int8_t* __restrict__ B, int anti, int64_t rows, int d, int steps,
                                                          int corr_shift, int out_shift, const int8_t* H_in, int8_t* H_out)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int nb = (d + 31) >> 5, pitch = nb * 32 + 16;  // (rows 16 bytes apart modulo the banks: fragment reads do not collide)
    char* sh[2] = {lds, lds + RECUR_ROWS * pitch};
    char* sA = lds + 2 * RECUR_ROWS * pitch;
    char* sB = sA + RECUR_ROWS * pitch;
    int* part = (int*)(sB + RECUR_ROWS * pitch);  // [2][8 waves][32 rows]: shares of the next step's dot products
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t row0 = (int64_t)blockIdx.x * RECUR_ROWS;
    const int n = lane & 31, half = lane >> 5;
    const int cb0 = wave * CB;

    // theta fragments: resident ones now (blocks past the matrix stay zero)
    u32x4 wr[CB][RES];
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int kb = 0; kb < RES; ++kb) {
            wr[c][kb] = u32x4{0u, 0u, 0u, 0u};
            if (cb0 + c < nb && kb < nb) wr[c][kb] = Wp[((int64_t)(cb0 + c) * nb + kb) * 64 + lane];
        }
    // state and factors of the 32 rows (rows past the end re-read the last one; columns past d are zero)
    for (int i = tid; i < RECUR_ROWS * nb * 2; i += 512) {
        const int r = i / (nb * 2), k = (i - r * (nb * 2)) * 16;
        const int64_t row = min(row0 + r, rows - 1);
        u32x4 h = {0u, 0u, 0u, 0u}, a = h, b = h;
        if (k < d) {
            const int64_t f = (anti ? row >> 1 : row) * d + k;
            h = *(const u32x4*)(H_in + row * d + k);
            a = *(const u32x4*)(A + f);
            b = *(const u32x4*)(B + f);
        }
        *(u32x4*)(sh[0] + r * pitch + k) = h;
        *(u32x4*)(sh[1] + r * pitch + k) = u32x4{0u, 0u, 0u, 0u};
        *(u32x4*)(sA + r * pitch + k) = a;
        *(u32x4*)(sB + r * pitch + k) = b;
    }
    __syncthreads();
    // first dot products: a wave takes 4 rows, 16 lanes a row
    {
        const int r = wave * 4 + (lane >> 4);
        int acc = 0;
        for (int k = (lane & 15) * 16; k < d; k += 256) {
            const u32x4 h = *(const u32x4*)(sh[0] + r * pitch + k), b = *(const u32x4*)(sB + r * pitch + k);
#pragma unroll
            for (int w = 0; w < 4; ++w) acc = __builtin_amdgcn_sdot4((int)h[w], (int)b[w], acc, false);
        }
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if ((lane & 15) == 0) part[r] = acc;
        for (int i = tid; i < 7 * 32; i += 512) part[32 + i] = 0;
    }
    __syncthreads();
    const bool neg = anti && ((row0 + n) & 1);  // the odd member of a pair uses -B

    // streamed k blocks, PF in flight, the first ones of a step asked for as it begins (under the resident blocks)
    constexpr bool STREAM = RES < 8 * CB;
    u32x4 ws[PF][STREAM ? CB : 1];
    auto stream = [&](u32x4(&w)[STREAM ? CB : 1], int kb) __attribute__((always_inline)) {
        if constexpr (STREAM) {
            const int k = min(kb, nb - 1);
#pragma unroll
            for (int c = 0; c < CB; ++c) w[c] = Wp[((int64_t)min(cb0 + c, nb - 1) * nb + k) * 64 + lane];  // clamped, unconditional
        }
    };
    for (int t = 0; t < steps; ++t) {
        const char* hs = sh[t & 1] + n * pitch + half * 16;
        char* hd = sh[(t + 1) & 1];
        i32x16 acc[CB];
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[c][e] = 0;
        if constexpr (STREAM) {
#pragma unroll
            for (int p = 0; p < PF; ++p) stream(ws[p], RES + p);
        }
        int dot = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) dot += part[(t & 1) * 256 + w * 32 + n];
        if (neg) dot = -dot;
#pragma unroll
        for (int kb = 0; kb < RES; ++kb) {
            if (kb < nb) {
                const u32x4 hf = *(const u32x4*)(hs + kb * 32);
#pragma unroll
                for (int c = 0; c < CB; ++c) MmaI8::mma(wr[c][kb], hf, acc[c]);
            }
        }
        if constexpr (STREAM) {
            for (int kb = RES; kb < nb; kb += PF) {
#pragma unroll
                for (int p = 0; p < PF; ++p) {
                    if (kb + p < nb) {
                        const u32x4 hf = *(const u32x4*)(hs + (kb + p) * 32);
#pragma unroll
                        for (int c = 0; c < CB; ++c) MmaI8::mma(ws[p][c], hf, acc[c]);
                    }
                    stream(ws[p], kb + p + PF);
                }
            }
        }
        int share = 0;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            if (cb0 + c < nb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = (cb0 + c) * 32 + q * 8 + half * 4;
                const uint32_t a4 = *(const uint32_t*)(sA + n * pitch + j), b4 = *(const uint32_t*)(sB + n * pitch + j);
                int y[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int ae = (int)(int8_t)(a4 >> (8 * e));
                    const int prod = DOT24 ? __mul24(dot, ae) : dot * ae;
                    y[e] = min(127, max(-127, (acc[c][4 * q + e] + (prod >> corr_shift)) >> out_shift));
                }
                const uint32_t o = __builtin_amdgcn_perm((uint32_t)y[1], (uint32_t)y[0], 0x0c0c0400u) |
                                   __builtin_amdgcn_perm((uint32_t)y[3], (uint32_t)y[2], 0x04000c0cu);
                if (j < d) {  // d is a multiple of 16: whole groups; columns past it stay zero
                    *(uint32_t*)(hd + n * pitch + j) = o;
                    share = __builtin_amdgcn_sdot4((int)o, (int)b4, share, false);
                }
            }
        }
        share += __shfl_xor(share, 32, 64);
        if (half == 0) part[((t + 1) & 1) * 256 + wave * 32 + n] = share;
        __syncthreads();
    }
    const char* hl = sh[steps & 1];
    for (int i = tid; i < RECUR_ROWS * (d >> 4); i += 512) {
        const int r = i / (d >> 4), k = (i - r * (d >> 4)) * 16;
        if (row0 + r < rows) *(u32x4*)(H_out + (row0 + r) * d + k) = *(const u32x4*)(hl + r * pitch + k);
    }
}

// From four steps on (below, laying theta out costs what the launches do).  Where most of theta has to stream (more than 768 wide)
// a step costs 10 us however few rows there are, so the rows have to fill half of the chip.  Measured (us, one launch per step / this):
// 1024 wide: 8192 members x 64 steps 983 / 732, 4096 x 32 346 / 342, 2500 x 32 312 / 337; 896: 4096 x 32 328 / 304;
// 768: 5000 x 16 173 / 113; 640: 300 x 16 129 / 91; 512: 8192 x 32 243 / 127; 272: 2076 x 36 262 / 98; 256: 100 x 64 367 / 81.
bool recur_i8_applies(int d_out, int d_in, int64_t rows, int steps, int compute_units)
{
    return d_out == d_in && d_in % 16 == 0 && steps >= 4 && (d_in <= 768 || (d_in <= 1024 && rows >= (int64_t)RECUR_ROWS * compute_units / 2));
}

egg_status launch_recur_i8(eggroll_ctx* c, const int8_t* A, const int8_t* B, int anti, int64_t rows, int d, int int_bound, int corr_shift,
                           int out_shift, int steps, const int8_t* W, const int8_t* H_in, int8_t* H_out)
{
    const int nb = (d + 31) / 32;
    egg_status st = reserve(c, c->i8_h, (size_t)nb * nb * 1024);
    if (st != EGG_OK) return st;
    u32x4* Wp = (u32x4*)c->i8_h.p;
    {
        KernelScope ks(c, "pack_theta");
        hipLaunchKernelGGL(pack_theta_kernel, dim3((unsigned)((nb * nb * 64 + 255) / 256)), dim3(256), 0, c->stream, W, d, nb, Wp);
        if ((st = check_hip(c, hipGetLastError(), "pack_theta launch")) != EGG_OK) return st;
    }
    // |u . B_i| <= d * 127 * (largest noise magnitude): below 2^23 the correction product fits the 24-bit multiplier
    const bool dot24 = (int64_t)d * 127 * noise_max(int_bound) < (int64_t(1) << 23);
    const size_t lds = (size_t)4 * RECUR_ROWS * (nb * 32 + 16) + 2 * 8 * 32 * sizeof(int);
    const dim3 g((unsigned)((rows + RECUR_ROWS - 1) / RECUR_ROWS)), b(512);
#define EGG_RECUR(CB, RES, PF, D24)                                                                                                \
    {                                                                                                                              \
        auto kern = recur_i8_kernel<CB, RES, PF, D24>;                                                                             \
        if ((st = ensure_dynamic_lds(c, (const void*)kern, lds, "recurrence smem attr")) != EGG_OK) return st;                     \
        KernelScope ks(c, "forward_recur_i8");                                                                                     \
        hipLaunchKernelGGL(kern, g, b, lds, c->stream, Wp, A, B, anti, rows, d, steps, corr_shift, out_shift, H_in, H_out);        \
        return check_hip(c, hipGetLastError(), "forward_recur_i8 launch");                                                         \
    }
#define EGG_RECUR_D(CB, RES, PF)                \
    {                                           \
        if (dot24) EGG_RECUR(CB, RES, PF, true) \
        EGG_RECUR(CB, RES, PF, false)           \
    }
    // (k blocks kept and in flight, measured at 1024 / 768 wide: kept ones are worth more than depth -- 3 + 4: 870 us for 8192 members
    // x 64 steps, 4 + 3: 798, 5 + 2: 727 to 740, 6 + 1: 732 and the best with few rows; 7 + 2 spills 56 registers: 783)
    static_assert(512 * 127 * 127 < (1 << 23), "up to 512 wide the product always fits");
    if (nb <= 8) EGG_RECUR(1, 8, 1, true)
    if (nb <= 16) EGG_RECUR(2, 16, 1, true)
    if (nb <= 24) EGG_RECUR_D(3, 10, 2)
    EGG_RECUR_D(4, 6, 1)
#undef EGG_RECUR_D
#undef EGG_RECUR
}

}  // namespace egg
