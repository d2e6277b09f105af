// Integer parameter update of the int8 model (App. "Parameter Update" of the integer pretraining
// section), bit-exact:
//   E = (diag(F) A)^T B    int8 x int8 -> int32 over the population, F_i in {-1, 0, 1}
//   theta <- clamp(theta + sign(E) [|E| >= threshold], -127, 127)      one bin per step
// Three kernels, each over several matrices at once (the integer model updates 6 L + 2 of them, most of 256 x 256, and one
// matrix alone leaves the chip idle): the factors are generated straight into K-packed panels (16 consecutive members of one
// column per 16-byte chunk) with F folded into the A panel (a sign flip or a zero: still int8); the int8 MFMA NT core
// contracts the panels over the members; where the tiles of all matrices together do not fill the chip, K is split over
// groups of workgroups, each group stores its int32 partial E, and an elementwise pass adds the partials (integer addition:
// the result does not depend on the order) and applies the threshold.  With one split the epilogue applies it directly.
// (Combining the partial tiles with atomics was measured 20x slower than the contraction itself: 64 scattered 4-byte
// atomics per instruction.)
#include "common.hpp"
#include "gemm_core.hpp"
#include <algorithm>

namespace egg {

// 4 x 4 bytes, rows in x[0..3], transposed in place
__device__ __forceinline__ void transpose4(uint32_t (&x)[4])
{
    const uint32_t a = __builtin_amdgcn_perm(x[1], x[0], 0x05010400u), b = __builtin_amdgcn_perm(x[1], x[0], 0x07030602u);
    const uint32_t c = __builtin_amdgcn_perm(x[3], x[2], 0x05010400u), d = __builtin_amdgcn_perm(x[3], x[2], 0x07030602u);
    x[0] = __builtin_amdgcn_perm(c, a, 0x05040100u);
    x[1] = __builtin_amdgcn_perm(c, a, 0x07060302u);
    x[2] = __builtin_amdgcn_perm(d, b, 0x05040100u);
    x[3] = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

// Panels: a thread owns 8 columns of 16 consecutive members -- one Threefry block per member (two with the table noise) -- and
// writes 8 chunks, 128 contiguous bytes.  Vector-ALU bound: the generator's 61 slots and 56 for the byte -> integer map per
// block.  Members past the end and members of fitness 0 contribute zero bytes to the A panel.
struct I8PackJob {
    StreamKey key;
    FastDiv div;        // work items per K group: d / 8
    uint32_t total;     // work items
    uint32_t first_wg;
    int d;
    const int8_t* F;    // NULL: a B panel
    u32x4* out;
};
constexpr int I8_BATCH = 20;  // matrices per launch
struct I8PackJobs {
    int count;
    I8PackJob job[2 * I8_BATCH];
};

template <bool TABLE>
__global__ __launch_bounds__(256) void gen_pack_i8_kernel(I8PackJobs jobs, uint32_t member_begin, int64_t members, IntMap im,
                                                          const int8_t* __restrict__ table)
{
    int j = 0;
    while (j + 1 < jobs.count && blockIdx.x >= jobs.job[j + 1].first_wg) ++j;
    const I8PackJob& J = jobs.job[j];
    const uint32_t i = (blockIdx.x - J.first_wg) * 256u + threadIdx.x;
    if (i >= J.total) return;
    const uint32_t kg = fast_div(J.div, i), c8 = i - kg * J.div.d;
    const int64_t m0 = (int64_t)kg * 16;
    uint32_t x[2][16];  // [half of the 8 columns][member]
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        uint32_t w0, w1;
        const uint32_t member = member_begin + (uint32_t)(m0 + e);
        if constexpr (TABLE) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                noise_words(J.key, member, 2 * c8 + h, w0, w1);
                x[h][e] = (uint32_t)(uint8_t)table[w0 & 0xFFFFu] | ((uint32_t)(uint8_t)table[w0 >> 16] << 8) |
                          ((uint32_t)(uint8_t)table[w1 & 0xFFFFu] << 16) | ((uint32_t)(uint8_t)table[w1 >> 16] << 24);
            }
        } else {
            noise_words(J.key, member, c8, w0, w1);
            x[0][e] = int4_from_word(im, w0);
            x[1][e] = int4_from_word(im, w1);
        }
    }
    if (J.F) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int fv = (int)J.F[min(m0 + e, members - 1)];
            const int f = m0 + e < members ? fv : 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // bytewise negation without a carry between bytes: -b = (b ^ 0xFF) + 1 (no byte is -128)
                const uint32_t n = x[h][e] ^ 0xFFFFFFFFu;
                const uint32_t neg = ((n & 0x7F7F7F7Fu) + 0x01010101u) ^ (n & 0x80808080u);
                x[h][e] = f > 0 ? x[h][e] : (f < 0 ? neg : 0u);
            }
        }
    }
    u32x4* o = J.out + (int64_t)kg * J.d + c8 * 8;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        u32x4 r[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            uint32_t q[4] = {x[h][4 * w], x[h][4 * w + 1], x[h][4 * w + 2], x[h][4 * w + 3]};
            transpose4(q);
            r[0][w] = q[0]; r[1][w] = q[1]; r[2][w] = q[2]; r[3][w] = q[3];
        }
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) o[h * 4 + cc] = r[cc];
    }
}

// one bin towards sign(e) where |e| reaches the threshold; four entries per word
__device__ __forceinline__ uint32_t move4(uint32_t theta4, const i32x4& e, int threshold)
{
    uint32_t out = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int v = e[b];
        const int mag = v < 0 ? -v : v;  // |E| < 2^31 is guaranteed by the host-side size check
        int t = (int)(int8_t)(theta4 >> (8 * b));
        if (v != 0 && mag >= threshold) t += v > 0 ? 1 : -1;
        t = min(127, max(-127, t));
        out |= ((uint32_t)t & 0xFFu) << (8 * b);
    }
    return out;
}

// elementwise pass after a split-K contraction: adds the partial E of every split, 4 entries per thread (16 made a 256 x 256
// matrix 16 workgroups that walked 128 partials one after the other: 37 us of memory latency)
struct I8ApplyJob {
    const i32x4* parts;
    int nsplit;
    uint32_t first_wg;
    i32x4* E_out;
    uint32_t* theta;
    int64_t n4;
};
struct I8ApplyJobs {
    int count;
    I8ApplyJob job[I8_BATCH];
};
__global__ __launch_bounds__(256) void apply_threshold_kernel(I8ApplyJobs jobs, int threshold)
{
    int j = 0;
    while (j + 1 < jobs.count && blockIdx.x >= jobs.job[j + 1].first_wg) ++j;
    const I8ApplyJob& J = jobs.job[j];
    const int64_t i = (int64_t)(blockIdx.x - J.first_wg) * 256 + threadIdx.x;
    if (i >= J.n4) return;
    i32x4 e = J.parts[i];
    int sp = 1;
    for (; sp + 8 <= J.nsplit; sp += 8) {  // eight partials in flight
        i32x4 p[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) p[k] = J.parts[(sp + k) * J.n4 + i];
#pragma unroll
        for (int k = 0; k < 8; ++k) e += p[k];
    }
    for (; sp < J.nsplit; ++sp) e += J.parts[sp * J.n4 + i];
    if (J.E_out) J.E_out[i] = e;
    J.theta[i] = move4(J.theta[i], e, threshold);
}

// Epilogue of the contraction.  Rows of the product are columns k of theta (P = B panel), its
// columns are rows j of theta (Q = F*A panel): a lane of the MFMA layout owns 4 consecutive k of
// one j.  The int32 accumulators of a 32-row block are parked in the wave's LDS slice and re-read
// row-wise, so that a lane finishes 16 consecutive entries of one theta row with 16-byte accesses.
struct I8UpdEpi {
    typedef int value_t;
    struct Args {
        int32_t* E;      // optional output [d_out][d_in]; split-K: the split's partial E
        int8_t* theta;   // [d_out][d_in]
        int d_out, d_in, threshold;
        int split;       // != 0: only store the partial E
    };
    const Args a;
    char* const stage;
    const int lane;
    int row_pitch;

    static constexpr __host__ __device__ int pitch(int wtm) { return wtm * 4 + 16; }
    static constexpr __host__ __device__ int lds_per_wave(int wtm) { return 32 * pitch(wtm); }
    __device__ __forceinline__ I8UpdEpi(const Args& a_, char* slice, int lane_) : a(a_), stage(slice), lane(lane_), row_pitch(0) {}
    template <class MT, int MB, int NB>
    __device__ __forceinline__ void extra_mma(typename MT::acc_t (&)[MB][NB], int, int, int, int) {}
    template <int MB, int NB>
    __device__ __forceinline__ void prefetch(int, int, int, int) { row_pitch = pitch(MB * 32); }
    __device__ __forceinline__ void column(int, bool) {}
    __device__ __forceinline__ void store4(int, int, const int (&v)[4], bool, int ml)
    {
        *(i32x4*)(stage + (lane & 31) * row_pitch + ml * 4) = i32x4{v[0], v[1], v[2], v[3]};
    }
    template <int WTM>
    __device__ __forceinline__ void flush(int mw0, int nb0, int n_rows)
    {
        constexpr int P = pitch(WTM), CPR = WTM / 16, PASSES = WTM / 32;
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the wave's own LDS writes have landed
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < PASSES; ++it) {
            const int c = it * 64 + lane;
            const int row = c / CPR, mc = (c % CPR) * 16;
            const int j = nb0 + row, k = mw0 + mc;
            if (j < n_rows && k < a.d_in) {  // d_in is a multiple of 16
                const char* src = stage + row * P + mc * 4;
                const int64_t idx = (int64_t)j * a.d_in + k;
                i32x4 e[4];
#pragma unroll
                for (int w = 0; w < 4; ++w) e[w] = *(const i32x4*)(src + w * 16);
                if (a.split) {
#pragma unroll
                    for (int w = 0; w < 4; ++w) *(i32x4*)(a.E + idx + 4 * w) = e[w];
                } else {
                    if (a.E) {
#pragma unroll
                        for (int w = 0; w < 4; ++w) *(i32x4*)(a.E + idx + 4 * w) = e[w];
                    }
                    u32x4 t = *(const u32x4*)(a.theta + idx);
#pragma unroll
                    for (int w = 0; w < 4; ++w) t[w] = move4(t[w], e[w], a.threshold);
                    *(u32x4*)(a.theta + idx) = t;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();  // the slice is reused by the next row block
    }
};

// contractions of several matrices in one launch: 128 x 128 tiles, two workgroups per CU
struct I8ContractJob {
    Operand P, Q;
    I8UpdEpi::Args ea;
    int tiles_m, tiles_n, per_split;  // K-chunks per split (whole stages)
    uint32_t first_wg;
};
struct I8ContractJobs {
    int count;
    I8ContractJob job[I8_BATCH];
};
static_assert(sizeof(I8ContractJobs) <= 3584 && sizeof(I8PackJobs) <= 3584, "kernel arguments");

__global__ __launch_bounds__(256, 2) void contract_i8_kernel(I8ContractJobs jobs, int kchunks, const char* zero_page)
{
    int j = 0;
    while (j + 1 < jobs.count && blockIdx.x >= jobs.job[j + 1].first_wg) ++j;
    const I8ContractJob& J = jobs.job[j];
    const int id = (int)(blockIdx.x - J.first_wg), tiles = J.tiles_m * J.tiles_n;
    const int split = id / tiles, kbeg = split * J.per_split;
    I8UpdEpi::Args ea = J.ea;
    if (ea.split) ea.E += (int64_t)split * ea.d_out * ea.d_in;
    gemm_nt_tile<MmaI8, 128, 128, 2, 2, true, I8UpdEpi>(J.P, J.Q, id - split * tiles, kbeg, min(kchunks - kbeg, J.per_split), J.tiles_m,
                                                        J.tiles_n, zero_page, ea);
}

static egg_status launch_i8_upd_gemm_big(eggroll_ctx* c, const Operand& P, const Operand& Q, int kchunks, const I8UpdEpi::Args& ea)
{
    constexpr int BM = 256, BN = 256, WM = 2, WN = 4;
    const int tiles_m = (P.rows + BM - 1) / BM, tiles_n = (Q.rows + BN - 1) / BN;
    const size_t lds = std::max(gemm_lds_bytes<BM, BN>(), (size_t)WM * WN * I8UpdEpi::lds_per_wave(BM / WM));
    auto kern = gemm_nt_kernel<MmaI8, BM, BN, WM, WN, true, I8UpdEpi, 1>;
    egg_status st = ensure_dynamic_lds(c, (const void*)kern, lds, "gemm smem attr");
    if (st != EGG_OK) return st;
    KernelScope ks(c, "update_gemm_i8");
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(WM * WN * 64), lds, c->stream, P, Q, kchunks, tiles_m, tiles_n,
                       (const char*)c->zero_page.p, ea);
    return check_hip(c, hipGetLastError(), "update_gemm_i8");
}

// one group of matrices: panels, contraction, threshold
static egg_status update_i8_group(eggroll_ctx* c, const I8UpdateJob* jobs, int count, uint32_t member_begin, int64_t N, int int_bound,
                                  const int8_t* F, int32_t threshold)
{
    const int64_t kgroups = (N + 15) / 16;
    egg_status st;
    auto pad = [](size_t b) { return (b + 255) & ~size_t(255); };
    size_t panels = 0;
    int64_t tiles = 0, entries = 0;
    for (int q = 0; q < count; ++q) {
        panels += pad((size_t)kgroups * jobs[q].d_out * 16) + pad((size_t)kgroups * jobs[q].d_in * 16);
        tiles += ((jobs[q].d_out + 127) / 128) * (int64_t)((jobs[q].d_in + 127) / 128);
        entries += (int64_t)jobs[q].d_out * jobs[q].d_in;
    }
    // K is split so that the group's tiles are at most two workgroups per CU -- one wave of them -- in whole 8-chunk stages
    // (128 members), at least four of them: shorter runs cost more in partial sums than they gain
    const bool big = count == 1 && ((jobs[0].d_out + 255) / 256) * (int64_t)((jobs[0].d_in + 255) / 256) >= 192;
    int64_t per_split = kgroups;
    int nsplit = 1;
    if (!big) {
        const int64_t stages = (kgroups + 7) / 8;
        const int64_t want = std::min<int64_t>(2 * (int64_t)c->compute_units / std::max<int64_t>(tiles, 1), stages / 4);
        if (want > 1) {
            per_split = (stages + want - 1) / want * 8;
            nsplit = (int)((kgroups + per_split - 1) / per_split);
        }
    }
    // (the partial sums first: they are of much the same size for a smaller group, which is tried where the panels do not fit)
    if (nsplit > 1 && (st = reserve(c, c->t_buf, (size_t)nsplit * entries * sizeof(int32_t))) != EGG_OK) return st;
    if ((st = reserve(c, c->pack_a, panels)) != EGG_OK) return st;

    const bool table = int_bound == EGG_INT_NOISE_NORMAL16;
    if (table && (st = ensure_normal_table(c)) != EGG_OK) return st;
    I8PackJobs pj{};
    I8ContractJobs cj{};
    I8ApplyJobs aj{};
    uint64_t pack_wgs = 0, apply_wgs = 0, gemm_wgs = 0;
    char* p = (char*)c->pack_a.p;
    int32_t* part = (int32_t*)c->t_buf.p;
    auto panel = [&](const StreamKey& key, int d, const int8_t* fit) {
        const uint64_t total = (uint64_t)kgroups * (uint64_t)(d / 8);
        pj.job[pj.count++] = I8PackJob{key, make_fast_div((uint32_t)(d / 8)), (uint32_t)total, (uint32_t)pack_wgs, d, fit, (u32x4*)p};
        pack_wgs += (total + 255) / 256;
        const Operand o{p, 16, (int64_t)d * 16, d};
        p += pad((size_t)kgroups * d * 16);
        return std::make_pair(o, total);
    };
    for (int q = 0; q < count; ++q) {
        const I8UpdateJob& J = jobs[q];
        // rows of the product = columns k of theta (B panel), columns = rows j of theta (F*A panel)
        const auto Q = panel(J.ka, J.d_out, F), P = panel(J.kb, J.d_in, nullptr);
        if (P.second >= (uint64_t(1) << 31) || Q.second >= (uint64_t(1) << 31)) return fail(c, EGG_EUNSUPPORTED, "pack grid too large");
        if (!operand_offsets_fit(P.first, 256) || !operand_offsets_fit(Q.first, 256)) return fail(c, EGG_EUNSUPPORTED, "operand strides too large for 32-bit tile offsets");
        const int tm = (J.d_in + 127) / 128, tn = (J.d_out + 127) / 128;
        I8UpdEpi::Args ea{J.E_out, J.theta, J.d_out, J.d_in, threshold, 0};
        if (nsplit > 1) {
            const int64_t n4 = (int64_t)J.d_out * J.d_in / 4;
            ea.E = part;
            ea.split = 1;
            aj.job[aj.count++] = I8ApplyJob{(const i32x4*)part, nsplit, (uint32_t)apply_wgs, (i32x4*)J.E_out, (uint32_t*)J.theta, n4};
            apply_wgs += (n4 + 255) / 256;
            part += (int64_t)nsplit * n4 * 4;
        }
        cj.job[cj.count++] = I8ContractJob{P.first, Q.first, ea, tm, tn, (int)per_split, (uint32_t)gemm_wgs};
        gemm_wgs += (uint64_t)tm * tn * nsplit;
    }
    if (pack_wgs > 0x7FFFFFFF || gemm_wgs > 0x7FFFFFFF || apply_wgs > 0x7FFFFFFF) return fail(c, EGG_EUNSUPPORTED, "update grid too large");
    {
        KernelScope ks(c, "update_pack_i8");
        const IntMap im = make_int_map(table ? 0 : int_bound);
        if (table) hipLaunchKernelGGL(gen_pack_i8_kernel<true>, dim3((unsigned)pack_wgs), dim3(256), 0, c->stream, pj, member_begin, N, im, (const int8_t*)c->norm_tab.p);
        else hipLaunchKernelGGL(gen_pack_i8_kernel<false>, dim3((unsigned)pack_wgs), dim3(256), 0, c->stream, pj, member_begin, N, im, (const int8_t*)nullptr);
        if ((st = check_hip(c, hipGetLastError(), "pack_i8 launch")) != EGG_OK) return st;
    }
    if (big) return launch_i8_upd_gemm_big(c, cj.job[0].P, cj.job[0].Q, (int)kgroups, cj.job[0].ea);
    {
        const size_t lds = std::max(gemm_lds_bytes<128, 128>(), (size_t)4 * I8UpdEpi::lds_per_wave(64));
        if ((st = ensure_dynamic_lds(c, (const void*)contract_i8_kernel, lds, "gemm smem attr")) != EGG_OK) return st;
        KernelScope ks(c, "update_gemm_i8");
        hipLaunchKernelGGL(contract_i8_kernel, dim3((unsigned)gemm_wgs), dim3(256), lds, c->stream, cj, (int)kgroups, (const char*)c->zero_page.p);
        if ((st = check_hip(c, hipGetLastError(), "update_gemm_i8")) != EGG_OK) return st;
    }
    if (nsplit > 1) {
        KernelScope ks(c, "apply_threshold");
        hipLaunchKernelGGL(apply_threshold_kernel, dim3((unsigned)apply_wgs), dim3(256), 0, c->stream, aj, threshold);
        if ((st = check_hip(c, hipGetLastError(), "apply_threshold launch")) != EGG_OK) return st;
    }
    return EGG_OK;
}

egg_status launch_update_i8_jobs(eggroll_ctx* c, const I8UpdateJob* jobs, int count, uint32_t member_begin, int64_t N, int int_bound,
                                 const int8_t* F, int32_t threshold)
{
    const int64_t kgroups = (N + 15) / 16;
    if (kgroups > 0x7FFFFFFF) return fail(c, EGG_EUNSUPPORTED, "population too large");
    // Matrices share a group while their panels stay within GROUP_BYTES of scratch: beyond that a single one has work enough for the
    // chip.  One that fills the chip with 256 x 256 tiles goes alone.  Where that much scratch is not to be had, smaller groups
    // do, down to the panels of one matrix.
    // (256 x 256 and 256 x 1024 matrices, 131072 ids, whole steps of the integer model: 1 GB 8145 us, 256 MB 8520, 64 MB 9545)
    constexpr size_t GROUP_BYTES = size_t(1) << 30;
    auto fills_chip = [](const I8UpdateJob& j) { return ((j.d_out + 255) / 256) * (int64_t)((j.d_in + 255) / 256) >= 192; };
    int most = I8_BATCH;
    for (int q = 0; q < count;) {
        int n = 0;
        size_t bytes = 0;
        while (q + n < count && n < most) {
            const size_t more = (size_t)kgroups * 16 * ((size_t)jobs[q + n].d_out + jobs[q + n].d_in);
            if (n > 0 && (bytes + more > GROUP_BYTES || fills_chip(jobs[q + n]) || fills_chip(jobs[q]))) break;
            bytes += more;
            ++n;
        }
        const egg_status st = update_i8_group(c, jobs + q, n, member_begin, N, int_bound, F, threshold);
        if (st == EGG_ENOMEM && n > 1) {  // (scratch is reserved before anything is enqueued)
            most = n / 2;
            continue;
        }
        if (st != EGG_OK) return st;
        q += n;
    }
    return EGG_OK;
}

}  // namespace egg
