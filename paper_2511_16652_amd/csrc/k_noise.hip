// eggroll_noise_gen: materialise factor entries [member][n] from the counter-based stream
// (Sec. 1: the factors are reconstructed on demand rather than kept; Alg. 1 sampling lines).
// Vectors made of whole 16-byte pieces (every multiple of 16 bytes: what the models use) go through noise_pieces_kernel;
// noise_gen_kernel takes any length, one Threefry block a thread: two normals, two raw words, or eight bounded integers.
#include "common.hpp"

namespace egg {

enum NoiseMode { NM_F32 = 0, NM_BF16 = 1, NM_I8 = 2, NM_RAW = 3, NM_I8_TABLE = 4 };

template <int MODE>
__global__ __launch_bounds__(256) void noise_gen_kernel(StreamKey key, uint32_t member_begin, int64_t members,
                                                        int64_t n, int64_t blocks_per_member, IntMap im,
                                                        const int8_t* __restrict__ table, void* __restrict__ out)
{
    constexpr int VPB = (MODE == NM_I8) ? 8 : (MODE == NM_I8_TABLE ? 4 : 2);  // values per Threefry block
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gid >= members * blocks_per_member) return;
    const int64_t m = gid / blocks_per_member;
    const uint32_t blk = (uint32_t)(gid - m * blocks_per_member);
    uint32_t w0, w1;
    noise_words(key, member_begin + (uint32_t)m, blk, w0, w1);
    const int64_t first = (int64_t)blk * VPB;  // index of this block's first value inside the member's vector
    const int64_t base = m * n + first;
    const bool full = first + VPB <= n;

    if constexpr (MODE == NM_F32 || MODE == NM_BF16) {
        float z0, z1;
        normal_pair<MODE == NM_F32>(w0, w1, z0, z1);
        if constexpr (MODE == NM_F32) {
            float* o = (float*)out + base;
            if (full && ((base & 1) == 0)) {
                *(float2*)o = make_float2(z0, z1);
            } else {
                o[0] = z0;
                if (full) o[1] = z1;
            }
        } else {
            uint16_t* o = (uint16_t*)out + base;
            const uint32_t pk = pack_bf16x2(z0, z1);
            if (full && ((base & 1) == 0)) {
                *(uint32_t*)o = pk;
            } else {
                o[0] = (uint16_t)(pk & 0xFFFFu);
                if (full) o[1] = (uint16_t)(pk >> 16);
            }
        }
    } else if constexpr (MODE == NM_RAW) {
        uint32_t* o = (uint32_t*)out + base;
        if (full && ((base & 1) == 0)) {
            *(uint2*)o = make_uint2(w0, w1);
        } else {
            o[0] = w0;
            if (full) o[1] = w1;
        }
    } else if constexpr (MODE == NM_I8_TABLE) {
        // value v of the block: 16-bit half v & 1 (low half first) of word v >> 1 indexes the table
        const uint32_t pk = (uint32_t)(uint8_t)table[w0 & 0xFFFFu] | ((uint32_t)(uint8_t)table[w0 >> 16] << 8) |
                            ((uint32_t)(uint8_t)table[w1 & 0xFFFFu] << 16) | ((uint32_t)(uint8_t)table[w1 >> 16] << 24);
        int8_t* o = (int8_t*)out + base;
        if (full && ((base & 3) == 0)) {
            *(uint32_t*)o = pk;
        } else {
            for (int b = 0; b < 4 && first + b < n; ++b) o[b] = (int8_t)((pk >> (8 * b)) & 0xFFu);
        }
    } else {
        const uint32_t p0 = int4_from_word(im, w0), p1 = int4_from_word(im, w1);
        int8_t* o = (int8_t*)out + base;
        if (full && ((base & 7) == 0)) {
            *(uint2*)o = make_uint2(p0, p1);
        } else {
            for (int b = 0; b < 8 && first + b < n; ++b) o[b] = (int8_t)(((b < 4 ? p0 : p1) >> (8 * (b & 3))) & 0xFFu);
        }
    }
}

// The same values by whole 16-byte pieces of the output, for vectors that are made of them (n * element size a multiple of
// 16; the output is then one run of pieces).  A thread expands the 2 or 4 Threefry blocks of one piece -- independent
// chains that fill each other's latency -- and stores it once; the member of a piece comes from a multiply instead of the
// 64-bit division that the general kernel spends on every block, which was as long as the generator itself.
// Several vectors of the same members (the factors of a layer's matrices) go out in one launch: a workgroup looks up its
// vector by its number.  Vector-ALU bound.
// Room for 20 vectors, or for 2: the host copies a launch's arguments, and a kilobyte of them is felt in a small call (attention of 16
// members x 16 heads x 64 x 32 with the one vector of factors it needs, three launches: 13.1 us a call with room for 20, 12.4 for 2).
constexpr int NOISE_JOBS = 20, NOISE_JOBS_FEW = 2;
template <int JOBS>
struct NoisePieces {
    int count;
    NoisePiece job[JOBS];
};

template <int MODE, int JOBS>
__global__ __launch_bounds__(256) void noise_pieces_kernel(uint32_t member_begin, IntMap im, const int8_t* __restrict__ table,
                                                           NoisePieces<JOBS> jobs)
{
    constexpr int BPP = (MODE == NM_BF16 || MODE == NM_I8_TABLE) ? 4 : 2;  // Threefry blocks per piece
    int j = 0;
    while (j + 1 < jobs.count && blockIdx.x >= jobs.job[j + 1].first_wg) ++j;
    const NoisePiece& J = jobs.job[j];
    const uint32_t i = (blockIdx.x - J.first_wg) * 256u + threadIdx.x;
    if (i >= J.total) return;
    const uint32_t m = fast_div(J.per_member, i);
    const uint32_t blk = (i - m * J.per_member.d) * BPP;
    if constexpr (MODE == NM_BF16 || MODE == NM_F32) {
        J.out[i] = normal_piece<MODE == NM_BF16>(J.key, member_begin + m, blk);
        return;
    }
    uint32_t w[2 * BPP];
#pragma unroll
    for (int b = 0; b < BPP; ++b) noise_words(J.key, member_begin + m, blk + b, w[2 * b], w[2 * b + 1]);
    uint32_t o[4];
    if constexpr (MODE == NM_RAW) {
#pragma unroll
        for (int b = 0; b < 4; ++b) o[b] = w[b];
    } else if constexpr (MODE == NM_I8_TABLE) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
            o[b] = (uint32_t)(uint8_t)table[w[2 * b] & 0xFFFFu] | ((uint32_t)(uint8_t)table[w[2 * b] >> 16] << 8) |
                   ((uint32_t)(uint8_t)table[w[2 * b + 1] & 0xFFFFu] << 16) | ((uint32_t)(uint8_t)table[w[2 * b + 1] >> 16] << 24);
    } else {
#pragma unroll
        for (int b = 0; b < 4; ++b) o[b] = int4_from_word(im, w[b]);
    }
    J.out[i] = noise_x4{o[0], o[1], o[2], o[3]};
}

static egg_status launch_noise_general(eggroll_ctx* c, const StreamKey& k, uint32_t member_begin, int64_t members, int64_t n,
                        egg_dtype dtype, egg_dist dist, int int_bound, void* out)
{
    const bool table = dist == EGG_NORMAL_INT16 || (dist == EGG_UNIFORM_INT && int_bound == EGG_INT_NOISE_NORMAL16);
    const int vpb = table ? 4 : (dist == EGG_UNIFORM_INT ? 8 : 2);
    const int64_t bpm = (n + vpb - 1) / vpb;
    if (bpm > (int64_t(1) << 32)) return fail(c, EGG_EUNSUPPORTED, "factor vector too long");
    const int64_t total = members * bpm;
    const int64_t grid = (total + 255) / 256;
    if (grid > 0x7FFFFFFF) return fail(c, EGG_EUNSUPPORTED, "noise_gen: too many elements for one call");
    IntMap im = make_int_map(dist == EGG_UNIFORM_INT && !table ? int_bound : 0);
    const int8_t* tab = (const int8_t*)c->norm_tab.p;
    KernelScope ks(c, "noise_gen");
    const dim3 g((unsigned)grid), b(256);
    if (dist == EGG_RAW)
        hipLaunchKernelGGL(noise_gen_kernel<NM_RAW>, g, b, 0, c->stream, k, member_begin, members, n, bpm, im, tab, out);
    else if (table)
        hipLaunchKernelGGL(noise_gen_kernel<NM_I8_TABLE>, g, b, 0, c->stream, k, member_begin, members, n, bpm, im, tab, out);
    else if (dist == EGG_UNIFORM_INT)
        hipLaunchKernelGGL(noise_gen_kernel<NM_I8>, g, b, 0, c->stream, k, member_begin, members, n, bpm, im, tab, out);
    else if (dtype == EGG_F32)
        hipLaunchKernelGGL(noise_gen_kernel<NM_F32>, g, b, 0, c->stream, k, member_begin, members, n, bpm, im, tab, out);
    else
        hipLaunchKernelGGL(noise_gen_kernel<NM_BF16>, g, b, 0, c->stream, k, member_begin, members, n, bpm, im, tab, out);
    return check_hip(c, hipGetLastError(), "noise_gen launch");
}

// first use on this context: build the table on the host and upload it (a blocking copy)
egg_status ensure_normal_table(eggroll_ctx* c)
{
    if (c->norm_tab.p) return EGG_OK;
    std::vector<int8_t> h(65536);
    normal_int_table(h.data());
    const egg_status st = reserve(c, c->norm_tab, 65536);
    if (st != EGG_OK) return st;
    return check_hip(c, hipMemcpy(c->norm_tab.p, h.data(), 65536, hipMemcpyHostToDevice), "upload of the integer normal table");
}

// whole pieces, 32-bit piece numbers (the exact division needs them below 2^31): everything else goes value by value
static bool whole_pieces(const NoiseJob& J, int per_piece, int64_t members)
{
    const int64_t ppm = J.n / per_piece;
    return J.n % per_piece == 0 && aligned16(J.out) && ppm < (int64_t(1) << 31) && members <= ((int64_t(1) << 31) - 256) / std::max<int64_t>(ppm, 1);
}

bool normal_pieces(const NoiseJob& J, int64_t members, egg_dtype dtype, NoisePiece& out)
{
    const int per_piece = dtype == EGG_F32 ? 4 : 8;
    if (J.n <= 0 || members <= 0 || !whole_pieces(J, per_piece, members)) return false;
    const uint32_t ppm = (uint32_t)(J.n / per_piece);
    out = NoisePiece{J.key, make_fast_div(ppm), (uint32_t)(members * ppm), 0, (noise_x4*)J.out};
    return true;
}

egg_status launch_noise_jobs(eggroll_ctx* c, const NoiseJob* jobs, int count, uint32_t member_begin, int64_t members, egg_dtype dtype,
                             egg_dist dist, int int_bound)
{
    const bool table = dist == EGG_NORMAL_INT16 || (dist == EGG_UNIFORM_INT && int_bound == EGG_INT_NOISE_NORMAL16);
    if (table) {
        const egg_status st = ensure_normal_table(c);
        if (st != EGG_OK) return st;
    }
    const int per_piece = dist == EGG_RAW ? 4 : (table || dist == EGG_UNIFORM_INT ? 16 : (dtype == EGG_F32 ? 4 : 8));  // values
    const IntMap im = make_int_map(dist == EGG_UNIFORM_INT && !table ? int_bound : 0);
    const int8_t* tab = (const int8_t*)c->norm_tab.p;
    NoisePieces<NOISE_JOBS> np{};
    uint32_t wgs = 0;
    auto flush = [&]() -> egg_status {
        if (np.count == 0) return EGG_OK;
        KernelScope ks(c, "noise_gen");
        const dim3 g(wgs), b(256);
        auto launch = [&](auto jobs_c, const auto& args) {
            constexpr int JOBS = decltype(jobs_c)::value;
            if (dist == EGG_RAW) hipLaunchKernelGGL((noise_pieces_kernel<NM_RAW, JOBS>), g, b, 0, c->stream, member_begin, im, tab, args);
            else if (table) hipLaunchKernelGGL((noise_pieces_kernel<NM_I8_TABLE, JOBS>), g, b, 0, c->stream, member_begin, im, tab, args);
            else if (dist == EGG_UNIFORM_INT) hipLaunchKernelGGL((noise_pieces_kernel<NM_I8, JOBS>), g, b, 0, c->stream, member_begin, im, tab, args);
            else if (dtype == EGG_F32) hipLaunchKernelGGL((noise_pieces_kernel<NM_F32, JOBS>), g, b, 0, c->stream, member_begin, im, tab, args);
            else hipLaunchKernelGGL((noise_pieces_kernel<NM_BF16, JOBS>), g, b, 0, c->stream, member_begin, im, tab, args);
        };
        if (np.count <= NOISE_JOBS_FEW) {
            NoisePieces<NOISE_JOBS_FEW> few{np.count, {}};
            for (int q = 0; q < np.count; ++q) few.job[q] = np.job[q];
            launch(std::integral_constant<int, NOISE_JOBS_FEW>{}, few);
        } else {
            launch(std::integral_constant<int, NOISE_JOBS>{}, np);
        }
        np.count = 0;
        wgs = 0;
        return check_hip(c, hipGetLastError(), "noise_gen launch");
    };
    egg_status st;
    for (int q = 0; q < count; ++q) {
        const NoiseJob& J = jobs[q];
        const int64_t ppm = J.n / per_piece;
        if (!whole_pieces(J, per_piece, members)) {
            if ((st = launch_noise_general(c, J.key, member_begin, members, J.n, dtype, dist, int_bound, J.out)) != EGG_OK) return st;
            continue;
        }
        if (ppm == 0 || members <= 0) continue;
        const uint32_t total = (uint32_t)(members * ppm), n_wg = (total + 255u) / 256u;
        if (np.count == NOISE_JOBS || wgs > 0x7FFFFFFFu - n_wg)
            if ((st = flush()) != EGG_OK) return st;
        np.job[np.count++] = NoisePiece{J.key, make_fast_div((uint32_t)ppm), total, wgs, (noise_x4*)J.out};
        wgs += n_wg;
    }
    return flush();
}

egg_status launch_noise(eggroll_ctx* c, const StreamKey& k, uint32_t member_begin, int64_t members, int64_t n,
                        egg_dtype dtype, egg_dist dist, int int_bound, void* out)
{
    const NoiseJob job{k, n, out};
    return launch_noise_jobs(c, &job, 1, member_begin, members, dtype, dist, int_bound);
}

}  // namespace egg
