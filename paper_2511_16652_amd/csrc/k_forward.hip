// Population forward of one linear layer (Sec. 4.2):
//   Y = X W^T   (shared MFMA GEMM over all N*S rows)   +   (sigma/sqrt r) t A_i^T   (epilogue)
// The epilogue regenerates exactly the factor entries A_i[j..j+3][:] that the lane's four outputs
// need -- for one row per member every entry of A is produced exactly once over the grid -- applies
// the correction in fp32, optionally keeps A_i for the update, applies the activation and stores.
#include "common.hpp"
#include "gemm_core.hpp"
#include "forward_fold.hpp"
#include "gemm_small.hpp"

namespace egg {

// Arguments of the forward epilogues
struct FwdArgs {
    StreamKey ka;
    uint32_t member_begin;
    int S, d_out;
    FastDiv by_s;  // n / S
    float c;       // sigma / sqrt(r); 0 switches the correction off
    int act, y_bf16;
    void* Y;
    const float* t;
    void* A_buf;         // REGEN: optional cache to fill; otherwise the materialised factors to read
    int pair_share;      // REGEN with antithetic pairs: distance of the lanes that hold the two rows of a pair (0: no sharing)
    const void* resid;   // optional [R][d_out] of the output dtype, added after the activation (residual stream)
    const void* next_B;  // LEAN_PROJ: the next layer's factors B[member][d_out][rank] (bf16; its rank is this layer's)
    float* next_part;    // LEAN_PROJ: partial projections [d_out / 128 slabs][R][rank]
};

// The store-only epilogue of the persistent kernel (LeanEpi): bf16 outputs whose correction is either off (c == 0) or already
// folded into the accumulators by extra_mma (S a multiple of 64: a wave tile's 64 columns belong to one member); the activation
// and the residual are fixed at compile time (bit 1: GELU, bit 2: residual).
// bit 3 (LEAN_PROJ): the rows this layer stores are the input of the next perturbed layer, whose rank-1 projection
// t'[n] = sum_m Y[n][m] B'[m] is formed here from the very bf16 values that are stored, so that Y is not read again
// by a projection pass: a lane adds its 4 x 8 products per column, the four lane groups of a column are summed by two
// shuffles, and the sum over the wave tile's 128 rows goes to a slab-partial that a small pass adds up in fixed order.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

template <int RANK, int LEAN>
struct LeanEpi {
    typedef float value_t;
    typedef FwdArgs Args;
    static constexpr int BLK = 16, WTM = 128, NBLK = 4;  // 16x16 blocks, wave tiles of 128 rows x 64 columns
    const Args a;
    RowStagerSwz sty;

    // The rank-r correction of a block is itself a small GEMM, Y[m][n] += sum_l A_i[m][l] * (c t[n][l]), and one more
    // MFMA per block adds it to the accumulators: 16 of its K-slots hold A_i[m][0..r) twice and
    // the fp32 value c*t split into two bf16 halves (hi, then lo = the rounding remainder), so the
    // products stay accurate to about 2^-16.  The epilogue that follows is then the plain store.
    static_assert(RANK <= 8, "16 K-slots hold r factor entries beside the hi and lo halves of c t");
    static constexpr int AW = RANK >= 2 ? RANK / 2 : 1;  // 32-bit words of one A_i[m][0..RANK) row in bf16
    // its operands are parked in the wave's staging slice (see prefetch)
    static constexpr int LDS_T = 0, LDS_A = 2048;  // byte offsets of t[64][RANK] fp32 and A_i[128][RANK] bf16 in the slice
    static constexpr int LDS_NB = 3072;            // LEAN_PROJ: the next layer's B'[128][RANK] bf16
    static constexpr bool PROJ = (LEAN & LEAN_PROJ) != 0;
    static_assert(!PROJ || RANK == 1 || RANK == 2 || RANK == 4, "the three runs of 256 RANK bytes fill the wave's 4 KB slice at rank 4");
    // Rank 1: B' of the lane's 4 rows of a row block as two bf16 pairs along the rows -- (r0, r1) and (r2, r3), the packing
    // of the values on their way to the store -- so that a column's share is two packed dot products per row block.
    // Rank 2 and 4 would need 16 RANK registers that way; there the products are formed when the staged rows are read back
    // for the store (flush): a lane then holds 8 consecutive outputs of one row, always the same 8 of the wave tile's 128,
    // and needs B' of those 8 only: bp[l][q] = (B'[8 cc + 2q][l], B'[8 cc + 2q + 1][l]), cc = lane % 16.
    static constexpr bool PROJ_ROWS = PROJ && RANK == 1, PROJ_FLUSH = PROJ && RANK > 1;
    uint32_t nb[PROJ_ROWS ? 8 : 1][2];
    uint32_t bp[PROJ_FLUSH ? RANK : 1][4];
    float tn = 0.f;  // rank 1: the lane's part of t'[n] for the current column
    // Store-only epilogue with residual: the lane's 8 residual pieces (4 bf16 each, one per row block) of the current
    // column block, and those of the next one, on their way while the current block is converted and staged.  Loaded
    // unconditionally from clamped addresses: a predicated load is a branch, and the counted waits behind a branch
    // degrade to "everything outstanding" -- the first version waited out one memory round trip per piece.
    static constexpr bool RESID = (LEAN & LEAN_RESID) != 0;
    // Two sets, used alternately by the column blocks (named at compile time: no copies between them, which the scheduler
    // would be free to hoist, with their wait, to right behind the loads).
    uint2 rres[RESID ? 2 : 1][RESID ? 8 : 1];
    int res_m0 = 0, res_rows = 0;  // first row of the lane's pieces in the wave tile; rows of the output (for the clamp)
    template <int SET>
    __device__ __forceinline__ void load_residual(int n)
    {
        if constexpr (RESID) {
            const uint16_t* rrow = (const uint16_t*)a.resid + (int64_t)min(n, res_rows - 1) * a.d_out;
#pragma unroll
            for (int i = 0; i < 8; ++i) rres[SET][i] = *(const uint2*)(rrow + min(res_m0 + i * BLK, a.d_out - 4));
        }
    }
    float pf_t[NBLK][RANK];

    // late in the main loop: the operands of extra_mma
    template <int MB, int NB>
    __device__ __forceinline__ void prefetch(int mw0, int nw0, int lane, int n_rows)
    {
        // The wave tile (128 rows x 64 columns, one member) needs t[nw0..+64)[0..r) and
        // A_i[mw0..+128)[0..r): two contiguous runs of 256 r bytes, brought into the wave's staging slice by 2 r
        // direct-to-LDS loads of one dword per lane.  No register holds them through the last stage; extra_mma
        // reads its fragments from the slice.  (The slice is idle here: the previous tile's flush is behind us.)
        static_assert(MB * BLK == WTM && NB == NBLK, "slice layout is that of a 128 x 64 wave tile");
        if (a.c == 0.f || nw0 >= n_rows || mw0 >= a.d_out) return;
        const int64_t member_l = (int64_t)fast_div(a.by_s, (uint32_t)nw0);
        const uint32_t* tsrc = (const uint32_t*)(a.t + (int64_t)nw0 * RANK);
        const uint32_t* asrc = (const uint32_t*)((const uint16_t*)a.A_buf + (member_l * a.d_out + mw0) * RANK);
        const int t_last = min(n_rows - nw0, 64) * RANK - 1;           // last valid dword of the t run
        const int a_last = min(a.d_out - mw0, 128) * RANK / 2 - 1;     // of the A run (d_out is a multiple of 4)
#pragma unroll
        for (int k = 0; k < RANK; ++k) {
            __builtin_amdgcn_global_load_lds((egg_glb_void*)(tsrc + min(k * 64 + lane, t_last)),
                                             (egg_lds_void*)(sty.base + LDS_T + k * 256), 4, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < RANK; ++k) {
            __builtin_amdgcn_global_load_lds((egg_glb_void*)(asrc + min(k * 64 + lane, a_last)),
                                             (egg_lds_void*)(sty.base + LDS_A + k * 256), 4, 0, 0);
        }
        if constexpr (PROJ) {
            const uint32_t* bsrc = (const uint32_t*)((const uint16_t*)a.next_B + (member_l * a.d_out + mw0) * RANK);
#pragma unroll
            for (int k = 0; k < RANK; ++k) {
                __builtin_amdgcn_global_load_lds((egg_glb_void*)(bsrc + min(k * 64 + lane, a_last)),
                                                 (egg_lds_void*)(sty.base + LDS_NB + k * 256), 4, 0, 0);
            }
        }
    }

    template <class MT, int MB, int NB>
    __device__ __forceinline__ void extra_mma(typename MT::acc_t (&acc)[MB][NB], int mw0, int nw0, int lane, int n_rows)
    {
        if constexpr (RESID) {
            static_assert(MB == 8 && BLK == 16, "eight row blocks of 16 per wave tile");
            res_m0 = mw0 + (lane / BLK) * 4;
            res_rows = n_rows;
            load_residual<0>(nw0 + (lane & (BLK - 1)));  // column block 0; older than the next tile's loads, so a wait for it waits for nothing else
        }
        if (a.c == 0.f || nw0 >= n_rows || mw0 >= a.d_out) return;  // unperturbed, or nothing of this wave tile is stored
        if constexpr (PROJ) {
            // into registers now: the slice becomes the staging area of the stores
            if constexpr (PROJ_ROWS) {
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    const uint2 w = *(const uint2*)(sty.base + LDS_NB + (i * BLK + (lane / BLK) * 4) * 2);
                    nb[i][0] = w.x;
                    nb[i][1] = w.y;
                }
            } else {
                const int cc = lane & 15;
                const int rows_left = a.d_out - (mw0 + cc * 8);  // rows past d_out hold copies: their factors count as 0
                const char* br = sty.base + LDS_NB + cc * 8 * RANK * 2;  // 8 rows x RANK bf16, l fastest
                uint32_t w[4 * RANK];
#pragma unroll
                for (int k = 0; k < RANK; ++k) {
                    const u32x4 v = *(const u32x4*)(br + 16 * k);
                    w[4 * k] = v[0]; w[4 * k + 1] = v[1]; w[4 * k + 2] = v[2]; w[4 * k + 3] = v[3];
                }
                constexpr int WPR = RANK / 2;  // dwords per row
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int lp = 0; lp < WPR; ++lp) {
                        const uint32_t ra = w[(2 * q) * WPR + lp], rb = w[(2 * q + 1) * WPR + lp];  // rows 2q, 2q + 1: (l, l + 1)
                        const bool in = 2 * q < rows_left;
                        bp[2 * lp][q] = in ? ((ra & 0xFFFFu) | (rb << 16)) : 0u;
                        bp[2 * lp + 1][q] = in ? ((ra >> 16) | (rb & 0xFFFF0000u)) : 0u;
                    }
            }
        }
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int l = 0; l < RANK; ++l) pf_t[j][l] = *(const float*)(sty.base + LDS_T + ((j * BLK + (lane & (BLK - 1))) * RANK + l) * 4);
        // K-slots 0..7 (hi part of c*t), 8..15 (lo part); the 16x16x32 block has 16 more, left at zero
        const int half = lane / BLK;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            uint32_t tb[4] = {0u, 0u, 0u, 0u};
            float ct[RANK];
            bf16_parts(a.c, pf_t[j], half == 1, ct);
#pragma unroll
            for (int l = 0; l < RANK; l += 2) tb[l >> 1] = half < 2 ? pack_bf16x2(ct[l], l + 1 < RANK ? ct[l + 1] : 0.f) : 0u;
            const u32x4 bfrag = {tb[0], tb[1], tb[2], tb[3]};
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                u32x4 afrag = {0u, 0u, 0u, 0u};
                const char* ar = sty.base + LDS_A + (i * BLK + (lane & (BLK - 1))) * RANK * 2;
                if constexpr (RANK == 1) afrag[0] = *(const uint16_t*)ar;
                else
#pragma unroll
                    for (int w = 0; w < AW; ++w) afrag[w] = *(const uint32_t*)(ar + 4 * w);
                MT::mma(afrag, bfrag, acc[i][j]);  // rows m >= d_out hold a clamped copy and are never stored
            }
        }
    }

    static constexpr __host__ __device__ int lds_per_wave(int wtm) { return RowStagerSwz::bytes(wtm); }

    __device__ __forceinline__ LeanEpi(const Args& a_, char* slice, int lane) : a(a_), sty{slice, lane, lane & (BLK - 1)} {}

    // the persistent kernel names the column block
    template <int J>
    __device__ __forceinline__ void column_at(int n, bool)
    {
        if constexpr (PROJ_ROWS) tn = 0.f;
        if constexpr (RESID) load_residual<(J + 1) & 1>(n + BLK);  // the next column block (past the last one: a clamped re-read that is never used)
    }

    // ... and the row block (a compile-time index into per-block registers)
    template <int I, int J = 0>
    __device__ __forceinline__ void store4_at(int m, int, const float (&v)[4], bool valid, int ml)
    {
        float y[4] = {v[0], v[1], v[2], v[3]};
        if constexpr ((LEAN & LEAN_GELU) != 0) gelu_bf16_grade4(y);
        if constexpr (RESID) {
            static_assert(!PROJ, "not combined with the residual form");
            // each output element is read here and written by flush exactly once, so Y may be the residual buffer itself
            // (rows and columns past the end hold clamped copies and are never stored)
            y[0] += bf16_lo(rres[J & 1][I].x); y[1] += bf16_hi(rres[J & 1][I].x);
            y[2] += bf16_lo(rres[J & 1][I].y); y[3] += bf16_hi(rres[J & 1][I].y);
        }
        const uint32_t p0 = pack_bf16x2(y[0], y[1]), p1 = pack_bf16x2(y[2], y[3]);
        if constexpr (PROJ_ROWS) {
            if (valid && m < a.d_out) {
                tn = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, p0), __builtin_bit_cast(bf16x2_t, nb[I][0]), tn, false);
                tn = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, p1), __builtin_bit_cast(bf16x2_t, nb[I][1]), tn, false);
            }
        }
        sty.put(RowStagerSwz::pitch(WTM), ml, p0, p1);
    }

    template <int W>
    __device__ __forceinline__ void flush(int mw0, int nb0, int n_rows)
    {
        if constexpr (PROJ_FLUSH) {
            // The stager's flush with the projections formed on the way out: the 16 lanes that read one staged row (8 outputs
            // each) multiply them with their B' and add up across the row of lanes.
            static_assert(W == WTM, "16 chunks of 8 outputs per staged row, 4 rows per pass of the wave");
            constexpr int P = RowStagerSwz::pitch(WTM);
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the wave's own LDS writes have landed
            __builtin_amdgcn_wave_barrier();
            const int cc = sty.lane & 15;
            const int m = mw0 + cc * 8;
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int r = it * 4 + (sty.lane >> 4);
                const int n = nb0 + r;
                const u32x4 v = *(const u32x4*)(sty.base + r * P + (((cc ^ r) & 15) << 4));
                if (n < n_rows && m < a.d_out) {
                    uint16_t* dst = (uint16_t*)a.Y + (int64_t)n * a.d_out + m;
                    if (m + 8 <= a.d_out) *(u32x4*)dst = v;
                    else *(uint2*)dst = make_uint2(v[0], v[1]);
                }
                const uint32_t vw[4] = {v[0], v[1], v[2], v[3]};  // (bit_cast of a vector element, v[q], reads element 0 whatever q is)
                float ts[RANK];
#pragma unroll
                for (int l = 0; l < RANK; ++l) {
                    ts[l] = 0.f;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        ts[l] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, vw[q]), __builtin_bit_cast(bf16x2_t, bp[l][q]), ts[l], false);
                }
#pragma unroll
                for (int l = 0; l < RANK; ++l) ts[l] = row_sum16(ts[l]);
                if (cc == 0 && n < n_rows && mw0 < a.d_out) {
                    float* dst = a.next_part + ((int64_t)(mw0 >> 7) * n_rows + n) * RANK;
                    if constexpr (RANK == 2) *(float2*)dst = make_float2(ts[0], ts[1]);
                    else *(float4*)dst = make_float4(ts[0], ts[1], ts[2], ts[3]);
                }
            }
            __builtin_amdgcn_wave_barrier();  // the slice is reused by the next column block
        } else {
            sty.template flush<WTM, BLK>((uint16_t*)a.Y, a.d_out, mw0, nb0, n_rows, a.d_out);
        }
        if constexpr (PROJ_ROWS) {
            static_assert(W == WTM, "slabs of 128 rows, four lane groups per column");
            float tsum = tn + __shfl_xor(tn, 16, 64);
            tsum += __shfl_xor(tsum, 32, 64);
            const int n = nb0 + (sty.lane & 15);
            if (sty.lane < 16 && n < n_rows && mw0 < a.d_out) a.next_part[(int64_t)(mw0 >> 7) * n_rows + n] = tsum;
        }
    }
};

// The general epilogue, for 4 consecutive outputs m .. m + 3 of a row n: correction in fp32, activation, residual, store, every
// option at run time.  Used by the parked form of the tiles and by the small kernels.  Where the factors come from:
//   REGEN  (rank 1, one row per member): regenerated in registers from the counter stream -- each entry of A is needed exactly
//          once over the grid, so nothing is stored or re-read (the cache is filled on the way if one is kept);
//   otherwise read from a materialised [member][d_out][RANK] buffer (written just before by the noise kernel, the caller's
//          A_cache if one was given).
template <bool BF16, int RANK, bool REGEN>
struct FwdRowEpi {
    static constexpr bool IS_BF16 = BF16;
    typedef float value_t;
    typedef FwdArgs Args;
    // groups whose side data is in flight while as many are finished; with REGEN their blocks are independent chains
    static constexpr int PARKED = (REGEN || RANK <= 2) ? 4 : (RANK == 4 ? 2 : 1);
    static constexpr int ZW = REGEN ? 1 : (BF16 ? 2 * RANK : 4 * RANK);  // 32-bit words of the 4 rows' factors
    // a bf16 residual travels with the side data while registers allow: read at the store, its latency stood behind every group
    // (512 -> 1024, 3236 rows in antithetic pairs, rank 1: the layer 26.3 us then, 22.3 now; 2048 -> 8192, 512 x 3 rows, rank 4: 99.8 / 94.2)
    static constexpr bool RESID_AHEAD = BF16 && (REGEN || RANK <= 4);
    struct Side {
        float t[RANK];
        uint32_t z[ZW];
        uint2 r;
    };
    const Args a;
    __device__ __forceinline__ FwdRowEpi(const Args& a_) : a(a_) {}
    template <class MT>
    __device__ __forceinline__ void extra(typename MT::acc_t&, int, int, int, int) const {}
    __device__ __forceinline__ void side(int m, int n, Side& s) const
    {
        if (RESID_AHEAD && a.resid && a.y_bf16) s.r = *(const uint2*)((const uint16_t*)a.resid + (int64_t)n * a.d_out + m);
        if (a.c == 0.f) return;  // unperturbed: there are no projections (t is NULL)
#pragma unroll
        for (int l = 0; l < RANK; ++l) s.t[l] = a.t[(int64_t)n * RANK + l];
        if constexpr (!REGEN) {
            const int64_t aoff = ((int64_t)fast_div(a.by_s, (uint32_t)n) * a.d_out + m) * RANK;  // element offset of A_i[m][0]
            const char* src = (const char*)a.A_buf + aoff * (BF16 ? 2 : 4);
            if constexpr (BF16 && RANK == 1) {
                const uint2 p = *(const uint2*)src;
                s.z[0] = p.x; s.z[1] = p.y;
            } else {
                // m and d_out are multiples of 4: 4 rows of 2 bf16 or 1 fp32 and more are 16-byte pieces
#pragma unroll
                for (int k = 0; k < ZW; k += 4) {
                    const uint4 p = *(const uint4*)(src + 4 * k);
                    s.z[k] = p.x; s.z[k + 1] = p.y; s.z[k + 2] = p.z; s.z[k + 3] = p.w;
                }
            }
        }
    }
    __device__ __forceinline__ void finish(int m, int n, const float (&v)[4], const Side& s, bool valid) const
    {
        float y[4] = {v[0], v[1], v[2], v[3]};
        const int64_t at = (int64_t)n * a.d_out + m;  // d_out is a multiple of 4: whole groups
        if (a.c != 0.f) {
            float z[4 * RANK];
            if constexpr (REGEN) {
                static_assert(RANK == 1, "in-register regeneration is the rank-1 path");
                const uint32_t member = a.member_begin + fast_div(a.by_s, (uint32_t)n), blk0 = (uint32_t)m >> 1;
                uint32_t pk[2] = {0u, 0u};
                if (a.pair_share) {
                    // antithetic pairs, one row per member: rows 2p and 2p + 1 need the same four factors and are held by lanes
                    // pair_share apart, so each generates one of the two Threefry blocks and they swap
                    const int b = n & 1;
                    uint32_t w0, w1;
                    noise_words(a.ka, member, blk0 + b, w0, w1);
                    float o0, o1;
                    normal_pair<!BF16>(w0, w1, o0, o1);
                    if constexpr (BF16) {
                        const uint32_t own = pack_bf16x2(o0, o1), oth = __shfl_xor(own, a.pair_share, 64);
                        pk[0] = b ? oth : own;
                        pk[1] = b ? own : oth;
                    } else {
                        const float x0 = __shfl_xor(o0, a.pair_share, 64), x1 = __shfl_xor(o1, a.pair_share, 64);
                        z[0] = b ? x0 : o0; z[1] = b ? x1 : o1;
                        z[2] = b ? o0 : x0; z[3] = b ? o1 : x1;
                    }
                } else {
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        uint32_t w0, w1;
                        noise_words(a.ka, member, blk0 + b, w0, w1);
                        normal_pair<!BF16>(w0, w1, z[2 * b], z[2 * b + 1]);
                        if constexpr (BF16) pk[b] = pack_bf16x2(z[2 * b], z[2 * b + 1]);
                    }
                }
                if constexpr (BF16) {
                    z[0] = bf16_lo(pk[0]); z[1] = bf16_hi(pk[0]);
                    z[2] = bf16_lo(pk[1]); z[3] = bf16_hi(pk[1]);
                }
                if (a.A_buf && valid) {  // (with pairs a kept cache goes the materialised way: here a row is a member)
                    if constexpr (BF16) *(uint2*)((uint16_t*)a.A_buf + at) = make_uint2(pk[0], pk[1]);
                    else *(float4*)((float*)a.A_buf + at) = make_float4(z[0], z[1], z[2], z[3]);
                }
            } else if constexpr (BF16) {
#pragma unroll
                for (int k = 0; k < ZW; ++k) {
                    z[2 * k] = bf16_lo(s.z[k]);
                    z[2 * k + 1] = bf16_hi(s.z[k]);
                }
            } else {
#pragma unroll
                for (int k = 0; k < ZW; ++k) z[k] = __uint_as_float(s.z[k]);
            }
            float tc[RANK];
#pragma unroll
            for (int l = 0; l < RANK; ++l) tc[l] = a.c * s.t[l];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float corr = 0.f;
#pragma unroll
                for (int l = 0; l < RANK; ++l) corr = fmaf(tc[l], z[e * RANK + l], corr);
                y[e] += corr;
            }
        }
        if (a.act == EGG_ACT_GELU) {
            if (a.y_bf16) gelu_bf16_grade4(y);
            else
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = 0.5f * y[e] * (1.0f + erff(y[e] * 0.70710678118654752f));
        }
        if (!valid) return;
        // each output element is read (residual) and then written by one lane, so Y may be the residual buffer itself (what the lanes
        // of clamped rows read of it is not used)
        if (a.y_bf16) {
            if (a.resid) {
                const uint2 rv = RESID_AHEAD ? s.r : *(const uint2*)((const uint16_t*)a.resid + at);
                y[0] += bf16_lo(rv.x); y[1] += bf16_hi(rv.x);
                y[2] += bf16_lo(rv.y); y[3] += bf16_hi(rv.y);
            }
            *(uint2*)((uint16_t*)a.Y + at) = make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
        } else {
            if (a.resid) {
                const float4 rv = *(const float4*)((const float*)a.resid + at);
                y[0] += rv.x; y[1] += rv.y; y[2] += rv.z; y[3] += rv.w;
            }
            *(float4*)((float*)a.Y + at) = make_float4(y[0], y[1], y[2], y[3]);
        }
    }
    // small kernels: one group at a time (their lanes do not hold pairs: pair_share is 0)
    __device__ __forceinline__ void apply4(int m, int n, const float (&v)[4]) const
    {
        Side s;
        side(m, n, s);
        finish(m, n, v, s, true);
    }
};

// fp32 products of up to four tiles of 32 x 32 per CU: a workgroup a tile, a wave a 16 x 16 block of it over all of K, four stages of K
// in flight.  K stays whole, so that a row does not depend on how many rows the call has.  Measured (whole calls with 4 rows per
// member at rank 1, us, 128 x 64 and 128 x 128 tiles / this): 256 x 64 x 256 18.5 / 14.1, x 2048 77.8 / 27.0; 512 x 512 x 1024 44.9 / 19.0;
// 1024 x 1024 x 1024 46.5 / 35.5; beyond the line, 1400 x 1000 x 1024 46.8 / 47.8, 2048 x 1024 x 1024 47.3 / 60.0.  (K split over the
// four waves of a tile, its partial sums added through LDS, was 13.8, 27.2, 19.7 and 39.2.)
static bool deep_f32_tiles(int64_t M, int64_t N, int compute_units) { return ((M + 31) / 32) * ((N + 31) / 32) <= 4 * (int64_t)compute_units; }

template <class MT, int BM, int BN, int WM, int WN, class Epi>
static egg_status launch_gemm(eggroll_ctx* c, const char* name, const Operand& P, const Operand& Q, int kchunks,
                              typename Epi::Args ea)
{
    // (128 x 128 tiles: two workgroups share a CU, so no wave may take more than half of the registers)
    auto kern = gemm_nt_kernel<MT, BM, BN, WM, WN, false, Epi, (BM * BN <= 128 * 128 ? 2 : 1)>;
    const int tiles_m = (P.rows + BM - 1) / BM, tiles_n = (Q.rows + BN - 1) / BN;
    const size_t lds = std::max(gemm_lds_bytes<BM, BN>(), (size_t)WM * WN * parked_bytes_per_wave<BM / WM>());
    if (ea.pair_share) ea.pair_share = BM / WM / 4;  // lanes per row of the parked epilogue
    if (!operand_offsets_fit(P, BM) || !operand_offsets_fit(Q, BN)) return fail(c, EGG_EUNSUPPORTED, "operand strides too large for 32-bit tile offsets");
    egg_status st = ensure_dynamic_lds(c, (const void*)kern, (size_t)lds, "gemm smem attr");
    if (st != EGG_OK) return st;
    const int64_t grid = (int64_t)tiles_m * tiles_n;
    if (grid > 0x7FFFFFFF) return fail(c, EGG_EUNSUPPORTED, "too many tiles");
    KernelScope ks(c, shaped_name(c, name, P.rows, kchunks * 16 / (Epi::IS_BF16 ? 2 : 4)));
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(WM * WN * 64), lds, c->stream, P, Q, kchunks, tiles_m, tiles_n,
                       (const char*)c->zero_page.p, ea);
    return check_hip(c, hipGetLastError(), name);
}

// t[n] = sum over the 128-row slabs of d_out of the partial projections, in slab order (a fixed order: run-to-run identical)
// (sixteen loads in flight, and workgroups of one wave: 8192 rows are 128 of them.  One load per addition in workgroups of 256
// took 14.7 us for 8192 rows x 64 slabs.)
__global__ __launch_bounds__(64) void sum_slabs_kernel(const float* __restrict__ part, int slabs, int64_t R, float* __restrict__ t)
{
    const int64_t n = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (n >= R) return;
    float acc = 0.f;
    for (int p = 0; p < slabs; p += 16) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = part[(int64_t)min(p + k, slabs - 1) * R + n];  // clamped, unconditional
#pragma unroll
        for (int k = 0; k < 16; ++k) acc = p + k < slabs ? acc + v[k] : acc;
    }
    t[n] = acc;
}

egg_status launch_sum_slabs(eggroll_ctx* c, const float* part, int slabs, int64_t R, float* t)
{
    KernelScope ks(c, "project_sum_slabs");
    hipLaunchKernelGGL(sum_slabs_kernel, dim3((unsigned)((R + 63) / 64)), dim3(64), 0, c->stream, part, slabs, R, t);
    return check_hip(c, hipGetLastError(), "project_sum_slabs");
}

bool forward_fuses_next_projection(const egg_shape& s, egg_dtype io, egg_dtype yd, float sigma, egg_act act, bool resid)
{
    const int64_t R = s.member_count * (int64_t)s.rows_per_member;
    const int64_t big_tiles = ((s.d_out + 255) / 256) * ((R + 255) / 256);
    return io == EGG_BF16 && yd == EGG_BF16 && sigma != 0.f && (s.rank == 1 || s.rank == 2 || s.rank == 4) && !s.antithetic && act == EGG_ACT_GELU && !resid &&
           s.rows_per_member % 64 == 0 && s.rows_per_member > 1 && big_tiles >= 192 && s.d_in % 64 == 0;
}

// The persistent kernel for store-only epilogues: one workgroup per compute unit walks the tiles.
template <class MT, int BM, int BN, int WM, int WN, class Epi>
static egg_status launch_gemm_persistent(eggroll_ctx* c, const char* name, const Operand& P, const Operand& Q, int kchunks,
                                         typename Epi::Args ea)
{
    auto kern = gemm_nt_persistent_kernel<MT, BM, BN, WM, WN, Epi>;
    const int tiles_m = (P.rows + BM - 1) / BM, tiles_n = (Q.rows + BN - 1) / BN;
    const size_t lds = gemm_lds_bytes<BM, BN>() + (size_t)WM * WN * Epi::lds_per_wave(BM / WM);
    if (ea.c != 0.f && ea.S % 64 != 0) return fail(c, EGG_EINVAL, "store-only epilogue launched with a correction left to apply");
    if (!operand_offsets_fit(P, BM) || !operand_offsets_fit(Q, BN)) return fail(c, EGG_EUNSUPPORTED, "operand strides too large for 32-bit tile offsets");
    egg_status st = ensure_dynamic_lds(c, (const void*)kern, lds, "gemm smem attr");
    if (st != EGG_OK) return st;
    const int64_t total = (int64_t)tiles_m * tiles_n;
    if (total > 0x7FFFFFFF) return fail(c, EGG_EUNSUPPORTED, "too many tiles");
    const unsigned grid = (unsigned)(total < c->compute_units ? total : c->compute_units);
    KernelScope ks(c, shaped_name(c, name, P.rows, kchunks * 8));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(WM * WN * 64), lds, c->stream, P, Q, kchunks, tiles_m, tiles_n,
                       (const char*)c->zero_page.p, ea);
    return check_hip(c, hipGetLastError(), name);
}

template <bool BF16, int RANK, bool REGEN>
static egg_status launch_forward_t(eggroll_ctx* c, const StreamKey& ka, const egg_shape& s, egg_dtype yd, float sigma,
                                   egg_act act, const void* W, const void* X, void* Y, const float* t, void* A_buf,
                                   const void* resid, const NextProjection* next)
{
    typedef FwdRowEpi<BF16, RANK, REGEN> Epi;
    const int esz = BF16 ? 2 : 4;
    const int64_t R = s.member_count * (int64_t)s.rows_per_member;
    // antithetic pairs: the epilogue sees pairs as members of 2S rows (noise id = row / 2S); the sign of
    // the odd member is already folded into its projections t
    const int anti = s.antithetic ? 2 : 1;
    Operand P{(const char*)W, (int64_t)s.d_in * esz, 16, s.d_out};
    Operand Q{(const char*)X, (int64_t)s.d_in * esz, 16, (int)R};
    const int kchunks = s.d_in * esz / 16;
    const int S = s.rows_per_member * anti;
    const int pairs = (REGEN && s.antithetic && sigma != 0.f) ? 1 : 0;
    FwdArgs ea{ka, (uint32_t)(s.member_begin / anti), S, s.d_out, make_fast_div((uint32_t)S), sigma / sqrtf((float)s.rank),
               (int)act, yd == EGG_BF16 ? 1 : 0, Y, t, A_buf, 0, resid, nullptr, nullptr};
    if constexpr (BF16) {
        if (next) {
            // the fused next-layer projection exists in one form: rank 1, 2 or 4 (the next layer's too), folded correction,
            // GELU, no residual
            if constexpr (!REGEN && (RANK == 1 || RANK == 2 || RANK == 4)) {
                if (forward_fuses_next_projection(s, EGG_BF16, yd, sigma, act, resid != nullptr)) {
                    const int slabs = (s.d_out + 127) / 128;
                    egg_status st = reserve(c, c->proj_part, (size_t)slabs * R * RANK * sizeof(float));
                    if (st != EGG_OK) return st;
                    ea.next_B = next->B;
                    ea.next_part = (float*)c->proj_part.p;
                    st = launch_gemm_persistent<MmaBf16Blk16, 256, 256, 2, 4, LeanEpi<RANK, LEAN_ON | LEAN_GELU | LEAN_PROJ>>(
                        c, "forward_gemm_bf16", P, Q, kchunks, ea);
                    if (st != EGG_OK) return st;
                    return launch_sum_slabs(c, (const float*)c->proj_part.p, slabs, R * RANK, next->t);
                }
            }
            return fail(c, EGG_EINVAL, "this layer cannot form the next layer's projections (ask forward_fuses_next_projection first)");
        }
        // bf16 out and no correction, or one that 16 neighbouring rows share among at most two members: folded into the
        // accumulators, store-only epilogue with the activation and the residual fixed at compile time.  The parked form is the
        // faster one where it applies (big tiles, S a multiple of 64, whole K stages).
        if (yd == EGG_BF16 && (ea.c == 0.f || (!REGEN && ea.S >= FOLD_MIN_ROWS))) {
            const bool parked = big_tiles(s.d_out, R, c->compute_units) && kchunks % 8 == 0 && (ea.c == 0.f || (RANK <= 8 && S % 64 == 0));
            if (!parked)
                return launch_forward_fold(c, FoldLayer{ea.S, s.d_out, s.d_in, s.rank, R, ea.c, act == EGG_ACT_GELU, W, X, A_buf, resid, Y, t});
            constexpr int LR = (REGEN || RANK > 8) ? 1 : RANK;
#define EGG_LEAN(L) \
    return launch_gemm_persistent<MmaBf16Blk16, 256, 256, 2, 4, LeanEpi<LR, L>>(c, "forward_gemm_bf16", P, Q, kchunks, ea)
            switch ((act == EGG_ACT_GELU ? LEAN_GELU : 0) | (resid ? LEAN_RESID : 0)) {
                case 0: EGG_LEAN(LEAN_ON);
                case LEAN_GELU: EGG_LEAN(LEAN_ON | LEAN_GELU);
                case LEAN_RESID: EGG_LEAN(LEAN_ON | LEAN_RESID);
                default: EGG_LEAN(LEAN_ON | LEAN_GELU | LEAN_RESID);
            }
#undef EGG_LEAN
        }
        // The correction per output (the same bits for any number of rows).  This epilogue is longer than a tile of 128 x 128 hides, so
        // the large tile pays earlier than in big_tiles: from more of them than half of the CUs, whatever of them is ragged (us,
        // 128 x 128 / 256 x 256: 3700 rows of 2048 -> 2100, S = 1 88.0 / 81.6; 3 rows per member at rank 4 100 / 93; 57344 of 2048 -> 104 250 / 231).
        const int deep = deep_tile(s.d_out, R, c->compute_units);
        if (deep == 32) return launch_gemm_deep<MmaBf16Blk16, Epi, 32>(c, "forward_gemm_bf16_small", P, Q, kchunks, ea);
        if (deep == 64) return launch_gemm_deep<MmaBf16Blk16, Epi, 64>(c, "forward_gemm_bf16_small", P, Q, kchunks, ea);
        ea.pair_share = pairs;
        if (((s.d_out + 255) / 256) * ((R + 255) / 256) > c->compute_units / 2)
            return launch_gemm<MmaBf16Blk16, 256, 256, 2, 4, Epi>(c, "forward_gemm_bf16", P, Q, kchunks, ea);
        // few rows against a large layer (the paper's own benchmark shape, batch 1024 on 8192 x 8192): tall
        // tiles keep one workgroup per CU busy where 256 x 256 tiles would leave half the chip idle
        const int64_t tall_tiles = ((s.d_out + 255) / 256) * ((R + 127) / 128);
        if (tall_tiles >= 192) {
            return launch_gemm<MmaBf16Blk16, 256, 128, 4, 2, Epi>(c, "forward_gemm_bf16_tall", P, Q, kchunks, ea);
        }
        return launch_gemm<MmaBf16Blk16, 128, 128, 2, 2, Epi>(c, "forward_gemm_bf16_small", P, Q, kchunks, ea);
    } else {
        if (next) return fail(c, EGG_EINVAL, "this layer cannot form the next layer's projections (ask forward_fuses_next_projection first)");
        // (every form runs the same chain of products, k ascending: a row is the same bits for any number of rows)
        if (deep_f32_tiles(s.d_out, R, c->compute_units)) return launch_gemm_deep<MmaF32Blk16, Epi, 32>(c, "forward_gemm_f32", P, Q, kchunks, ea);
        ea.pair_share = pairs;
        if (narrow_f32_tiles(s.d_out, R, c->compute_units)) return launch_gemm<MmaF32, 128, 64, 2, 2, Epi>(c, "forward_gemm_f32", P, Q, kchunks, ea);
        return launch_gemm<MmaF32, 128, 128, 2, 2, Epi>(c, "forward_gemm_f32", P, Q, kchunks, ea);
    }
}

egg_status launch_forward_gemm(eggroll_ctx* c, const StreamKey& ka, const egg_shape& s, egg_dtype io, egg_dtype yd,
                               float sigma, egg_act act, const void* W, const void* X, void* Y, const float* t,
                               bool regenerate, void* A_cache, const void* resid, const NextProjection* next, const void* A_ready)
{
    const bool bf = io == EGG_BF16;
    // rank 1 with one row per member (or the unperturbed pass): regenerate in the epilogue
    // (with antithetic pairs a kept cache has one entry per pair, not per row: that goes the materialised way)
    if (regenerate) {
        return bf ? launch_forward_t<true, 1, true>(c, ka, s, yd, sigma, act, W, X, Y, t, A_cache, resid, next)
                  : launch_forward_t<false, 1, true>(c, ka, s, yd, sigma, act, W, X, Y, t, A_cache, resid, next);
    }
    // otherwise materialise A once (into the caller's cache if there is one) and read it back
    void* A_buf = A_cache;
    if (A_ready && !A_cache) {
        A_buf = const_cast<void*>(A_ready);
    } else {
        const int anti = s.antithetic ? 2 : 1;  // one set of factors per pair
        if (!A_buf) {
            const size_t bytes = (size_t)(s.member_count / anti) * s.d_out * s.rank * (bf ? 2 : 4);
            egg_status st = reserve(c, c->a_buf, bytes);
            if (st != EGG_OK) return st;
            A_buf = c->a_buf.p;
        }
        const egg_status st = launch_noise(c, ka, (uint32_t)(s.member_begin / anti), s.member_count / anti, (int64_t)s.d_out * s.rank, io,
                                           EGG_NORMAL, 0, A_buf);
        if (st != EGG_OK) return st;
    }
#define EGG_FWD(B, R) return launch_forward_t<B, R, false>(c, ka, s, yd, sigma, act, W, X, Y, t, A_buf, resid, next)
    if (bf) {
        switch (s.rank) {
            case 1: EGG_FWD(true, 1);
            case 2: EGG_FWD(true, 2);
            case 4: EGG_FWD(true, 4);
            case 8: EGG_FWD(true, 8);
            default: EGG_FWD(true, 16);
        }
    } else {
        switch (s.rank) {
            case 1: EGG_FWD(false, 1);
            case 2: EGG_FWD(false, 2);
            case 4: EGG_FWD(false, 4);
            case 8: EGG_FWD(false, 8);
            default: EGG_FWD(false, 16);
        }
    }
#undef EGG_FWD
}

}  // namespace egg
