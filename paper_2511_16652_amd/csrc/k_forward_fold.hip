// The bf16 forward layer with the rank-r correction folded into the accumulators, for row groups of any length.
//
//   Y[n][m] += sum_l A_i[m][l] (c t[n][l]),  i = n / S
//
// is a contraction over the rank once the 16 columns (rows of X) of an MFMA block are allowed to belong to different members:
// the 32 K-slots of one v_mfma_f32_16x16x32_bf16 hold two members' factors A_a[m][0..r), A_b[m][0..r), each twice, against the
// bf16 halves (hi, then the rounding remainder lo) of c t -- and a column's entries are zero in the slots of the member it does
// not belong to.  With S >= 15 sixteen neighbouring rows touch at most two members, so one MFMA per block does it up to rank 8
// (two at rank 16); products are accurate to about 2^-16, as in the parked form of k_forward.hip, which needs a whole wave tile
// of 64 columns to belong to one member.  What follows is the store-only epilogue.  The general epilogue, which these shapes
// took before, applies the correction per element on the vector ALUs behind run-time decisions: at 33300 rows of 2048 -> 8192
// (S = 100, rank 2, GELU) the layer is 978 us with this form and was 1232.
// The operands come straight from memory (t and A of a column block: one batch of loads per block, the next block's in flight
// under this block's MFMAs); 16 rows x r entries of A are neighbours, so a load instruction touches few lines.
#include "forward_fold.hpp"
#include "gemm_core.hpp"
#include "gemm_small.hpp"

namespace egg {

struct FoldArgs {
    FastDiv by_s;   // n / S
    int d_out, rank;
    float c;
    void* Y;
    const float* t;
    const void* A;
    const void* resid;
};

// AW: 32-bit words of factors a lane holds per block: 1 (rank 1, 2), 2 (rank 4), 4 (rank 8, and each half of rank 16);
// 0: nothing to correct.  MB: 16-row blocks of a wave tile.
template <int AW, int LEAN, int MB>
struct FoldEpi {
    typedef float value_t;
    typedef FoldArgs Args;
    static constexpr int NB = 4, BLK = 16, WTM = MB * BLK;
    static constexpr bool RESID = (LEAN & LEAN_RESID) != 0;
    const Args a;
    RowStagerSwz sty;
    // residual pieces of the current and the next column block (two sets named at compile time; see k_forward.hip)
    uint2 rres[RESID ? 2 : 1][RESID ? MB : 1];
    int res_m0 = 0, res_rows = 0;
    static constexpr __host__ __device__ int lds_per_wave(int wtm) { return RowStagerSwz::bytes(wtm); }
    __device__ __forceinline__ FoldEpi(const Args& a_, char* slice, int lane) : a(a_), sty{slice, lane, lane & (BLK - 1)} {}
    template <int, int>
    __device__ __forceinline__ void prefetch(int, int, int, int) {}

    template <int SET>
    __device__ __forceinline__ void load_residual(int n)
    {
        if constexpr (RESID) {
            const uint16_t* rrow = (const uint16_t*)a.resid + (int64_t)min(n, res_rows - 1) * a.d_out;
#pragma unroll
            for (int i = 0; i < MB; ++i) rres[SET][i] = *(const uint2*)(rrow + min(res_m0 + i * BLK, a.d_out - 4));
        }
    }

    // operands of one MFMA per block of a column block: the lane's K-slots 8 (lane / 16) .. + 7
    struct Frag {
        uint32_t af[MB][AW > 0 ? AW : 1];
        float tv[AW > 0 ? 2 * AW : 1];
        bool own;  // the lane's column belongs to the member of the lane's slots
    };
    // up to rank 8: lane groups 0, 1 hold the block's first member (hi, lo), groups 2, 3 its second; at rank 16 the four groups
    // are (hi, terms 0..7), (hi, 8..15), (lo, 0..7), (lo, 8..15) of member number `pass`
    __device__ __forceinline__ void fetch(Frag& f, int mw0, int nb0, int lane, int n_rows, int pass) const
    {
        if constexpr (AW > 0) {
            const bool r16 = AW == 4 && a.rank == 16;
            const int g = lane >> 4;
            const int n = min(nb0 + (lane & 15), n_rows - 1);
            const int first = (int)fast_div(a.by_s, (uint32_t)min(nb0, n_rows - 1)), last = (int)fast_div(a.by_s, (uint32_t)min(nb0 + 15, n_rows - 1));
            const int slot = first + (r16 ? pass : g >> 1);
            const int member = min(slot, last), l0 = r16 ? (g & 1) * 8 : 0;
            f.own = (int)fast_div(a.by_s, (uint32_t)n) == slot;
            const float* tp = a.t + (int64_t)n * a.rank + l0;
#pragma unroll
            for (int l = 0; l < 2 * AW; ++l) f.tv[l] = tp[AW == 1 ? min(l, a.rank - 1) : l];
            const uint16_t* A0 = (const uint16_t*)a.A + (int64_t)member * a.d_out * a.rank + l0;
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int m = min(mw0 + i * BLK + (lane & 15), a.d_out - 1);  // rows m >= d_out hold a clamped copy and are never stored
                if constexpr (AW == 1) f.af[i][0] = *(const uint32_t*)(A0 + (a.rank == 1 ? m & ~1 : 2 * m));  // d_out is even: the word is inside
                else if constexpr (AW == 2) {
                    const uint2 v = *(const uint2*)(A0 + (int64_t)m * 4);
                    f.af[i][0] = v.x; f.af[i][1] = v.y;
                } else {
                    const u32x4 v = *(const u32x4*)(A0 + (int64_t)m * a.rank);
                    f.af[i][0] = v[0]; f.af[i][1] = v[1]; f.af[i][2] = v[2]; f.af[i][3] = v[3];
                }
            }
        }
    }
    template <class MT, int NB_>
    __device__ __forceinline__ void fold(const Frag& f, typename MT::acc_t (&acc)[MB][NB_], int j, int mw0, int lane) const
    {
        if constexpr (AW > 0) {
            const int g = lane >> 4;
            const bool lo_half = (AW == 4 && a.rank == 16) ? (g >> 1) != 0 : (g & 1) != 0;
            uint32_t tb[4] = {0u, 0u, 0u, 0u};
            float v[2 * AW];
            bf16_parts(a.c, f.tv, lo_half, v);
#pragma unroll
            for (int w = 0; w < AW; ++w) {
                const uint32_t p = pack_bf16x2(v[2 * w], (AW == 1 && a.rank == 1) ? 0.f : v[2 * w + 1]);
                tb[w] = f.own ? p : 0u;
            }
            const u32x4 bfrag = {tb[0], tb[1], tb[2], tb[3]};
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                u32x4 afrag = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int w = 0; w < AW; ++w) afrag[w] = f.af[i][w];
                if constexpr (AW == 1) {
                    // rank 1: the row's factor is one half of the word
                    const int m = min(mw0 + i * BLK + (lane & 15), a.d_out - 1);
                    if (a.rank == 1) afrag[0] = (afrag[0] >> ((m & 1) * 16)) & 0xFFFFu;
                }
                MT::mma(afrag, bfrag, acc[i][j]);
            }
        }
    }

    template <class MT, int MB_, int NB_>
    __device__ __forceinline__ void extra_mma(typename MT::acc_t (&acc)[MB_][NB_], int mw0, int nw0, int lane, int n_rows)
    {
        static_assert(MB_ == MB && NB_ == NB, "wave tile of the launched kernel");
        if constexpr (RESID) {
            res_m0 = mw0 + (lane / BLK) * 4;
            res_rows = n_rows;
            load_residual<0>(nw0 + (lane & (BLK - 1)));
        }
        if constexpr (AW > 0) {
            if (nw0 >= n_rows || mw0 >= a.d_out) return;  // nothing of this wave tile is stored
            Frag f[2];
            fetch(f[0], mw0, nw0, lane, n_rows, 0);
            static_for<0, NB>([&](auto jc) __attribute__((always_inline)) {
                constexpr int j = decltype(jc)::value;
                if constexpr (j + 1 < NB) fetch(f[(j + 1) & 1], mw0, nw0 + (j + 1) * BLK, lane, n_rows, 0);
                fold<MT, NB>(f[j & 1], acc, j, mw0, lane);
            });
            if (AW == 4 && a.rank == 16) {
                // the second member of the blocks that have one (others multiply by zero)
                static_for<0, NB>([&](auto jc) __attribute__((always_inline)) {
                    constexpr int j = decltype(jc)::value;
                    fetch(f[0], mw0, nw0 + j * BLK, lane, n_rows, 1);
                    fold<MT, NB>(f[0], acc, j, mw0, lane);
                });
            }
        }
    }

    template <int J>
    __device__ __forceinline__ void column_at(int n, bool)
    {
        if constexpr (RESID) load_residual<(J + 1) & 1>(n + BLK);  // the next column block (past the last one: a clamped re-read that is never used)
    }
    template <int I, int J>
    __device__ __forceinline__ void store4_at(int, int, const float (&v)[4], bool, int ml)
    {
        float y[4] = {v[0], v[1], v[2], v[3]};
        if constexpr ((LEAN & LEAN_GELU) != 0) gelu_bf16_grade4(y);
        if constexpr (RESID) {
            // each output element is read here and written by flush exactly once, so Y may be the residual buffer itself
            y[0] += bf16_lo(rres[J & 1][I].x); y[1] += bf16_hi(rres[J & 1][I].x);
            y[2] += bf16_lo(rres[J & 1][I].y); y[3] += bf16_hi(rres[J & 1][I].y);
        }
        sty.put(RowStagerSwz::pitch(WTM), ml, pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
    }
    template <int W>
    __device__ __forceinline__ void flush(int mw0, int nb0, int n_rows)
    {
        static_assert(W == WTM, "wave tile of the launched kernel");
        sty.template flush<WTM, BLK>((uint16_t*)a.Y, a.d_out, mw0, nb0, n_rows, a.d_out);
    }
};

// the same for one 16 x 16 block whose 4-row groups are stored straight from registers
template <int AW, int LEAN>
struct FoldSmallEpi {
    typedef float value_t;
    typedef FoldArgs Args;
    static constexpr bool IS_BF16 = true;
    const Args a;
    __device__ __forceinline__ FoldSmallEpi(const Args& a_) : a(a_) {}
    template <class MT>
    __device__ __forceinline__ void extra(typename MT::acc_t& acc, int m0, int n0, int lane, int n_rows) const
    {
        if constexpr (AW > 0) {
            const FoldEpi<AW, LEAN_ON, 1> e(a, nullptr, lane);
            typename FoldEpi<AW, LEAN_ON, 1>::Frag f;
            typename MT::acc_t one[1][1] = {{acc}};
            e.fetch(f, m0, n0, lane, n_rows, 0);
            e.template fold<MT, 1>(f, one, 0, m0, lane);
            if (AW == 4 && a.rank == 16) {
                e.fetch(f, m0, n0, lane, n_rows, 1);
                e.template fold<MT, 1>(f, one, 0, m0, lane);
            }
            acc = one[0][0];
        }
    }
    __device__ __forceinline__ void apply4(int m, int n, const float (&v)[4]) const
    {
        float y[4] = {v[0], v[1], v[2], v[3]};
        const int64_t at = (int64_t)n * a.d_out + m;  // d_out is a multiple of 4: whole groups
        if constexpr ((LEAN & LEAN_GELU) != 0) gelu_bf16_grade4(y);
        if constexpr ((LEAN & LEAN_RESID) != 0) {
            const uint2 r = *(const uint2*)((const uint16_t*)a.resid + at);
            y[0] += bf16_lo(r.x); y[1] += bf16_hi(r.x);
            y[2] += bf16_lo(r.y); y[3] += bf16_hi(r.y);
        }
        *(uint2*)((uint16_t*)a.Y + at) = make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
    }
};

template <int BM, int BN, int WM, int WN, int WG_PER_CU, bool TAIL, int AW, int LEAN>
static egg_status launch_fold_t(eggroll_ctx* c, const char* name, const Operand& P, const Operand& Q, int kchunks, const FoldArgs& ea)
{
    typedef FoldEpi<AW, LEAN, BM / WM / 16> Epi;
    static_assert(BN / WN == 64, "four column blocks per wave tile");
    auto kern = gemm_nt_persistent_kernel<MmaBf16Blk16, BM, BN, WM, WN, Epi, TAIL, WG_PER_CU>;
    const int tiles_m = (P.rows + BM - 1) / BM, tiles_n = (Q.rows + BN - 1) / BN;
    const size_t lds = gemm_lds_bytes<BM, BN>() + (size_t)WM * WN * Epi::lds_per_wave(BM / WM);
    if (!operand_offsets_fit(P, BM) || !operand_offsets_fit(Q, BN)) return fail(c, EGG_EUNSUPPORTED, "operand strides too large for 32-bit tile offsets");
    const egg_status st = ensure_dynamic_lds(c, (const void*)kern, lds, "gemm smem attr");
    if (st != EGG_OK) return st;
    const int64_t total = (int64_t)tiles_m * tiles_n;
    if (total > 0x7FFFFFFF) return fail(c, EGG_EUNSUPPORTED, "too many tiles");
    const int64_t most = (int64_t)c->compute_units * WG_PER_CU;
    KernelScope ks(c, shaped_name(c, name, P.rows, kchunks * 8));
    hipLaunchKernelGGL(kern, dim3((unsigned)std::min(total, most)), dim3(WM * WN * 64), lds, c->stream, P, Q, kchunks, tiles_m, tiles_n,
                       (const char*)c->zero_page.p, ea);
    return check_hip(c, hipGetLastError(), name);
}

// tiles that do not fill the chip: one workgroup per CU with four stages in flight
template <int AW, int LEAN>
static egg_status launch_fold_deep(eggroll_ctx* c, const Operand& P, const Operand& Q, int kchunks, const FoldArgs& ea)
{
    constexpr int BM = 128, BN = 128, WM = 2, WN = 2;
    typedef FoldEpi<AW, LEAN, BM / WM / 16> Epi;
    auto kern = gemm_nt_deep_kernel<MmaBf16Blk16, BM, BN, WM, WN, false, Epi>;
    const int tiles_m = (P.rows + BM - 1) / BM, tiles_n = (Q.rows + BN - 1) / BN;
    const size_t lds = 2 * gemm_lds_bytes<BM, BN>() + (size_t)WM * WN * Epi::lds_per_wave(BM / WM);
    if (!operand_offsets_fit(P, BM) || !operand_offsets_fit(Q, BN)) return fail(c, EGG_EUNSUPPORTED, "operand strides too large for 32-bit tile offsets");
    const egg_status st = ensure_dynamic_lds(c, (const void*)kern, lds, "gemm smem attr");
    if (st != EGG_OK) return st;
    KernelScope ks(c, shaped_name(c, "forward_gemm_bf16_small", P.rows, kchunks * 8));
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(WM * WN * 64), lds, c->stream, P, Q, kchunks, tiles_m, tiles_n,
                       (const char*)c->zero_page.p, c->conservative_waits ? 1 : 0, ea);
    return check_hip(c, hipGetLastError(), "forward_gemm_bf16_small");
}

template <int AW, int LEAN>
static egg_status launch_fold_aw(eggroll_ctx* c, const Operand& P, const Operand& Q, int kchunks, const FoldArgs& ea)
{
    // 256 x 256 tiles or four times as many of 128 x 128, two workgroups per CU or, where that leaves CUs empty, one.  K that is not made of whole stages takes the loaders with the zero page.
    const int deep = deep_tile(P.rows, Q.rows, c->compute_units);
    if (deep == 32) return launch_gemm_deep<MmaBf16Blk16, FoldSmallEpi<AW, LEAN>, 32>(c, "forward_gemm_bf16_small", P, Q, kchunks, ea);
    if (deep == 64) return launch_gemm_deep<MmaBf16Blk16, FoldSmallEpi<AW, LEAN>, 64>(c, "forward_gemm_bf16_small", P, Q, kchunks, ea);
    if (big_tiles(P.rows, Q.rows, c->compute_units)) {
        if constexpr (AW > 0)  // (whole stages and nothing to correct: the parked form's kernel)
            if (kchunks % 8 == 0) return launch_fold_t<256, 256, 2, 4, 1, false, AW, LEAN>(c, "forward_gemm_bf16", P, Q, kchunks, ea);
        return launch_fold_t<256, 256, 2, 4, 1, true, AW, LEAN>(c, "forward_gemm_bf16", P, Q, kchunks, ea);
    }
    if (((P.rows + 127) / 128) * (((int64_t)Q.rows + 127) / 128) <= c->compute_units) return launch_fold_deep<AW, LEAN>(c, P, Q, kchunks, ea);
    return launch_fold_t<128, 128, 2, 2, 2, true, AW, LEAN>(c, "forward_gemm_bf16_small", P, Q, kchunks, ea);
}

template <int LEAN>
static egg_status launch_fold_lean(eggroll_ctx* c, const FoldLayer& l, const Operand& P, const Operand& Q, int kchunks, const FoldArgs& ea)
{
    if (l.c == 0.f) return launch_fold_aw<0, LEAN>(c, P, Q, kchunks, ea);
    if (l.rank <= 2) return launch_fold_aw<1, LEAN>(c, P, Q, kchunks, ea);
    if (l.rank == 4) return launch_fold_aw<2, LEAN>(c, P, Q, kchunks, ea);
    return launch_fold_aw<4, LEAN>(c, P, Q, kchunks, ea);
}

egg_status launch_forward_fold(eggroll_ctx* c, const FoldLayer& l)
{
    if (l.c != 0.f && l.S < FOLD_MIN_ROWS) return fail(c, EGG_EINVAL, "folded layer: fewer than %d rows per member", FOLD_MIN_ROWS);
    const Operand P{(const char*)l.W, (int64_t)l.d_in * 2, 16, l.d_out};
    const Operand Q{(const char*)l.X, (int64_t)l.d_in * 2, 16, (int)l.R};
    const FoldArgs ea{make_fast_div((uint32_t)l.S), l.d_out, l.rank, l.c, l.Y, l.t, l.A, l.resid};
    const int kchunks = l.d_in / 8;
    if (l.gelu) return l.resid ? launch_fold_lean<LEAN_ON | LEAN_GELU | LEAN_RESID>(c, l, P, Q, kchunks, ea) : launch_fold_lean<LEAN_ON | LEAN_GELU>(c, l, P, Q, kchunks, ea);
    return l.resid ? launch_fold_lean<LEAN_ON | LEAN_RESID>(c, l, P, Q, kchunks, ea) : launch_fold_lean<LEAN_ON>(c, l, P, Q, kchunks, ea);
}

}  // namespace egg
