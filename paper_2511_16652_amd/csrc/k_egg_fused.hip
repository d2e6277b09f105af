// The integer model at its pretraining width (D = 256) in one kernel: a workgroup takes 32, 96 or 128 members through all layers and
// all tokens of the call, bit-exact (the passes it stands for are in k_egg_model.hip; they remain for other widths and for shifts whose
// folded arithmetic could overflow).
//
// A member's row depends on no other, so nothing has to leave the CU but the recurrent state and the logits.  Launched pass by pass, a
// layer was eight launches that moved every activation row through memory: 113 us per layer and token for 32768 members, 48 here (whole
// step of 6 layers and 4 tokens 3300 -> 1700 us).  What remains is the weights, 768 KB per layer and token into every CU from L2 (64
// bytes/ns would be 12 us), the members' factors, and the arithmetic: per CU and layer 25 thousand cycles of MFMAs (11 us) and 48
// thousand of vector ALU (22 us), which hide little of each other: two waves to a SIMD, and all waves of a workgroup multiply and
// finish at the same time.  Wave w of eight owns outputs 32 w .. 32 w + 31 of every 256-wide product for all rows of the workgroup:
//   * weight fragments come from a copy laid out in the order of their use (a small kernel writes it at the start of the call; one
//     KB per load and wave); each weight byte enters a CU once per workgroup, through a ring of four k steps that runs on over the epilogues;
//   * the products' rows are permuted (weight_row) so that a lane's accumulators of a 32 x 32 block are 16 neighbouring outputs of
//     one row: factors, biases and state are read as 16-byte pieces, and y, the gates' operands and the state stay in registers of the
//     lane that owns them from one product to the next;
//   * activations that the next product reads lie in LDS, 256 bytes a row, 16-byte pieces XOR-swizzled by the row (no bank conflicts);
//     row sums (normalisation, u . B) are added over the waves through small tables in LDS;
//   * the gates and residual sums run on packed 16-bit arithmetic; shift, saturation and packing of the outputs are v_ashr_pk_i8_i32.
// Tried: two workgroups of four waves and 64 rows on a CU (1170 us of 1160), 64 rows on sixteen waves with 128 registers (1200), a start
// of every second workgroup half a product later and wave priorities around the products (no change).
#include "common.hpp"
#include "gemm_core.hpp"
#include <algorithm>

namespace egg {

typedef short i16x2 __attribute__((ext_vector_type(2)));

constexpr int EGG_D = 256, EGG_SLAB = EGG_D * EGG_D;   // a slab: 256 outputs x 256 inputs
constexpr int EGG_LAYER_SLABS = 12;                    // Uf, Wf, Wh, Uh; mlp1 0, 1, mlp2 0, mlp1 2, mlp2 1, mlp1 3, mlp2 2, 3

struct EggFusedArgs {
    const u32x4* w;            // weights in the order of use: 12 slabs per layer, then the head
    const int8_t *emb, *ln1, *ln2, *ln_out, *bias;   // bias: [L][2][D]
    const int8_t *embA, *embB, *headA, *headB;       // factors [ids][n]
    const int8_t* factors;     // layer 0's; A and B of Wf, Uf, Wh, Uh in turn, A1, B1, A2, B2
    int64_t fD, f4D;           // bytes of a factor array of D and of 4 D values per id
    const uint8_t* tokens;     // [T][rows]
    const int8_t* S_in;        // [L][rows][D]
    int8_t *S_out, *logits;    // logits: [T][rows][256]
    int64_t rows;
    int L, T, anti, corr_shift, out_shift;
};

// row of the weight slab behind row m of a 32 x 32 block's first operand: accumulators 4 q + e of lane half h are row 8 q + 4 h + e
__device__ __forceinline__ int weight_row(int m) { return 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3); }

// slabs in the order of their use; a thread moves 16 bytes: [slab][wave][k step][lane]
__global__ __launch_bounds__(256) void egg_lay_weights_kernel(const int8_t* __restrict__ gru_w, const int8_t* __restrict__ mlp1,
                                                              const int8_t* __restrict__ mlp2, const int8_t* __restrict__ head, int L,
                                                              u32x4* __restrict__ out)
{
    const int slab = blockIdx.x >> 4;
    const int at = ((blockIdx.x & 15) << 8) + threadIdx.x;   // 16-byte piece of the slab
    const int lane = at & 63, ks = (at >> 6) & 7, wave = at >> 9;
    const int j = wave * 32 + weight_row(lane & 31), k = (2 * ks + (lane >> 5)) * 16;
    const int layer = slab / EGG_LAYER_SLABS, s = slab % EGG_LAYER_SLABS;
    const int8_t* src;
    if (layer == L) src = head + (size_t)j * EGG_D + k;
    else if (s < 4) {
        const int m = s == 0 ? 1 : s == 1 ? 0 : s;   // Uf, Wf, Wh, Uh
        src = gru_w + ((size_t)layer * 4 + m) * EGG_SLAB + (size_t)j * EGG_D + k;
    } else {
        constexpr int SECOND = 0x0D4;   // slabs 4 + i that belong to the second matrix: i = 2, 4, 6, 7
        const int i = s - 4;
        const bool second = (SECOND >> i) & 1;
        const int c = second ? (i == 7 ? 3 : i / 2 - 1) : (i < 2 ? i : (i + 1) / 2);
        if (second) src = mlp2 + ((size_t)layer * EGG_D + j) * (4 * EGG_D) + c * EGG_D + k;
        else src = mlp1 + ((size_t)layer * 4 + c) * EGG_SLAB + (size_t)j * EGG_D + k;
    }
    out[(size_t)slab * (EGG_SLAB / 16) + at] = *(const u32x4*)src;
}

// ---- packed bytes ------------------------------------------------------------------------------------------------------
__device__ __forceinline__ i16x2 as_pair(uint32_t w) { return __builtin_bit_cast(i16x2, w); }
__device__ __forceinline__ uint32_t as_word(i16x2 p) { return __builtin_bit_cast(uint32_t, p); }
__device__ __forceinline__ i16x2 even_bytes(uint32_t w) { return (i16x2)(as_pair(w) << (short)8) >> (short)8; }   // 0 and 2, sign-extended
__device__ __forceinline__ i16x2 odd_bytes(uint32_t w) { return as_pair(w) >> (short)8; }                       // 1 and 3
__device__ __forceinline__ uint32_t merge_bytes(i16x2 even, i16x2 odd) { return __builtin_amdgcn_perm(as_word(odd), as_word(even), 0x06020400u); }
__device__ __forceinline__ i16x2 sat127(i16x2 v)
{
    return __builtin_elementwise_max(__builtin_elementwise_min(v, (i16x2){127, 127}), (i16x2){-127, -127});
}
__device__ __forceinline__ i16x2 clip(i16x2 v) { return __builtin_elementwise_max(v, (i16x2){-127, -127}); }
// I8(a + b) of four bytes in [-127, 127]: with the bytes in the upper halves of 16 bits the saturating addition does the clipping,
// but for -128
__device__ __forceinline__ uint32_t add_sat4(uint32_t a, uint32_t b)
{
    const uint32_t ae = __builtin_amdgcn_perm(a, a, 0x020C000Cu), be = __builtin_amdgcn_perm(b, b, 0x020C000Cu);
    const i16x2 low = {-127 * 256, -127 * 256};
    const i16x2 e = __builtin_elementwise_max(__builtin_elementwise_add_sat(as_pair(ae), as_pair(be)), low);
    const i16x2 o = __builtin_elementwise_max(__builtin_elementwise_add_sat(as_pair(a & 0xFF00FF00u), as_pair(b & 0xFF00FF00u)), low);
    return __builtin_amdgcn_perm(as_word(o), as_word(e), 0x07030501u);
}
__device__ __forceinline__ uint32_t ashr_pack4(int a, int b, int c, int d, int sh)   // four values shifted right and saturated to [-128, 127]
{
    const uint32_t lo = (uint16_t)__builtin_amdgcn_ashr_pk_i8_i32(a, b, sh), hi = (uint16_t)__builtin_amdgcn_ashr_pk_i8_i32(c, d, sh);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}
__device__ __forceinline__ uint32_t abs_sum4(uint32_t w, uint32_t acc) { return __builtin_amdgcn_sad_u8(w ^ 0x80808080u, 0x80808080u, acc); }
__device__ __forceinline__ int dot16(const u32x4& a, const u32x4& b)
{
    int d = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) d = __builtin_amdgcn_sdot4((int)a[q], (int)b[q], d, false);
    return d;
}
// sum of the two lanes of a row, in both
__device__ __forceinline__ int halves_sum(int v)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 p = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    return (int)(p[0] + p[1]);
}

// What the barriers of this kernel order is LDS only: loads of weights and factors stay in flight across them.
__device__ __forceinline__ void lds_phase()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// A uniform pointer (to global memory) that stays one: added to a lane's offset only in the access itself.  (Otherwise sums of both are
// kept over the loops, two registers each.)
#define EGG_GLOBAL __attribute__((address_space(1)))
__device__ __forceinline__ EGG_GLOBAL const int8_t* uniform(const int8_t* p)
{
    EGG_GLOBAL const int8_t* g = (EGG_GLOBAL const int8_t*)p;
    asm volatile("" : "+s"(g));
    return g;
}
__device__ __forceinline__ u32x4 load16(const int8_t* base, uint32_t at) { return *(EGG_GLOBAL const u32x4*)(uniform(base) + at); }
// keeps a packed value packed: what was unpacked from it, or goes into it, does not live on in its place
__device__ __forceinline__ void hold(u32x4& v) { asm volatile("" : "+v"(v)); }

// Products of 24-bit integers whose operands are picked out of packed words by the multiply itself (the destination is a whole register, so
// none of the hazards of partial writes apply): a whole word and signed byte E, signed bytes E of both, unsigned byte E and signed half H
#define EGG_MUL_SDWA(OPS, A, S0, B, S1) asm("v_mul_i32_i24_sdwa %0, " OPS " dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:" S0 " src1_sel:" S1 : "=v"(d) : "v"(A), "v"(B))
template <int E>
__device__ __forceinline__ int mul24_word_byte(int a, uint32_t b)
{
    int d;
    if constexpr (E == 0) EGG_MUL_SDWA("%1, sext(%2)", a, "DWORD", b, "BYTE_0");
    else if constexpr (E == 1) EGG_MUL_SDWA("%1, sext(%2)", a, "DWORD", b, "BYTE_1");
    else if constexpr (E == 2) EGG_MUL_SDWA("%1, sext(%2)", a, "DWORD", b, "BYTE_2");
    else EGG_MUL_SDWA("%1, sext(%2)", a, "DWORD", b, "BYTE_3");
    return d;
}
template <int E>
__device__ __forceinline__ int mul24_bytes(uint32_t a, uint32_t b)
{
    int d;
    if constexpr (E == 0) EGG_MUL_SDWA("sext(%1), sext(%2)", a, "BYTE_0", b, "BYTE_0");
    else if constexpr (E == 1) EGG_MUL_SDWA("sext(%1), sext(%2)", a, "BYTE_1", b, "BYTE_1");
    else if constexpr (E == 2) EGG_MUL_SDWA("sext(%1), sext(%2)", a, "BYTE_2", b, "BYTE_2");
    else EGG_MUL_SDWA("sext(%1), sext(%2)", a, "BYTE_3", b, "BYTE_3");
    return d;
}
template <int E>
__device__ __forceinline__ int mul24_ubyte_half(uint32_t a, i16x2 b)   // half E / 2
{
    int d;
    const uint32_t bw = as_word(b);
    if constexpr (E == 0) EGG_MUL_SDWA("%1, sext(%2)", a, "BYTE_0", bw, "WORD_0");
    else if constexpr (E == 1) EGG_MUL_SDWA("%1, sext(%2)", a, "BYTE_1", bw, "WORD_0");
    else if constexpr (E == 2) EGG_MUL_SDWA("%1, sext(%2)", a, "BYTE_2", bw, "WORD_1");
    else EGG_MUL_SDWA("%1, sext(%2)", a, "BYTE_3", bw, "WORD_1");
    return d;
}
#undef EGG_MUL_SDWA

// RB blocks of 32 rows to a workgroup
template <int RB, bool DOT24>
__global__ __launch_bounds__(512, RB == 1 ? 4 : 2) void egg_layers_kernel(EggFusedArgs a)
{
    constexpr int ROWS = 32 * RB, BUF = ROWS * EGG_D, WAVES = 8;
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    // activations [row][256]: u, the state (then even quarters of the hidden row), f^ (odd quarters); byte offsets
    constexpr int bufU = 0, bufS = BUF, bufF = 2 * BUF;
    // five tables [row][wave] behind the buffers: byte offsets
    constexpr int TROW = WAVES * 4, TAB = ROWS * TROW, t_abs = 3 * BUF;   // sums of |y|
    constexpr int t_u0 = t_abs + TAB;                 // u . B of the product that reads u
    constexpr int t_u1 = t_u0 + TAB;                  // u . B_Wh
    constexpr int t_s = t_u1 + TAB;                   // s . B_Uf
    constexpr int t_h = t_s + TAB;                    // f^ . B_Uh, hidden . B_mlp2

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    const uint32_t col = wave * 32 + h * 16;         // first of this lane's 16 columns
    const int swz = n & 15;
    int rd = n * EGG_D + ((h ^ swz) << 4);           // operand reads: + block, ^ k step << 5
    int tr = n * TROW;                               // row of a table
    int wr = n * EGG_D + (((2 * wave + h) ^ swz) << 4);
    const int cs = a.corr_shift, sh = a.corr_shift + a.out_shift;
    // Arrays of rows and of factors are addressed from the workgroup's first row and id, uniformly but for one offset of the lane.  Rows
    // past the end repeat the last one and are not stored; factor arrays are long enough for whole workgroups.
    const int last = (int)min((int64_t)ROWS, a.rows - row0) - 1;
    const int64_t id0 = a.anti ? row0 >> 1 : row0;
    const int ids_block = a.anti ? 16 : 32;          // per block of 32 rows
    const int nid = n >> a.anti;                     // (row0 is even)
    int n_row = n, n_id = nid;
    auto row_at = [&](int b) __attribute__((always_inline)) { return (uint32_t)(min(32 * b + n_row, last) * EGG_D + col); };
    auto live = [&](int b) __attribute__((always_inline)) { return 32 * b + n_row <= last; };
    uint32_t f_lane = (uint32_t)(nid * EGG_D + col), f_lane4 = (uint32_t)(nid * 4 * EGG_D + col);
    const bool neg = a.anti && (n & 1);

    // Weight fragments: a ring of four k steps that runs on from one product to the next, so that their stream does not stop while an
    // epilogue runs; w points at the product's slab.
    i32x16 acc[RB], acc2[RB];
    u32x4 wf[4];
    const u32x4* const w_first = a.w + wave * 512;
    const u32x4* w = w_first;   // (uniform)
    auto load_w = [&](const u32x4* slab, int ks) __attribute__((always_inline)) {
        wf[ks & 3] = load16((const int8_t*)(slab + ks * 64), lane * 16);
    };
    auto multiply_then = [&](int buf, i32x16 (&c)[RB], const u32x4* next) __attribute__((always_inline)) {
        int at = rd + buf;   // (one register and immediate offsets of the blocks: those of a buffer at 64 KB would not fit)
        asm volatile("" : "+v"(at));
        constexpr int AHEAD = RB > 2 ? 2 : 1;   // operand pieces so far ahead, no further (the compiler would ask for all 8 RB of them first)
        u32x4 x[AHEAD + 1];
        auto piece = [&](int p) __attribute__((always_inline)) { return *(const u32x4*)(lds + (p % RB) * 32 * EGG_D + (at ^ ((p / RB) << 5))); };
#pragma unroll
        for (int p = 0; p < AHEAD; ++p) x[p] = piece(p);
#pragma unroll
        for (int p = 0; p < 8 * RB; ++p) {
            const int ks = p / RB, b = p % RB;
            if (p + AHEAD < 8 * RB) x[(p + AHEAD) % (AHEAD + 1)] = piece(p + AHEAD);
            MmaI8::mma(wf[ks & 3], x[p % (AHEAD + 1)], c[b]);
            if (b == RB - 1) load_w(ks < 4 ? w : next, (ks + 4) & 7);
            __builtin_amdgcn_sched_barrier(0x6);   // (what needs only the vector ALU may move up between the products)
        }
        w = next;
    };
    auto multiply = [&](int buf, i32x16 (&c)[RB]) __attribute__((always_inline)) { multiply_then(buf, c, w + EGG_SLAB / 16); };
    auto clear = [&](i32x16 (&c)[RB]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) c[b][e] = 0;
    };
    // (four blocks: their epilogues one after the other, or their temporaries spill)
    auto one_block = [&]() __attribute__((always_inline)) { if constexpr (RB > 3) __builtin_amdgcn_sched_barrier(0); };
    auto store_act = [&](int buf, int b, const u32x4& v) __attribute__((always_inline)) {
        int at = wr + buf;
        asm volatile("" : "+v"(at));
        *(u32x4*)(lds + b * 32 * EGG_D + at) = v;
    };
    auto put = [&](int t, int b, int part) __attribute__((always_inline)) {
        *(int*)(lds + t + b * 32 * TROW + tr + wave * 4) = halves_sum(part);   // (both halves store the same)
    };
    auto get = [&](int t, int b) __attribute__((always_inline)) {
        int sum = 0;
#pragma unroll
        for (int g = 0; g < WAVES / 4; ++g) {
            const i32x4 p = *(const i32x4*)(lds + t + b * 32 * TROW + tr + 16 * g);
            sum += (p[0] + p[1]) + (p[2] + p[3]);
        }
        return sum;
    };
    auto dot_of = [&](int t, int b) __attribute__((always_inline)) {
        const int d = get(t, b);
        return neg ? -d : d;
    };
    // four outputs of a block: I8((acc + (dot A >> cs)) >> os), the two shifts folded as in the streaming kernel
    // (clipped at -127 here, or, `raw`, saturated to [-128, 127]: what takes them apart into pairs clips a pair at a time)
    auto finish4 = [&](const i32x16& c, int q, uint32_t aw, int dot, int shift, bool raw) __attribute__((always_inline)) {
        const int low = -(127 << shift);
        int p[4];
        if constexpr (DOT24) {
            p[0] = mul24_word_byte<0>(dot, aw); p[1] = mul24_word_byte<1>(dot, aw); p[2] = mul24_word_byte<2>(dot, aw); p[3] = mul24_word_byte<3>(dot, aw);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = dot * (int)(int8_t)(aw >> (8 * e));
        }
        int t[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            t[e] = (int)((uint32_t)c[4 * q + e] << cs) + p[e];
            if (!raw) t[e] = max(t[e], low);
        }
        return ashr_pack4(t[0], t[1], t[2], t[3], shift);
    };
    // a row's |y| over this wave's columns
    u32x4 y[RB];
    auto put_abs = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            uint32_t s = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) s = abs_sum4(y[b][q], s);
            put(t_abs, b, (int)s);
        }
    };
    // u = LN(ln, y) of this lane's columns -> bufU; its dot products with up to two factor rows.  DIVIDE(x, mav) on floats: the factor
    // r = (1 + 2^-19) / mav, a few ulp either way, lifts every exact quotient above its integer, and the excess of the others stays below
    // 1 / mav up to 128, from where on the result is clipped.
    auto normalise = [&](const int8_t* ln, const u32x4 (&B0)[RB], const u32x4 (&B1)[RB], bool second) __attribute__((always_inline)) {
        const u32x4 lv = load16(ln, col);
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int mav = max(get(t_abs, b) >> 8, 1);
            const float r = __builtin_amdgcn_rcpf((float)mav) * 1.0000019073486328125f;
            int d0 = 0, d1 = 0;
            u32x4 u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t yw = y[b][q], lw = lv[q];
                int v[4] = {mul24_bytes<0>(yw, lw), mul24_bytes<1>(yw, lw), mul24_bytes<2>(yw, lw), mul24_bytes<3>(yw, lw)};
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = max((int)((float)v[e] * r), -127);
                u[q] = ashr_pack4(v[0], v[1], v[2], v[3], 0);
            }
            store_act(bufU, b, u);
            d0 += dot16(u, B0[b]);
            if (second) d1 += dot16(u, B1[b]);
            put(t_u0, b, d0);
            if (second) put(t_u1, b, d1);
        }
    };
    // this lane's pieces of a factor array: the address is formed where it is used (the pointers of a layer's twelve arrays, kept, spill)
    const int8_t* F = a.factors;
    const int64_t layer_bytes = 10 * a.fD + 2 * a.f4D;
    auto load_from = [&](const int8_t* f, u32x4 (&v)[RB]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < RB; ++b)
            v[b] = load16(f + (id0 + b * ids_block) * EGG_D, f_lane);
    };
    auto load_f = [&](int n_d, int n_4d, u32x4 (&v)[RB]) __attribute__((always_inline)) {   // behind n_d arrays of D and n_4d of 4 D values
        load_from(F + n_d * a.fD + n_4d * a.f4D, v);
    };

    u32x4 fa[RB], fb[RB], fc[RB];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) load_w(w, ks);
    for (int t = 0; t < a.T; ++t) {
        asm volatile("" : "+v"(n_row), "+v"(n_id), "+v"(f_lane));   // (as in the loop over layers)
        // y = I8(emb[token] + (A[token] (+-B) >> cs))
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int tok = (uint8_t)uniform((const int8_t*)a.tokens + (int64_t)t * a.rows + row0)[(uint32_t)min(32 * b + n_row, last)];
            int m = uniform(a.embA + (id0 + b * ids_block) * 256)[(uint32_t)(n_id * 256 + tok)];
            if (neg) m = -m;
            const u32x4 bv = load16(a.embB + (id0 + b * ids_block) * EGG_D, f_lane);
            const u32x4 ev = load16(a.emb, (uint32_t)(tok * EGG_D + col));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t o = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int v = (int)(int8_t)(ev[q] >> (8 * e)) + ((m * (int)(int8_t)(bv[q] >> (8 * e))) >> cs);
                    o |= (uint32_t)(min(127, max(-127, v)) & 0xFF) << (8 * e);
                }
                y[b][q] = o;
            }
        }
        put_abs();
        const int8_t* S_from = t == 0 ? a.S_in : a.S_out;
        for (int i = 0; i < a.L; ++i) {
            const int8_t* const S = S_from + ((int64_t)i * a.rows + row0) * EGG_D;
            const int8_t* const bias = a.bias + (int64_t)i * 2 * EGG_D;
            F = a.factors + i * layer_bytes;
            u32x4 s[RB];
            // what is derived from these is formed anew in every layer: kept over the loop, it takes registers that the accumulators need
            asm volatile("" : "+v"(n_row), "+v"(rd), "+v"(wr), "+v"(tr), "+v"(f_lane), "+v"(f_lane4));
            // ---- the state to LDS, s . B_Uf -----------------------------------------------------------------------------
#pragma unroll
            for (int b = 0; b < RB; ++b)
                s[b] = load16(S, row_at(b));
            load_f(3, 0, fb);
            load_f(1, 0, fa);
            load_f(5, 0, fc);
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                int d = 0;
                store_act(bufS, b, s[b]);
                d += dot16(s[b], fb[b]);
                put(t_s, b, d);
            }
            lds_phase();
            // ---- u = LN(ln1, y); s @ Uf -----------------------------------------------------------------------------------
            load_f(2, 0, fb);
            clear(acc);
            multiply(bufS, acc);
            normalise(a.ln1 + (int64_t)i * EGG_D, fa, fc, true);
            u32x4 a2[RB];
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const int d = dot_of(t_s, b);
#pragma unroll
                for (int q = 0; q < 4; ++q) a2[b][q] = finish4(acc[b], q, fb[b][q], d, sh, true);
                hold(a2[b]);
            }
            load_f(0, 0, fa);
            load_f(7, 0, fb);
            lds_phase();
            // ---- u @ Wf, first gate -> f^; u @ Wh -------------------------------------------------------------------------
            clear(acc);
            multiply(bufU, acc);
            u32x4 f[RB];     // f + 127
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const int d = dot_of(t_u0, b);
                int dh = 0;
                one_block();
                const u32x4 bv = load16(bias, col);
                u32x4 fh;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t a1 = finish4(acc[b], q, fa[b][q], d, sh, true), a2w = a2[b][q], sw = s[b][q];
                    const i16x2 k127 = {127, 127};
                    const i16x2 fe = sat127(clip(even_bytes(a1)) + clip(even_bytes(a2w)) + even_bytes(bv[q])) + k127;
                    const i16x2 fo = sat127(clip(odd_bytes(a1)) + clip(odd_bytes(a2w)) + odd_bytes(bv[q])) + k127;
                    // (f + 127) s: at most 254 x 127, inside 16 bits; its quotient needs no clipping
                    fh[q] = merge_bytes((fe * even_bytes(sw)) >> (short)8, (fo * odd_bytes(sw)) >> (short)8);
                    f[b][q] = merge_bytes(fe, fo);
                }
                store_act(bufF, b, fh);
                dh += dot16(fh, fb[b]);
                hold(s[b]);
                hold(f[b]);
                put(t_h, b, dh);
            }
            load_f(4, 0, fa);
            clear(acc);
            multiply(bufU, acc);
            load_f(6, 0, fb);
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const int d = dot_of(t_u1, b);
#pragma unroll
                for (int q = 0; q < 4; ++q) a2[b][q] = finish4(acc[b], q, fa[b][q], d, sh, true);
                hold(a2[b]);
            }
            lds_phase();
            // ---- f^ @ Uh, second gate -> the new state; y += it ------------------------------------------------------------
            clear(acc);
            multiply(bufF, acc);
            load_f(8, 1, fa);
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const int d = dot_of(t_h, b);
                one_block();
                const u32x4 bv = load16(bias + EGG_D, col);
                u32x4 hn;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t a4 = finish4(acc[b], q, fb[b][q], d, sh, true), a3 = a2[b][q], sw = s[b][q], fw = f[b][q];
                    const i16x2 de = sat127(clip(even_bytes(a3)) + clip(even_bytes(a4)) + even_bytes(bv[q])) - even_bytes(sw);
                    const i16x2 dd = sat127(clip(odd_bytes(a3)) + clip(odd_bytes(a4)) + odd_bytes(bv[q])) - odd_bytes(sw);
                    const int low = -(127 << 8);   // (f + 127)(h^ - s) takes 17 bits
                    const int p0 = max(mul24_ubyte_half<0>(fw, de), low), p1 = max(mul24_ubyte_half<1>(fw, dd), low);
                    const int p2 = max(mul24_ubyte_half<2>(fw, de), low), p3 = max(mul24_ubyte_half<3>(fw, dd), low);
                    hn[q] = add_sat4(sw, ashr_pack4(p0, p1, p2, p3, 8));
                    y[b][q] = add_sat4(y[b][q], hn[q]);
                }
                hold(y[b]);
                if (live(b)) store16_untracked((int8_t*)uniform(a.S_out + ((int64_t)i * a.rows + row0) * EGG_D) + row_at(b), hn);
            }
            put_abs();
            lds_phase();
            // ---- u = LN(ln2, y) -------------------------------------------------------------------------------------------
            normalise(a.ln2 + (int64_t)i * EGG_D, fa, fa, false);
            lds_phase();
            // ---- the MLP, its hidden row a quarter at a time: quarter c in bufS (even) or bufF, multiplied on behind the next barrier --
            int part[RB];
#pragma unroll
            for (int b = 0; b < RB; ++b) part[b] = 0;
            clear(acc2);
#pragma unroll 1
            for (int c = 0; c < 4; ++c) {
                const int8_t* const Aq = F + 8 * a.fD + c * EGG_D;
                const int8_t* const Bq = Aq + 2 * a.fD + a.f4D;
#pragma unroll
                for (int b = 0; b < RB; ++b) {
                    fa[b] = load16(Aq + (id0 + b * ids_block) * (4 * EGG_D), f_lane4);
                    fb[b] = load16(Bq + (id0 + b * ids_block) * (4 * EGG_D), f_lane4);
                }
                clear(acc);
                multiply(bufU, acc);
                const int dst = (c & 1) ? bufF : bufS;
#pragma unroll
                for (int b = 0; b < RB; ++b) {
                    const int d = dot_of(t_u0, b);
                    u32x4 hid;
#pragma unroll
                    for (int q = 0; q < 4; ++q) hid[q] = finish4(acc[b], q, fa[b][q], d, sh, false);
                    store_act(dst, b, hid);
                    part[b] += dot16(hid, fb[b]);
                }
                if (c > 0) multiply((c & 1) ? bufS : bufF, acc2);
                if (c == 3) {
#pragma unroll
                    for (int b = 0; b < RB; ++b) put(t_h, b, part[b]);
                    load_f(9, 1, fa);
                }
                lds_phase();
            }
            multiply(bufF, acc2);
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                const int d = dot_of(t_h, b);
#pragma unroll
                for (int q = 0; q < 4; ++q) y[b][q] = add_sat4(y[b][q], finish4(acc2[b], q, fa[b][q], d, sh + 1, false));
            }
            put_abs();
        }
        // ---- logits = LN(ln_out, y) @ head ----------------------------------------------------------------------------------
        load_from(a.headB, fb);
        load_from(a.headA, fa);
        lds_phase();
        normalise(a.ln_out, fb, fb, false);
        lds_phase();
        clear(acc);
        multiply_then(bufU, acc, w_first);
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int d = dot_of(t_u0, b);
            u32x4 o;
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = finish4(acc[b], q, fa[b][q], d, sh, false);
            if (live(b)) store16_untracked((int8_t*)uniform(a.logits + ((int64_t)t * a.rows + row0) * 256) + row_at(b), o);
        }
        lds_phase();   // t_abs, t_u0 and bufU are the next token's
    }
}

bool egg_fused_applies(int D, int int_bound, int corr_shift, int out_shift)
{
    // the folded shifts (see k_int8.hip) at both widths of a product, 256 and 1024
    const int sh = corr_shift + out_shift + 1;
    const int64_t nmax = noise_max(int_bound), d = 4 * EGG_D;
    return D == EGG_D && sh <= 23 && ((d * 127 * 127) << corr_shift) + d * 127 * nmax * nmax < (int64_t(1) << 31);
}

size_t egg_fused_weight_bytes(int L) { return (size_t)(EGG_LAYER_SLABS * L + 1) * EGG_SLAB; }

template <int RB>
static egg_status launch_layers(eggroll_ctx* c, const EggFusedArgs& a, bool dot24)
{
    auto kern = dot24 ? egg_layers_kernel<RB, true> : egg_layers_kernel<RB, false>;
    constexpr size_t lds = 3 * 32 * RB * EGG_D + 5 * 32 * RB * 8 * sizeof(int);
    const egg_status st = ensure_dynamic_lds(c, (const void*)kern, lds, "integer model smem attr");
    if (st != EGG_OK) return st;
    KernelScope ks(c, "egg_layers_i8");
    hipLaunchKernelGGL(kern, dim3((unsigned)((a.rows + 32 * RB - 1) / (32 * RB))), dim3(512), lds, c->stream, a);
    return check_hip(c, hipGetLastError(), "integer model launch");
}

egg_status launch_egg_fused(eggroll_ctx* c, const EggFusedModel& m, int int_bound, const egg_model_i8& P)
{
    EggFusedArgs a{};
    a.w = (const u32x4*)m.weights;
    a.emb = P.emb; a.ln1 = P.ln1; a.ln2 = P.ln2; a.ln_out = P.ln_out; a.bias = P.gru_b;
    a.embA = m.embA; a.embB = m.embB; a.headA = m.headA; a.headB = m.headB; a.factors = m.factors;
    a.fD = m.fD; a.f4D = m.f4D;
    a.tokens = m.tokens; a.S_in = m.S_in; a.S_out = m.S_out; a.logits = m.logits;
    a.rows = m.rows; a.L = m.L; a.T = m.T; a.anti = m.anti; a.corr_shift = m.corr_shift; a.out_shift = m.out_shift;
    const int slabs = EGG_LAYER_SLABS * m.L + 1;
    {
        KernelScope ks(c, "egg_lay_weights");
        hipLaunchKernelGGL(egg_lay_weights_kernel, dim3((unsigned)(slabs * 16)), dim3(256), 0, c->stream, P.gru_w, P.mlp1, P.mlp2, P.head, m.L, (u32x4*)m.weights);
        const egg_status st = check_hip(c, hipGetLastError(), "integer model weights launch");
        if (st != EGG_OK) return st;
    }
    const bool dot24 = (int64_t)4 * EGG_D * 127 * noise_max(int_bound) < (int64_t(1) << 23);
    // Rows of a workgroup: what a CU's share of the workgroups takes, by the measured us per layer and token -- 32 rows 17, and 30 for the
    // two of them that fit on a CU together; 96 rows 34; 128 rows 47.  (Whole calls, us, with 32 / 96 / 128 rows: 3470 members, 5
    // layers, 4 tokens 418 / 754 / 914; 18804, 3, 3 531 / 489 / 563; 32768, 6, 4 1899 / 2224 / 1700.  64 rows were never the best.)
    auto per_cu = [&](int rows) { return (m.rows + rows * (int64_t)c->compute_units - 1) / (rows * (int64_t)c->compute_units); };
    const int64_t p1 = per_cu(32), t1 = p1 / 2 * 30 + p1 % 2 * 17, t3 = per_cu(96) * 34, t4 = per_cu(128) * 47;
    if (t1 <= t3 && t1 <= t4) return launch_layers<1>(c, a, dot24);
    return t3 <= t4 ? launch_layers<3>(c, a, dot24) : launch_layers<4>(c, a, dot24);
}

}  // namespace egg
