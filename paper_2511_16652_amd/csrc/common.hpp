// Host-side plumbing shared by the translation units of libeggroll: the context (stream, scratch,
// error text, optional per-kernel event timing) and launch helpers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <map>
#include <string>
#include <vector>

#include "../../include/eggroll.h"
#include "rng.hpp"

struct eggroll_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string err;
    int compute_units = 256;  // of the device (grid size of persistent kernels)
    int cache_layout = 0;  // egg_cache_layout of the forward/update caches
    bool conservative_waits = false;  // diagnostic: the kernels that count their loads in flight wait for everything instead

    // scratch, grown on demand and kept for the life of the context
    struct Buf {
        void* p = nullptr;
        size_t bytes = 0;
    };
    Buf t_buf;        // projections t[R][r] fp32 (forward) / int32 dots (int8 path)
    Buf a_buf, b_buf; // materialised [member][d][r] factors when the caller keeps no cache
    Buf fnorm;        // update: power-of-two normaliser of the fitness vector
    Buf pack_a;       // update: K-packed diag(f)A panel
    Buf pack_b;       // update: K-packed B panel
    Buf i8_a, i8_b;   // int8 path: factors, generated once per episode
    Buf i8_h;         // int8 path: ping-pong state
    Buf gru;          // integer GRU cell: factors of its four matrices, gate and matmul intermediates
    Buf zero_page;    // 256 zero bytes (K-tail loads of the GEMM core)
    Buf lut;          // integer log-likelihood: EXP2 table and the thresholds that invert LOG2
    Buf norm_tab;     // integer normal noise: the 65536-entry table round(16 z) (uploaded on first use)
    Buf model;        // multi-layer drivers: activations of one chunk of members
    Buf model_g;      // multi-layer updates: fp32 G of the matrix being updated
    Buf proj_part;    // fused next-layer projection: per (128-row slab of d_out, row) partial sums
    Buf next_b;       // fused next-layer projection through the C ABI: the next layer's factors B'[member][d_out]
    // buffers that a later, larger call outgrew: kept until eggroll_trim / eggroll_destroy, because work already
    // enqueued -- or a HIP graph captured earlier -- may still hold their addresses
    std::vector<Buf> retired;
    uint64_t scratch_generation = 0;  // bumped whenever a scratch buffer is replaced

    // profiling
    bool prof = false;
    struct Rec {
        const char* name;
        hipEvent_t a, b;
    };
    std::vector<Rec> recs;
    std::vector<hipEvent_t> free_events;
    std::map<std::string, int> shaped_names;  // interned "kernel[d_out x d_in]" labels (node addresses are stable)
};

namespace egg {

// sum over the 16 lanes of a DPP row, left in every lane of the row
__device__ __forceinline__ float row_sum16(float x)
{
#define EGG_DPP_ADD(CTRL) x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
    EGG_DPP_ADD(0xB1)   // quad_perm [1, 0, 3, 2]
    EGG_DPP_ADD(0x4E)   // quad_perm [2, 3, 0, 1]
    EGG_DPP_ADD(0x141)  // row_half_mirror: the other quad of the half row
    EGG_DPP_ADD(0x140)  // row_mirror: the other half row
#undef EGG_DPP_ADD
    return x;
}

// sum over the wave, left in every lane: lanes 32 apart first, then 16, 8, 4, 2, 1 -- the order, and so the bits, of a butterfly of
// shuffles, each of which is an LDS round trip (a row of rank 8 takes 48 of them); the swaps and DPP forms stay in the vector ALU
__device__ __forceinline__ float wave_sum(float x)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    u32x2 p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
#define EGG_DPP_ADD(CTRL) x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
    EGG_DPP_ADD(0x128)  // row_ror:8
    EGG_DPP_ADD(0x124)  // row_ror:4 (lanes 8 apart agree: the lane 4 away in either direction)
    EGG_DPP_ADD(0x4E)   // quad_perm [2, 3, 0, 1]
    EGG_DPP_ADD(0xB1)   // quad_perm [1, 0, 3, 2]
#undef EGG_DPP_ADD
    return x;
}

egg_status fail(eggroll_ctx* c, egg_status s, const char* fmt, ...);
egg_status check_hip(eggroll_ctx* c, hipError_t e, const char* what);
egg_status reserve(eggroll_ctx* c, eggroll_ctx::Buf& b, size_t bytes);
// scratch that a call is faster with and can do without: false where there is no memory for it, or a capture, which an allocation would
// end, is under way
bool try_reserve(eggroll_ctx* c, eggroll_ctx::Buf& b, size_t bytes);

// RAII bracket: records events around one kernel launch when profiling is on
struct KernelScope {
    eggroll_ctx* c;
    const char* name;
    hipEvent_t a = nullptr, b = nullptr;
    KernelScope(eggroll_ctx* ctx, const char* n);
    ~KernelScope();
};

// A kernel that needs more than the default dynamic LDS must have its limit raised; this does it on first use (and again
// only if a later launch needs more), instead of on every launch.  The limit belongs to the function, not to a context:
// the bookkeeping is process-wide (per device).
egg_status ensure_dynamic_lds(eggroll_ctx* c, const void* kern, size_t bytes, const char* what);

// label of a per-shape timing row, e.g. forward_gemm_bf16[8192x2048]; only built when profiling is on
inline const char* shaped_name(eggroll_ctx* c, const char* base, int d_out, int d_in)
{
    if (!c->prof) return base;
    char buf[96];
    snprintf(buf, sizeof buf, "%s[%dx%d]", base, d_out, d_in);
    return c->shaped_names.emplace(buf, 0).first->first.c_str();
}

// int_bound arguments: a bound in [0, 127] (uniform integers) or EGG_INT_NOISE_NORMAL16 (the table of round(16 z))
inline bool valid_int_bound(int b) { return (b >= 0 && b <= 127) || b == EGG_INT_NOISE_NORMAL16; }
// largest |value| the selected integer noise can take: 16 * Phi^-1(1 - 2^-17) rounds to 69 for the table
inline int noise_max(int b) { return b == EGG_INT_NOISE_NORMAL16 ? 69 : b; }
void normal_int_table(int8_t* out);  // host: fills the 65536 entries

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

egg_status validate_shape(eggroll_ctx* c, const egg_shape* s, bool need_rows, bool forward_pass);

// entry points implemented per translation unit (kernel launchers)
egg_status launch_noise(eggroll_ctx* c, const StreamKey& k, uint32_t member_begin, int64_t members, int64_t n,
                        egg_dtype dtype, egg_dist dist, int int_bound, void* out);
egg_status ensure_normal_table(eggroll_ctx* c);  // c->norm_tab holds the table of round(16 z)
// several vectors of the same members and type (the factors of a layer's matrices): one launch for those made of whole
// 16-byte pieces, of up to 20 vectors
struct NoiseJob {
    StreamKey key;
    int64_t n;  // values per member
    void* out;
};
egg_status launch_noise_jobs(eggroll_ctx* c, const NoiseJob* jobs, int count, uint32_t member_begin, int64_t members, egg_dtype dtype,
                             egg_dist dist, int int_bound);
// normals that another kernel draws along with its own work: false where the vectors are not made of whole 16-byte pieces
bool normal_pieces(const NoiseJob& job, int64_t members, egg_dtype dtype, NoisePiece& out);
// How the rows of a member (of a pair) are shared among workgroups of the projection pass: `parts` of `rows` each.  ready: B_cache holds
// the factors already (otherwise every workgroup draws its member's, and fills B_cache if there is one).
struct ProjectSplit {
    int parts, rows;
    bool ready;
};
ProjectSplit project_split(const eggroll_ctx* c, const egg_shape& s, egg_dtype io, bool ready);
egg_status launch_project(eggroll_ctx* c, const StreamKey& kb, const egg_shape& s, egg_dtype io, const void* X,
                          float* t, void* B_cache, bool panel, const ProjectSplit& split, const NoisePiece* along = nullptr);
// the projection pass can draw these vectors as well, in workgroups of its own
bool project_draws_along(const eggroll_ctx* c, const egg_shape& s, egg_dtype io, const ProjectSplit& split, const NoisePiece& along);
// A layer whose output feeds the next perturbed layer directly (up-projection -> down-projection) can form that
// layer's projections (same rank, 1, 2 or 4) in its own epilogue, from the bf16 values it stores: B = the next layer's
// factors [member][d_out][rank] bf16, t = where the projections [rows][rank] go.  Supported where
// forward_fuses_next_projection says so.
struct NextProjection {
    const void* B;
    float* t;
};
// one row per member at rank 1 (a kept cache of pairs apart): the epilogue draws the factors A itself
inline bool forward_regenerates(const egg_shape& s, float sigma, const void* A_cache)
{
    return sigma == 0.f || (s.rank == 1 && s.rows_per_member == 1 && !(s.antithetic && A_cache));
}
bool forward_fuses_next_projection(const egg_shape& s, egg_dtype io, egg_dtype yd, float sigma, egg_act act, bool resid);
// regenerate: forward_regenerates of the call (A_cache may since have become A_ready); A_ready: the factors A that eggroll_noise_gen would write for
// this layer, already drawn by the caller (NULL: drawn here)
egg_status launch_forward_gemm(eggroll_ctx* c, const StreamKey& ka, const egg_shape& s, egg_dtype io, egg_dtype yd,
                               float sigma, egg_act act, const void* W, const void* X, void* Y, const float* t,
                               bool regenerate, void* A_cache, const void* resid, const NextProjection* next, const void* A_ready);
egg_status launch_update(eggroll_ctx* c, const StreamKey& ka, const StreamKey& kb, const egg_shape& s,
                         egg_dtype noise_dtype, const float* fitness, float scale, int accumulate, float* G, void* W,
                         egg_dtype w_dtype, float lr, const void* A_cache, const void* B_cache, bool b_panel);
egg_status forward_linear(eggroll_ctx* c, egg_key key, const egg_shape& shape, egg_dtype io_dtype, egg_dtype y_dtype, float sigma,
                          egg_act act, const void* W, const void* X, void* Y, void* A_cache, void* B_cache, const void* resid,
                          float* t_fixed = nullptr, const float* t_ready = nullptr, const NextProjection* next = nullptr,
                          const void* A_ready = nullptr);
egg_status checked_forward(eggroll_ctx* c, egg_key key, const egg_shape* shape, egg_dtype io_dtype, egg_dtype y_dtype,
                           float sigma, egg_act act, const void* W, const void* X, const void* R_in, bool need_r, void* Y,
                           void* A_cache, void* B_cache, float* t_fixed, size_t t_capacity, const float* t_in = nullptr,
                           bool want_next = false, uint32_t next_layer = 0, float* t_next = nullptr);
// unperturbed glue of the decoder workload
egg_status launch_embed_rows(eggroll_ctx* c, int64_t rows, int d, int vocab, const void* emb, const int32_t* tokens, void* X);
egg_status launch_rmsnorm(eggroll_ctx* c, int64_t rows, int d, float eps, const void* gain, const void* X, void* Y);
egg_status launch_rmsnorm_proj(eggroll_ctx* c, int64_t rows, int S, int d, float eps, const void* gain, const void* X, void* Y, int nc,
                               const void* const* B, float* const* t);
// Bo != NULL: also t_next[row] = sum_j O[row][j] * Bo[member][j] (Bo: [members][heads * head_dim] bf16, rank-1 factors of the
// layer that reads O)
egg_status launch_attention(eggroll_ctx* c, int64_t members, int S, int heads, int head_dim, const void* Q, const void* K,
                            const void* V, void* O, const void* Bo = nullptr, float* t_next = nullptr);
// t[n] = sum over slabs p of part[p][n], in slab order
egg_status launch_sum_slabs(eggroll_ctx* c, const float* part, int slabs, int64_t R, float* t);
egg_status launch_token_loglik(eggroll_ctx* c, int64_t members, int S, int vocab, const void* logits, const int32_t* tokens, float* out);
// multi-layer drivers
egg_status launch_mlp_stack_forward(eggroll_ctx* c, egg_key key, const egg_shape& s, int L, int d_ff, float sigma,
                                    const void* W1, const void* W2, const void* X, void* Y, int64_t chunk_members);
egg_status launch_mlp_stack_update(eggroll_ctx* c, egg_key key, const egg_shape& s, int L, int d_ff, const float* fitness,
                                   float scale, float lr, void* W1, void* W2);
egg_status launch_decoder_forward(eggroll_ctx* c, egg_key key, const egg_shape& s, const egg_decoder_cfg& cfg,
                                  const egg_decoder_weights& w, float sigma, const int32_t* tokens, void* logits, float* loglik,
                                  int64_t chunk_members);
egg_status launch_decoder_update(eggroll_ctx* c, egg_key key, const egg_shape& s, const egg_decoder_cfg& cfg, const float* fitness,
                                 float scale, float lr, const egg_decoder_weights& w);
egg_status launch_forward_i8(eggroll_ctx* c, const StreamKey& ka, const StreamKey& kb, const egg_shape& s,
                             int int_bound, int corr_shift, int out_shift, int steps, const int8_t* W,
                             const int8_t* H_in, int8_t* H_out);

// many time steps in one kernel (k_recur_i8.hip), for the shapes that recur_i8_applies accepts
bool recur_i8_applies(int d_out, int d_in, int64_t rows, int steps, int compute_units);
egg_status launch_recur_i8(eggroll_ctx* c, const int8_t* A, const int8_t* B, int anti, int64_t rows, int d, int int_bound, int corr_shift,
                           int out_shift, int steps, const int8_t* W, const int8_t* H_in, int8_t* H_out);

// GRU gating fused into the epilogue of an integer matmul (see I8Args in k_int8.hip)
struct I8Gate {
    int mode;  // 1: f and f^,  2: h
    const int8_t *other, *state, *f, *bias;
    int8_t* out2;
};
egg_status launch_i8_matmul(eggroll_ctx* c, const int8_t* A, const int8_t* B, int anti, int64_t rows, int d_out, int d_in,
                            int int_bound, int corr_shift, int out_shift, const int8_t* W, const int8_t* src, int8_t* dst,
                            int* dots, bool dots_ready, const I8Gate* gate, const int8_t* B_next = nullptr, int* dots_next = nullptr);
egg_status launch_zero_i32(eggroll_ctx* c, int* p0, int* p1, int64_t n);  // clears one or two int32 vectors (p1 may be NULL)
egg_status launch_dots_i8(eggroll_ctx* c, const int8_t* X0, const int8_t* B0, const int8_t* B1, const int8_t* X1, const int8_t* B2,
                          int64_t rows, int d, int anti, int* d0, int* d1, int* d2);
// factors, weights and intermediates of one GRU cell (matrix order: Wf, Uf, Wh, Uh)
struct GruStep {
    const int8_t *A[4], *B[4], *W[4];
    const int8_t *bf, *bh;
    int8_t *a1, *a3, *f, *fh;  // [rows][D] each
    int* dot[4];               // [rows] each: u.B_Wf, s.B_Uf, u.B_Wh, f^.B_Uh
    bool u_dots_ready = false; // dot[0] and dot[2] were filled by whoever produced u
    bool s_dot_ready = false;  // dot[1] was filled by the previous step's last epilogue
    bool fh_dot_zeroed = false;// dot[3] is zero: the first gate's epilogue accumulates f^.B_Uh there
    int* dot_s_next = nullptr; // zeroed [rows]: the last epilogue accumulates h.B_Uf for the next step there
};
egg_status launch_gru_step(eggroll_ctx* c, const GruStep& g, int anti, int64_t rows, int D, int int_bound, int corr_shift,
                           int out_shift, const int8_t* u, const int8_t* state, int8_t* next);
egg_status launch_gru_i8(eggroll_ctx* c, egg_key key, const egg_shape& s, int int_bound, int corr_shift, int out_shift,
                         int steps, const int8_t* const W[4], const int8_t* bf, const int8_t* bh, const int8_t* U,
                         const int8_t* S_in, int8_t* S_out);
// optional by-products of the normalisation pass: dot products of the normalised rows with up to two factor
// arrays (what the matmuls that consume u need), and up to two int32 vectors cleared for later accumulation
struct LnExtras {
    const int8_t* B[2] = {nullptr, nullptr};  // [ids][D]
    int* dot[2] = {nullptr, nullptr};         // [rows]
    int* zero[2] = {nullptr, nullptr};        // [rows]
    int anti = 0;
};
egg_status launch_layernorm_i8(eggroll_ctx* c, const int8_t* add, int8_t* y, const int8_t* ln, int8_t* u, int64_t rows, int D,
                               const LnExtras* extras = nullptr);
egg_status launch_embed_i8(eggroll_ctx* c, egg_key key, const egg_shape& s, int int_bound, int corr_shift, const int8_t* emb,
                           const uint8_t* tokens, int8_t* Y);
egg_status launch_egg_forward_i8(eggroll_ctx* c, egg_key key, const egg_shape& s, int L, int int_bound, int corr_shift, int T,
                                 const egg_model_i8& P, const uint8_t* tokens, const int8_t* S_in, int8_t* S_out,
                                 int8_t* logits);
// the whole forward pass in one kernel at D = 256 (k_egg_fused.hip); factors: per layer A and B of Wf, Uf, Wh, Uh, then A1, B1, A2, B2,
// fD bytes an array of D values per id and f4D one of 4 D
struct EggFusedModel {
    const int8_t *embA, *embB, *headA, *headB, *factors;
    int64_t fD, f4D;
    int8_t* weights;  // scratch, egg_fused_weight_bytes(L)
    const uint8_t* tokens;
    const int8_t* S_in;
    int8_t *S_out, *logits;
    int64_t rows;
    int L, T, anti, corr_shift, out_shift;
};
bool egg_fused_applies(int D, int int_bound, int corr_shift, int out_shift);
size_t egg_fused_weight_bytes(int L);
egg_status launch_egg_fused(eggroll_ctx* c, const EggFusedModel& m, int int_bound, const egg_model_i8& P);
egg_status launch_loglik_i8(eggroll_ctx* c, int64_t rows, const int8_t* logits, const uint8_t* targets, int accumulate, int32_t* out);
// integer updates of several matrices of one population
struct I8UpdateJob {
    StreamKey ka, kb;
    int d_out, d_in;
    int8_t* theta;
    int32_t* E_out;  // optional
};
egg_status launch_update_i8_jobs(eggroll_ctx* c, const I8UpdateJob* jobs, int count, uint32_t member_begin, int64_t N, int int_bound,
                                 const int8_t* F, int32_t threshold);

}  // namespace egg
