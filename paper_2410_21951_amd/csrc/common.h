// Internal declarations shared by the HIP translation units of libvadusa.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <string>
#include <tuple>
#include <type_traits>
#include <utility>
#include <vector>

#include "vadusa.h"

typedef uint16_t bf16_t;   // raw bfloat16 bits

#define MASK_WORDS (VADUSA_MAX_TREE_NODES / 32)
#define LN_EPS 1e-5f

__device__ __forceinline__ float bf2f(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }
__device__ __forceinline__ bf16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest, ties to even
    return (bf16_t)(u >> 16);
}
__device__ __forceinline__ float ldf(const float* p) { return *p; }
__device__ __forceinline__ float ldf(const bf16_t* p) { return bf2f(*p); }
__device__ __forceinline__ void stf(float* p, float v) { *p = v; }
__device__ __forceinline__ void stf(bf16_t* p, float v) { *p = f2bf(v); }

// Every pointer the kernels dereference points into device (global) memory.  A pointer read from
// memory is a generic pointer to the compiler and would be accessed with FLAT instructions (slower
// to issue, and tied to the LDS counter as well); the helpers below state the address space.
#if defined(__HIP_DEVICE_COMPILE__)
#define VADUSA_GLOBAL __attribute__((address_space(1)))
#else
#define VADUSA_GLOBAL
#endif
template <class T>
__device__ __forceinline__ T ldg(const T* p) { return *(const VADUSA_GLOBAL T*)p; }   // scalar T only
// 8- and 16-byte loads (HIP's uint2 / uint4 / float2 are classes: their copy would go back to a generic reference)
typedef uint32_t vadusa_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t vadusa_u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint4 ldg4(const void* p) {
    const vadusa_u32x4 v = *(const VADUSA_GLOBAL vadusa_u32x4*)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint2 ldg2(const void* p) {
    const vadusa_u32x2 v = *(const VADUSA_GLOBAL vadusa_u32x2*)p;
    return make_uint2(v.x, v.y);
}

// Stores / loads that are coherent across the whole GPU without cache maintenance
// (write-through to / read from the memory side), for values that a workgroup reads back through memory.
__device__ __forceinline__ void stw32(void* p, uint32_t v) {
    __hip_atomic_store((VADUSA_GLOBAL uint32_t*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void stwi(int32_t* p, int32_t v) { stw32(p, (uint32_t)v); }
__device__ __forceinline__ int32_t ldci(const int32_t* p) {
    return __hip_atomic_load((const VADUSA_GLOBAL int32_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Offset of element (r, k) of a bf16 activation matrix kept in MFMA-operand tiles:
// [row tile of 16][k-step of 32][lane = (r & 15) + 16 * ((k & 31) >> 3)][k & 7], nks = K / 32.
// A wave reads one (row tile, k-step) as the A operand with one contiguous KiB load.
__device__ __forceinline__ size_t toff(int r, int k, int nks) {
    return ((size_t)((r >> 4) * nks + (k >> 5)) * 64 + (r & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}
// KV cache of one (layer, sequence, head): kv_cap(max_positions) positions (whole blocks of 32) x 64 dimensions,
// kept in the operand tiles of the attention, so that every operand of a 32-key block is one contiguous KiB
// per wave load (a row-major cache makes such a load touch 16 cache lines and use half of each):
//   K: [block of 32 keys][key tile t][k-step s][lane][8]: key k = pos & 31 sits in tile t = (k >> 2) & 1 (tile 0:
//      keys 0-3, 8-11, 16-19, 24-27 of the block; tile 1: the others) at row c = ((k >> 3) << 2) | (k & 3); k-step
//      s = dim >> 5; lane = c + 16 * ((dim & 31) >> 3).  (With this row order the lane that holds query c's scores
//      after S^T = K Q^T holds them for eight consecutive keys: exactly a B fragment of P^T for O^T += V^T P^T.)
//   V: [block of 32 keys][dimension tile dt = dim >> 4][lane][8]: lane = (dim & 15) + 16 * ((pos & 31) >> 3),
//      element pos & 7 (V transposed: a lane holds eight consecutive positions of one dimension).
__host__ __device__ inline int cdiv(int a, int b) { return (a + b - 1) / b; }
__host__ __device__ inline int kv_cap(int maxpos) { return (maxpos + 31) & ~31; }
__host__ __device__ inline size_t kc_off(int pos, int dim) {
    const int k = pos & 31, t = (k >> 2) & 1, c = ((k >> 3) << 2) | (k & 3);
    return (size_t)(pos >> 5) * 2048 + (size_t)(((t * 2 + (dim >> 5)) * 64 + c + 16 * ((dim & 31) >> 3)) * 8 + (dim & 7));
}
__host__ __device__ inline size_t vc_off(int pos, int dim) {
    return (size_t)(pos >> 5) * 2048 + (size_t)((((dim >> 4) * 64) + (dim & 15) + 16 * ((pos & 31) >> 3)) * 8 + (pos & 7));
}
// Two floats to a pair of bf16 (round to nearest even): one v_cvt_pk_bf16_f32 on the device.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    typedef __attribute__((ext_vector_type(2))) float f32x2_cvt;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_cvt;
    const f32x2_cvt v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_cvt));
}

// GELU with the exact (erf) definition, v Phi(v); erfc by the rational approximation 7.1.26 of Abramowitz &
// Stegun (absolute error below 1.5e-7, the size of an fp32 rounding of the result, which is then
// stored as bf16): one exponential, one reciprocal and a fifth-degree polynomial instead of the
// library routine's two branches.  Its constants are scaled for |v| in place of |v| / sqrt 2, powers of two and erfc / 2 = Phi(-|v|).
__device__ __forceinline__ float gelu_s(float v) {
    const float t = __builtin_amdgcn_rcpf(1.f + 0.23164190f * fabsf(v));   // one instruction, 1 ulp: far below the approximation's own error
    const float poly = t * (0.127414796f + t * (-0.142248368f + t * (0.7107068705f + t * (-0.7265760135f + t * 0.5307027145f))));
    const float u = v * 0.84932180f;                                        // 2^-(u u) = exp(-v^2 / 2)
    const float tail = poly * __builtin_amdgcn_exp2f(-(u * u));
    return v * (v < 0.f ? tail : 1.f - tail);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// The same sums without LDS traffic: DPP lane permutations inside each row of 16 lanes (swap
// with the quad neighbour, the other pair of the quad, the mirrored half row, the mirrored row:
// after each step twice as many lanes hold the same partial sum), then the four row sums are
// read from lanes 0, 16, 32 and 48.  Every lane returns the total; all 64 lanes must be active.
template <int CTRL>
__device__ __forceinline__ int dpp_perm(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false); }
// sums over the 4 lanes of a quad and over the 16 lanes of a row; every lane gets the total.  The
// additions pair the same values as an xor-butterfly of __shfl_xor would, so the results are the same bits.
__device__ __forceinline__ float quad_sum(float v) {
    v += __int_as_float(dpp_perm<0xB1>(__float_as_int(v)));
    v += __int_as_float(dpp_perm<0x4E>(__float_as_int(v)));
    return v;
}
__device__ __forceinline__ float row16_sum(float v) {
    v = quad_sum(v);
    v += __int_as_float(dpp_perm<0x141>(__float_as_int(v)));
    v += __int_as_float(dpp_perm<0x140>(__float_as_int(v)));
    return v;
}
// Combining a value with the ones 16 and 32 lanes away (the four rows of a wave), every lane gets
// the result.  gfx950 swaps rows between two registers in the vector ALU: with both operands the
// same value, one register then holds rows {0, 0, 2, 2} and the other rows {1, 1, 3, 3} (16-lane
// swap), or halves {lo, lo} and {hi, hi} (32-lane swap), and combining the two registers lane by
// lane is the exchange, without a trip through the LDS permute unit.
typedef unsigned int vadusa_u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float rows_max(float v) {
    vadusa_u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}
__device__ __forceinline__ float rows_sum(float v) {
    vadusa_u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(r.x) + __uint_as_float(r.y);
    r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);
}
// Sum over the two lanes l and l ^ 32.
__device__ __forceinline__ float half_sum(float v) {
    const vadusa_u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r.x) + __uint_as_float(r.y);
}

__device__ __forceinline__ int wave_sum_i_dpp(int v) {
    v += dpp_perm<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_perm<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_perm<0x141>(v);   // row_half_mirror
    v += dpp_perm<0x140>(v);   // row_mirror
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) +
           __builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48);
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
    v += __int_as_float(dpp_perm<0xB1>(__float_as_int(v)));
    v += __int_as_float(dpp_perm<0x4E>(__float_as_int(v)));
    v += __int_as_float(dpp_perm<0x141>(__float_as_int(v)));
    v += __int_as_float(dpp_perm<0x140>(__float_as_int(v)));
    return (__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0)) +
            __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16))) +
           (__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32)) +
            __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48)));
}

// Shapes that every kernel needs (passed by value).
struct Dims {
    int Ly, d, nH, F, V1, Hh, maxpos, Bmax, Mmax;   // model / capacity
    int B, M;                                        // current batch; rows per sequence (a ragged prompt pass: of the longest)
    int R;                                           // rows of the forward: B * M, or the rows that a ragged prompt pass has
    int last_only;                                   // the vocabulary map's rows are the sequences' last rows, one behind the other (else all rows)
    int keys;                                        // no sequence attends to more keys than this (for the choice of kernels)
};

// Pointers to one layer's parameters on the device.
struct LayerW {
    const float *ln1_g, *ln1_b, *bqkv, *bo, *ln2_g, *ln2_b, *b1, *b2;
    const void *Wqkv, *Wo, *W1, *W2;   // element type follows the context dtype
    // bf16 model only: LayerNorm folded into the following linear map (see k_layer.hip)
    float *cs_qkv, *t_qkv, *cs_w1, *t_w1;
};
struct DraftW {
    const void* W1; const float* b1; const void* W2;
};

// Decoding state and scratch on the device (all inside the caller's arena).
struct DevState {
    // model
    const void *E_text, *E_speech, *P;
    const float *lnf_g, *lnf_b;
    const void* W_out;
    float *cs_out, *t_out;          // bf16 model: folded final LayerNorm for the vocabulary map
    // KV cache, element type = dtype: [Ly][Bmax][nH] times kv_cap(maxpos) positions x 64 dimensions in the order of kc_off / vc_off
    void *Kc, *Vc;
    // activations
    float* x;        // [R][d]  residual stream
    bf16_t* xb;      // bf16 model: [R][d] copy of the residual stream, operand tiles (rows padded to a multiple of 16)
    float* stats;    // bf16 model: [R][groups][2] per group of 16, 32 or 64 columns: mean, sum of squared deviations
    size_t draft_stride;   // elements from one draft head's rdraft to the next
    int32_t* kerr;   // [4] error flag that the next synchronising call reports
    long long* tprof; // [128][8] timing points (device clock, 100 MHz; -DVADUSA_CLOCK_BUILD)
    void* q;         // [R][d]
    void* att;       // [R][d]
    void* hid;       // [R][F]
    void* hn;        // [rows of a step][d]  final-LayerNorm'd node states (inspection)
    float* logits;   // [R][V1]
    void* hbest;     // [Bmax][d]
    void* rdraft;    // [Hh][Bmax][d]
    float* zdraft;   // [Bmax][Hh][V1]
    // integer state
    int32_t *L, *root, *finished, *draft_topk /*[Bmax][Hh][MAX_TOPK]*/;
    int32_t *tok /*[R]*/, *n_rows /*[Bmax]*/, *edge_ok /*[R]*/, *path /*[Bmax][MAX_DRAFT_HEADS+2]*/;
    int32_t *out_tok /*[Bmax][maxpos]*/, *n_out /*[Bmax]*/;
    int32_t *acc_tok /*[Bmax][MAX_DRAFT_HEADS+1]*/, *acc_len /*[Bmax]*/;
    int32_t *chunk_tok /*[R]*/;
    int32_t *row_seq /*[R]*/, *row0 /*[Bmax]*/;   // ragged prompt pass: each row's sequence, each sequence's first row (null: sequence b has rows b * M ..)
    int32_t *pass_tables;  // where vadusa_prefill puts n_rows, row0, chunk_tok and row_seq of all its passes
    int32_t *override_topk /*[Bmax][Hh][MAX_TOPK]*/;
    // tree tables (index 0: current tree, 1: causal chunk used by prefill)
    int32_t *t_parent[2], *t_depth[2], *t_rank[2];
    uint32_t* t_mask[2];   // [Mmax][MASK_WORDS]
    float* staging;        // floats on their way in (weights) or out (readers)
};

struct vadusa_ctx {
    vadusa_config cfg;
    hipStream_t stream;
    char* arena;
    size_t arena_bytes;
    DevState s;
    std::vector<LayerW> layers;
    std::vector<DraftW> draft;
    size_t elem;                 // bytes per stored element (4 or 2)
    int state;                   // 0 created, 1 weights loaded, 2 ready, 3 verification pending
    int batch;                   // current batch
    int M;                       // nodes of the pending / last verification
    std::vector<int32_t> L_ub;   // host upper bound of each sequence's committed length
    std::vector<char> pending;   // per sequence: verification waits for compaction
    std::vector<int32_t> tree_parent, tree_rank, tree_depth;   // last uploaded tree
    size_t staging_floats;
    float* uniforms;             // [max_batch * max_tree_nodes][V+1]: the caller's random numbers of a stochastic step
    float* scores;               // same shape: perturbed scores that replace the logits in such a step
    int sampled;                 // the pending / last verification was a stochastic one
    int big_min;                 // k_big's tiles, and attention workgroups of two query tiles, from this many on; -1, below -1: k_tile of 256 x 128, 128 x 64 outputs for every
                                 // map (environment VADUSA_BIG_MIN_UNITS, for tests of small shapes); 0: the rules
    int32_t* pinned;             // host memory that the last kernel of a call writes results into (null: none)
    size_t pinned_words;
    std::vector<int32_t> unpinned;   // its stand-in
    int errored;                 // the error word was raised: every call but vadusa_prefill refuses until that resets the context
    std::string err;
};

// Launches a kernel and keeps the first failure of this thread until launched() or fail() in api.hip takes it.  The launch's
// own status and not hipGetLastError: that also returns what any other library's call on the thread left behind.
extern thread_local hipError_t launch_status;
template <class... P, class... A>
void launch(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t st, A&&... args) {
#if defined(__HIPCC__)
    std::tuple<P...> values(std::forward<A>(args)...);
    const hipError_t e = std::apply([&](auto&... v) {
        void* p[] = {(void*)&v...};
        return hipLaunchKernel((const void*)kernel, grid, block, p, lds, st);
    }, values);
#else   // host emulation of the kernels
    const hipError_t e = hipLaunchKernelGGL(kernel, grid, block, lds, st, std::forward<A>(args)...);
#endif
    if (e != hipSuccess && launch_status == hipSuccess) launch_status = e;
}

// Epilogues of the fp32 model's linear map.
enum {
    EPI_GELU = 1,       // out[r][n] = gelu(acc + bias)
    EPI_RESID = 2,      // x[r][n] += acc + bias
    EPI_F32 = 3,        // outf[r][n] = acc
    EPI_SILU_RESID = 4, // out[r][n] = in[r][n] + silu(acc + bias)   (needs N == K)
    EPI_QKV = 5         // n < d: q[r][n]; else key / value rows of the KV cache at L[b] + node
};

struct GemmArgs {
    const void* X;      // [R][K]
    const void* W;      // [N][K]
    const float* bias;  // [N] (not read for EPI_F32)
    int R, K, N;
    int epi;
    void* out;          // [R][N]
    float* outf;        // fp32 target (EPI_RESID: x, EPI_F32: logits)
    // EPI_QKV
    void *Kc, *Vc;      // layer base of the cache
    const int32_t* L;
    int M, nH, maxpos, d;
    uint32_t m_magic;   // ceil(2^32 / M) (0: M = 1)
    const float *ln_g, *ln_b;      // X = LayerNorm of these rows with this scale and shift (null: the rows as they are)
    size_t z_w, z_b, z_x, z_out;   // several draft heads in one launch: how far a head's weights, bias (bytes), X and result (elements) are ahead of the previous head's
};

// Phases of a bf16 step, as VADUSA_DBG_PHASE_CLOCK counts them: 0 embedding; 1 + 5 l .. layer l (QKV, attention,
// out-projection, FFN1, FFN2); then H + TP_*, H = 1 + 5 * n_layers.  TP_COMMIT: first map of the draft heads; TP_TOPK: draft
// lists and, beside them, the compaction of the KV cache.
enum { TP_HEAD = 0, TP_EDGES, TP_SELECT, TP_FINAL, TP_COMMIT, TP_DRAFT2, TP_TOPK, TP_COUNT };
// bf16 model: embedding, decoder layers and (head) the vocabulary map (see k_layer.hip).  Prompt passes (prefill_mode) are ragged; without
// head the last layer ends with its keys and values, with it only the sequences' last rows go on behind its attention where D.last_only.
void launch_layers(const Dims& D, const DevState& s, const std::vector<LayerW>& layers, int table, int prefill_mode, bool head, int big_min, hipStream_t st);
// edge decisions, and (select) the path choice of every sequence
void launch_verify_tail(const Dims& D, const DevState& s, int tau, int ignore_eos, bool select, hipStream_t st);
// (select: path choice,) continuation, draft heads, draft lists and KV compaction; host: memory the GPU can write that takes the results (see
// dev_finalize), or null
void launch_continue(const Dims& D, const DevState& s, const std::vector<DraftW>& draft, int seq0, int nseq, int prefill_mode, int ignore_eos, bool select, int32_t* host, int dtype, hipStream_t st);
void launch_pack_w_ln(const float* src, const float* gamma, const float* beta, void* dst, float* colsum,
                      float* tvec, int N, int K, hipStream_t st);
void launch_add_vec(float* dst, const float* src, int n, hipStream_t st);

// ---- launch wrappers (each enqueues on `st`, no synchronisation) ----
void launch_embed32(const Dims& D, const DevState& s, int prefill_mode, int table, hipStream_t st);
// fp32 model: the same as launch_layers, and the draft heads' maps (see k_fp32.hip)
void launch_layers32(const Dims& D, const DevState& s, const std::vector<LayerW>& layers, int table, int prefill_mode, bool head, hipStream_t st);
void launch_draft32(const Dims& D, const DevState& s, const std::vector<DraftW>& draft, int seq0, int nseq, hipStream_t st);
void launch_layernorm(const float* x, const float* g, const float* b, void* out, int R, int d, int dtype, hipStream_t st);
void launch_pack_w(const float* src, void* dst, int N, int K, hipStream_t st);
void launch_topk(const Dims& D, const DevState& s, int seq0, int nseq, hipStream_t st);
void launch_perturb(const float* logits, const float* u, float* scores, int rows, int V1, float temperature,
                    float top_p, int tau, hipStream_t st);
void launch_convert(const float* src, void* dst, size_t n, int dtype, hipStream_t st);
// na words from a, nb from b, nc from c, one behind the other, into host memory the GPU can write
void launch_gather(const int32_t* a, int na, const int32_t* b, int nb, const int32_t* c, int nc, int32_t* host, hipStream_t st);
void launch_advance(const DevState& s, int B, hipStream_t st);
void launch_reset(const DevState& s, int B, hipStream_t st);   // committed lengths, finished, outputs and paths back to zero
void launch_read_kv(const Dims& D, const void* cache_layer, int seq, int which, int pos0, int npos, float* out, int dtype, hipStream_t st);
void launch_to_float(const void* src, float* dst, size_t n, int dtype, hipStream_t st);
