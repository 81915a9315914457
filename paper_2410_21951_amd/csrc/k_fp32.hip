// The linear maps and the attention of the fp32 model (weights [N][K] row-major, activations [R][K] row-major, everything
// in fp32).  These models are small: a launch is a few microseconds whatever it computes, so what counts is few launches
// (LayerNorm is part of the map behind it, the draft heads share a launch) and no long dependent chains inside one.
#include "common.h"

typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// D = A B + C, A 16 x 4 (lane: row lane & 15, k lane >> 4), B 4 x 16 alike; lane l, element i of D: column l & 15, row
// 4 (l >> 4) + i.  Products and sums are fp32.
__device__ __forceinline__ f32x4_t mfma_16x16x4(float a, float b, f32x4_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
#else   // host emulation of the kernels: the wave's operands meet in an array, between two lane exchanges
    __shared__ float ops[4][2][64];
    const int w = (int)(threadIdx.x >> 6), l = (int)(threadIdx.x & 63);
    ops[w][0][l] = a;
    ops[w][1][l] = b;
    (void)__shfl(0u, 0, 64);
    for (int i = 0; i < 4; ++i)
        for (int k = 0; k < 4; ++k) c[i] = fmaf(ops[w][0][4 * (l >> 4) + i + 16 * k], ops[w][1][(l & 15) + 16 * k], c[i]);
    (void)__shfl(0u, 0, 64);
    return c;
#endif
}
__device__ __forceinline__ float4 ldgf4(const float* p) {
    const uint4 v = ldg4(p);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
__device__ __forceinline__ float gelu_f(float v) { return 0.5f * v * (1.f + erff(v * 0.70710678118654752f)); }
__device__ __forceinline__ float silu_f(float v) { return v / (1.f + __expf(-v)); }

// ---------------------------------------------------------------------------
// Y = X W^T (+ bias) with the epilogues of common.h, X = LayerNorm(x) where LN.  One workgroup per
// 16 rows x 16 columns, the four waves split the reduction in steps of 16 (a lane's four consecutive values of a row are
// four matrix instructions' operands; both operands take the same order, so no value moves between lanes), eight steps
// requested at a time.  A wave keeps 16 accumulators, which makes 64 partial sums of K / 64 products, added pairwise, in the
// wave and then through LDS: with one chain of K / 4 per wave a model's logits were twice as far from 64-bit arithmetic (two
// and three layers: 4.4e-7 and 5.2e-7 against 2.4e-7 and 2.5e-7) and a step took 1 to 3 % less (two layers, d = 256, 16 rows:
// 94 us against 96).  Launch bounds of two: the accumulators stay where additions can read them (2.5 % of a step).
// What bounds it is the chain of waits from the launch to the store, so what the first loads' addresses need arrives in registers with the wave (the
// leading arguments), the epilogue's inputs are asked for before the products, and every thread finishes one output.  (One wave finishing all,
// with bias, residual value and length read at the end and the kind of map found at run time: a step of two layers, d = 256, 16 rows, 94.6 us; now 72.7.)
// u0, u1: LayerNorm's scale and shift (U: a pointer, LN), or what a draft head's weights (bytes) and X (elements) are ahead of the previous head's (U: a number).
// ---------------------------------------------------------------------------
template <int EPI, class U>
__global__ __launch_bounds__(256, 2) void k_lin32(const float* X, const float* W, int R, int K, int N, U u0, U u1, GemmArgs a) {
    constexpr bool LN = std::is_same<U, const float*>::value;
    constexpr int CH = 8;
    __shared__ f32x4_t red[4 * 64];
    __shared__ float s_mean[16], s_rstd[16];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, lc = lane & 15, gq = lane >> 4;
    const int n0 = blockIdx.x * 16, r0 = blockIdx.y * 16, z = blockIdx.z;
    const float *ln_g = nullptr, *ln_b = nullptr;
    if constexpr (LN) {
        ln_g = u0;
        ln_b = u1;
    } else {
        W = (const float*)((const char*)W + z * u0);
        X += z * u1;
    }
    const float* Wt = W + (size_t)n0 * K;   // the workgroup's columns and rows
    const float* Xt = X + (size_t)r0 * K;
    const uint32_t wrow = (uint32_t)min(lc, N - 1 - n0) * (uint32_t)K + 4u * gq, xrow = (uint32_t)min(lc, R - 1 - r0) * (uint32_t)K + 4u * gq;
    const int steps = K >> 4, lo = (steps * wave) >> 2, hi = (steps * (wave + 1)) >> 2;
    float4 w[CH], x[CH], lg[CH], lb[CH];
    auto load4 = [&](int s, int i0) {   // steps s + i0 .. s + i0 + 3; one beyond the last re-reads it and is not multiplied
#pragma unroll
        for (int i = i0; i < i0 + 4; ++i) {
            const int k = 16 * min(s + i, steps - 1);
            w[i] = ldgf4(Wt + k + wrow);
            x[i] = ldgf4(Xt + k + xrow);
            if constexpr (LN) { lg[i] = ldgf4(ln_g + k + 4 * gq); lb[i] = ldgf4(ln_b + k + 4 * gq); }
        }
    };
    auto load = [&](int s) {
        load4(s, 0);
        if (s + 4 < hi) load4(s, 4);
    };
    constexpr int NV = 6;   // values up to K = 384 stay in registers and are requested at once
    const int row = tid >> 4, part = tid & 15;
    const float* p = Xt + (uint32_t)min(row, R - 1 - r0) * (uint32_t)K + 4 * part;
    float4 v[NV];
    if constexpr (LN)
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j] = 64 * j + 4 * part < K ? ldgf4(p + 64 * j) : make_float4(0.f, 0.f, 0.f, 0.f);
    load(lo);
    // this thread's output, and what it needs beside the sum
    const int r = r0 + lc, n = n0 + 4 * gq + wave, rr = min(r, R - 1), nn = min(n, N - 1);
    float bias = 0.f, old = 0.f;
    int pos = 0, seq = 0;
    if (EPI != EPI_F32) bias = ldg((const float*)((const char*)a.bias + z * a.z_b) + nn);
    if (EPI == EPI_RESID) old = ldg(a.outf + (size_t)rr * N + nn);
    if (EPI == EPI_SILU_RESID) old = ldg(X + (size_t)rr * K + nn);
    if (EPI == EPI_QKV) {
        seq = a.m_magic ? (int)(((uint64_t)(uint32_t)rr * a.m_magic) >> 32) : rr;
        pos = ldg(a.L + seq);
    }
    if constexpr (LN) {   // mean and variance of the 16 rows: 16 threads each (biased variance, eps 1e-5)
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < NV; ++j) sum += (v[j].x + v[j].y) + (v[j].z + v[j].w);
        for (int k = 64 * NV; k + 4 * part < K; k += 64) { const float4 u = ldgf4(p + k); sum += (u.x + u.y) + (u.z + u.w); }
        const float mu = row16_sum(sum) / K;
        float sq = 0.f;
        auto add = [&](const float4& u) {
            sq += ((u.x - mu) * (u.x - mu) + (u.y - mu) * (u.y - mu)) + ((u.z - mu) * (u.z - mu) + (u.w - mu) * (u.w - mu));
        };
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (64 * j + 4 * part < K) add(v[j]);
        for (int k = 64 * NV; k + 4 * part < K; k += 64) add(ldgf4(p + k));
        sq = row16_sum(sq);
        if (part == 0) { s_mean[row] = mu; s_rstd[row] = rsqrtf(sq / K + LN_EPS); }
        __syncthreads();
    }
    const float mu = LN ? s_mean[lc] : 0.f, rstd = LN ? s_rstd[lc] : 1.f;
    f32x4_t acc[4][4];   // [step mod 4][which of a lane's four values]
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i >> 2][i & 3] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    for (int s = lo; s < hi; s += CH) {
        if (s > lo) load(s);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (s + i >= hi) break;
            float4 u = x[i];
            if constexpr (LN) {
                const float4 g = lg[i], b = lb[i];
                u = make_float4((u.x - mu) * rstd * g.x + b.x, (u.y - mu) * rstd * g.y + b.y, (u.z - mu) * rstd * g.z + b.z, (u.w - mu) * rstd * g.w + b.w);
            }
            f32x4_t(&a4)[4] = acc[i & 3];
            a4[0] = mfma_16x16x4(w[i].x, u.x, a4[0]);   // weights first: a lane then holds four consecutive columns of one row
            a4[1] = mfma_16x16x4(w[i].y, u.y, a4[1]);
            a4[2] = mfma_16x16x4(w[i].z, u.z, a4[2]);
            a4[3] = mfma_16x16x4(w[i].w, u.w, a4[3]);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i][0] = (acc[i][0] + acc[i][1]) + (acc[i][2] + acc[i][3]);
    red[tid] = (acc[0][0] + acc[1][0]) + (acc[2][0] + acc[3][0]);
    __syncthreads();
    auto sum_of = [&](int w) { return ((const float*)&red[w * 64 + lane])[wave]; };
    const float y = ((sum_of(0) + sum_of(1)) + (sum_of(2) + sum_of(3))) + bias;
    if (r >= R || n >= N) return;
    if constexpr (EPI == EPI_GELU) ((float*)a.out)[(size_t)r * N + n] = gelu_f(y);
    if constexpr (EPI == EPI_RESID) a.outf[(size_t)r * N + n] = old + y;
    if constexpr (EPI == EPI_F32) a.outf[z * a.z_out + (size_t)r * N + n] = y;
    if constexpr (EPI == EPI_SILU_RESID) ((float*)a.out)[z * a.z_out + (size_t)r * N + n] = old + silu_f(y);
    if constexpr (EPI == EPI_QKV) {   // (a workgroup's columns are all queries, all keys or all values: d is a multiple of 64)
        if (n0 < a.d) { ((float*)a.out)[(size_t)r * a.d + n] = y; return; }
        const int which = n0 >= 2 * a.d, c = n - (which + 1) * a.d, head = c >> 6, dim = c & 63;
        pos += r - seq * a.M;
        if (pos < a.maxpos) {
            const size_t hb = ((size_t)seq * a.nH + head) * kv_cap(a.maxpos) * 64;
            if (which) ((float*)a.Vc)[hb + vc_off(pos, dim)] = y;
            else ((float*)a.Kc)[hb + kc_off(pos, dim)] = y;
        }
    }
}

template <int EPI, class U>
static void lin32_launch(const GemmArgs& a, U u0, U u1, hipStream_t st, int nz) {
    launch(k_lin32<EPI, U>, dim3(cdiv(a.N, 16), cdiv(a.R, 16), nz), dim3(256), 0, st, (const float*)a.X, (const float*)a.W, a.R, a.K, a.N, u0, u1, a);
}
static void lin32(const GemmArgs& a, hipStream_t st, int nz = 1) {
    switch (a.epi) {
    case EPI_QKV: lin32_launch<EPI_QKV>(a, a.ln_g, a.ln_b, st, nz); break;
    case EPI_GELU: lin32_launch<EPI_GELU>(a, a.ln_g, a.ln_b, st, nz); break;
    case EPI_RESID: lin32_launch<EPI_RESID>(a, a.z_w, a.z_x, st, nz); break;
    case EPI_SILU_RESID: lin32_launch<EPI_SILU_RESID>(a, a.z_w, a.z_x, st, nz); break;
    default:
        if (a.ln_g) lin32_launch<EPI_F32>(a, a.ln_g, a.ln_b, st, nz);
        else lin32_launch<EPI_F32>(a, a.z_w, a.z_x, st, nz);
    }
}

// ---------------------------------------------------------------------------
// Tree-masked attention (Sec. 2.1): one workgroup per (row, head).  A row sees cache positions [0, L) and, among the rows
// of this forward (stored at cache rows L + m), those whose bit is set in its mask row (table 1, a causal pass of the
// prompt: rows 0 .. n).  The four waves take 32-key blocks round-robin with a private online softmax: two lanes share a
// key's score (32 dimensions each, 16-byte loads), then a lane is a dimension and takes the block's 32 values as eight
// 16-byte loads; the four results merge through LDS.  What bounds it is the chain from the launch to the first score: the first block and the query are asked for at
// once, by leading arguments, and not behind the length, an LDS copy of the query and a barrier, and the mask's words come with them (a step of two layers, 16 rows, some 200 keys: 74.6 -> 72.8 us).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_attn32(const float* q, const float* Kc, const float* Vc, const int32_t* L_of, const int32_t* rows_of, int M, int nH, int maxpos, int table, const uint32_t* mask, float* att) {
    __shared__ float s_o[4][64], s_m[4], s_l[4];
    const int n = blockIdx.x, head = blockIdx.y, b = blockIdx.z, tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const size_t r = (size_t)b * M + n, at = r * nH * 64 + head * 64;
    const int L = ldg(L_of + b), rows = ldg(rows_of + b), key = lane & 31, half = lane >> 5;
    const size_t hb = ((size_t)b * nH + head) * kv_cap(maxpos) * 64;
    const float *Kh = Kc + hb, *Vh = Vc + hb;
    float4 kv[8], vv[8], qv[8];
    auto load = [&](int p0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // eight dimensions of the lane's key are 32 contiguous bytes
            const float* kp = Kh + kc_off(p0 + key, 32 * half + 8 * i);
            kv[2 * i] = ldgf4(kp);
            kv[2 * i + 1] = ldgf4(kp + 4);
            const float* vp = Vh + vc_off(p0 + 8 * i, lane);   // eight positions of the lane's dimension as well
            vv[2 * i] = ldgf4(vp);
            vv[2 * i + 1] = ldgf4(vp + 4);
        }
    };
    load(32 * wave < kv_cap(maxpos) ? 32 * wave : 0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float4 v = ldgf4(q + at + 32 * half + 4 * i);
        qv[i] = make_float4(v.x * 0.125f, v.y * 0.125f, v.z * 0.125f, v.w * 0.125f);
    }
    // table 1 may have more rows than the mask table has entries: its words are not used
    const uint4 mw = ldg4(mask + (size_t)(table == 1 ? 0 : n) * MASK_WORDS);
    float* out = att + at;
    if (n >= rows) { if (wave == 0) out[lane] = 0.f; return; }
    const int T = min(table == 1 ? L + n + 1 : L + M, maxpos);   // (a causal row sees nothing behind itself)
    float m = -INFINITY, l = 0.f, o = 0.f;
    for (int p0 = 32 * wave; p0 < T; p0 += 128) {
        if (p0 > 32 * wave) load(p0);
        float sc = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            sc = fmaf(qv[i].x, kv[i].x, sc); sc = fmaf(qv[i].y, kv[i].y, sc); sc = fmaf(qv[i].z, kv[i].z, sc); sc = fmaf(qv[i].w, kv[i].w, sc);
        }
        sc = half_sum(sc);
        const int pos = p0 + key, mm = pos - L;
        bool see = pos < T;
        const uint32_t lower = mm & 32 ? mw.y : mw.x, upper = mm & 32 ? mw.w : mw.z, word = mm & 64 ? upper : lower;
        if (mm >= 0 && table != 1) see &= (word >> (mm & 31)) & 1u;
        float mx = see ? sc : -INFINITY;
        mx = fmaxf(mx, __int_as_float(dpp_perm<0xB1>(__float_as_int(mx))));
        mx = fmaxf(mx, __int_as_float(dpp_perm<0x4E>(__float_as_int(mx))));
        mx = fmaxf(mx, __int_as_float(dpp_perm<0x141>(__float_as_int(mx))));
        mx = fmaxf(mx, __int_as_float(dpp_perm<0x140>(__float_as_int(mx))));
        const float mn = fmaxf(m, rows_max(mx));
        const float p = see ? __expf(sc - mn) : 0.f;
        const float corr = mn == -INFINITY ? 1.f : __expf(m - mn);   // (a block without a visible key leaves everything as it was)
        l = l * corr + 0.5f * wave_sum_dpp(p);                          // each key sits in two lanes
        m = mn;
        o *= corr;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float v4[4] = {vv[i].x, vv[i].y, vv[i].z, vv[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {   // (a key that is not seen may hold anything)
                const float pk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p), 4 * i + j));
                o = fmaf(pk, pk == 0.f ? 0.f : v4[j], o);
            }
        }
    }
    s_o[wave][lane] = o;
    if (lane == 0) { s_m[wave] = m; s_l[wave] = l; }
    __syncthreads();
    if (wave) return;
    const float mx = fmaxf(fmaxf(s_m[0], s_m[1]), fmaxf(s_m[2], s_m[3]));
    float lt = 0.f, acc = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float f = s_m[w] == -INFINITY ? 0.f : __expf(s_m[w] - mx);
        lt += f * s_l[w];
        acc += f * s_o[w][lane];
    }
    out[lane] = acc / lt;
}

// Embedding, decoder layers and (head) the vocabulary map.
void launch_layers32(const Dims& D, const DevState& s, const std::vector<LayerW>& layers, int table, int prefill_mode, bool head, hipStream_t st) {
    const int R = D.B * D.M;
    const size_t kv_layer = (size_t)D.Bmax * D.nH * kv_cap(D.maxpos) * 64;
    launch_embed32(D, s, prefill_mode, table, st);
    GemmArgs base{};
    base.R = R; base.L = s.L; base.M = D.M; base.nH = D.nH; base.maxpos = D.maxpos; base.d = D.d;
    base.m_magic = D.M > 1 ? (uint32_t)(((1ull << 32) + D.M - 1) / D.M) : 0;
    for (int l = 0; l < D.Ly; ++l) {
        const LayerW& w = layers[l];
        GemmArgs a = base;
        a.X = s.x; a.ln_g = w.ln1_g; a.ln_b = w.ln1_b; a.W = w.Wqkv; a.bias = w.bqkv; a.K = D.d; a.N = 3 * D.d; a.epi = EPI_QKV;
        a.out = s.q; a.Kc = (float*)s.Kc + l * kv_layer; a.Vc = (float*)s.Vc + l * kv_layer;
        lin32(a, st);
        launch(k_attn32, dim3(D.M, D.nH, D.B), dim3(256), 0, st, (const float*)s.q, (const float*)a.Kc, (const float*)a.Vc, (const int32_t*)s.L, (const int32_t*)s.n_rows, D.M, D.nH, D.maxpos, table,
               (const uint32_t*)s.t_mask[0], (float*)s.att);
        GemmArgs o = base;
        o.X = s.att; o.W = w.Wo; o.bias = w.bo; o.K = D.d; o.N = D.d; o.epi = EPI_RESID; o.outf = s.x;
        lin32(o, st);
        GemmArgs f = base;
        f.X = s.x; f.ln_g = w.ln2_g; f.ln_b = w.ln2_b; f.W = w.W1; f.bias = w.b1; f.K = D.d; f.N = D.F; f.epi = EPI_GELU; f.out = s.hid;
        lin32(f, st);
        GemmArgs g = base;
        g.X = s.hid; g.W = w.W2; g.bias = w.b2; g.K = D.F; g.N = D.d; g.epi = EPI_RESID; g.outf = s.x;
        lin32(g, st);
    }
    if (head) {
        GemmArgs h = base;
        h.X = s.x; h.ln_g = s.lnf_g; h.ln_b = s.lnf_b; h.W = s.W_out; h.K = D.d; h.N = D.V1; h.epi = EPI_F32; h.outf = s.logits;
        lin32(h, st);
    }
}

// Both maps of the draft heads, a launch each for all heads.
void launch_draft32(const Dims& D, const DevState& s, const std::vector<DraftW>& draft, int seq0, int nseq, hipStream_t st) {
    auto ahead = [&](const void* a, const void* b) { return D.Hh > 1 ? (size_t)((const char*)b - (const char*)a) : 0; };
    const DraftW &d0 = draft[0], &d1 = draft[D.Hh > 1 ? 1 : 0];
    GemmArgs a{};
    a.X = (const float*)s.hbest + (size_t)seq0 * D.d; a.W = d0.W1; a.bias = d0.b1; a.R = nseq; a.K = D.d; a.N = D.d; a.epi = EPI_SILU_RESID;
    a.out = (float*)s.rdraft + (size_t)seq0 * D.d; a.z_w = ahead(d0.W1, d1.W1); a.z_b = ahead(d0.b1, d1.b1); a.z_out = (size_t)D.Bmax * D.d;
    lin32(a, st, D.Hh);
    GemmArgs z{};
    z.X = (const float*)s.rdraft + (size_t)seq0 * D.d; z.W = d0.W2; z.R = nseq; z.K = D.d; z.N = D.V1; z.epi = EPI_F32;
    z.outf = s.zdraft + (size_t)seq0 * D.V1; z.z_w = ahead(d0.W2, d1.W2); z.z_x = (size_t)D.Bmax * D.d; z.z_out = (size_t)D.Bmax * D.V1;
    lin32(z, st, D.Hh);
}
