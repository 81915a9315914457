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
// Y = X W^T (+ bias) with the epilogues of common.h, X = LayerNorm(x) where GemmArgs::ln_g is given.  One workgroup per
// 16 rows x 16 columns, the four waves split the reduction in steps of 16 (a lane's four consecutive values of a row are
// four matrix instructions' operands; both operands take the same order, so no value moves between lanes), eight steps
// requested at a time.  A wave keeps 16 accumulators, which makes 64 partial sums of K / 64 products, added pairwise, in the
// wave and then through LDS: with one chain of K / 4 per wave a model's logits were twice as far from 64-bit arithmetic (two
// and three layers: 4.4e-7 and 5.2e-7 against 2.4e-7 and 2.5e-7) and a step took 1 to 3 % less (two layers, d = 256, 16 rows:
// 94 us against 96).  Launch bounds of two: the accumulators stay where additions can read them (2.5 % of a step).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256, 2) void k_lin32(GemmArgs a) {
    constexpr int CH = 8;
    __shared__ f32x4_t red[4 * 64];
    __shared__ float s_mean[16], s_rstd[16];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lc = lane & 15, gq = lane >> 4;
    const int n0 = blockIdx.x * 16, r0 = blockIdx.y * 16, z = blockIdx.z;
    const float* X = (const float*)a.X + z * a.z_x;
    const float* W = (const float*)((const char*)a.W + z * a.z_w) + (size_t)min(n0 + lc, a.N - 1) * a.K + 4 * gq;
    const float* xrow = X + (size_t)min(r0 + lc, a.R - 1) * a.K + 4 * gq;
    const int steps = a.K >> 4, lo = (steps * wave) >> 2, hi = (steps * (wave + 1)) >> 2;
    float4 w[CH], x[CH], lg[CH], lb[CH];
    auto load = [&](int s) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int k = 16 * min(s + i, steps - 1);
            w[i] = ldgf4(W + k);
            x[i] = ldgf4(xrow + k);
            if (a.ln_g) { lg[i] = ldgf4(a.ln_g + k + 4 * gq); lb[i] = ldgf4(a.ln_b + k + 4 * gq); }
        }
    };
    if (a.ln_g) {   // mean and variance of the 16 rows: 16 threads each (biased variance, eps 1e-5)
        constexpr int NV = 6;   // values up to K = 384 stay in registers and are requested at once
        const int row = tid >> 4, part = tid & 15;
        const float* p = X + (size_t)min(r0 + row, a.R - 1) * a.K + 4 * part;
        float4 v[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j] = 64 * j + 4 * part < a.K ? ldgf4(p + 64 * j) : make_float4(0.f, 0.f, 0.f, 0.f);
        load(lo);
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < NV; ++j) sum += (v[j].x + v[j].y) + (v[j].z + v[j].w);
        for (int k = 64 * NV; k + 4 * part < a.K; k += 64) { const float4 u = ldgf4(p + k); sum += (u.x + u.y) + (u.z + u.w); }
        const float mu = row16_sum(sum) / a.K;
        float sq = 0.f;
        auto add = [&](const float4& u) {
            sq += ((u.x - mu) * (u.x - mu) + (u.y - mu) * (u.y - mu)) + ((u.z - mu) * (u.z - mu) + (u.w - mu) * (u.w - mu));
        };
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (64 * j + 4 * part < a.K) add(v[j]);
        for (int k = 64 * NV; k + 4 * part < a.K; k += 64) add(ldgf4(p + k));
        sq = row16_sum(sq);
        if (part == 0) { s_mean[row] = mu; s_rstd[row] = rsqrtf(sq / a.K + LN_EPS); }
        __syncthreads();
    } else {
        load(lo);
    }
    const float mu = a.ln_g ? s_mean[lc] : 0.f, rstd = a.ln_g ? s_rstd[lc] : 1.f;
    f32x4_t acc[4][4];   // [step mod 4][which of a lane's four values]
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i >> 2][i & 3] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    for (int s = lo; s < hi; s += CH) {
        if (s > lo) load(s);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (s + i >= hi) break;
            float4 v = x[i];
            if (a.ln_g) {
                const float4 g = lg[i], b = lb[i];
                v = make_float4((v.x - mu) * rstd * g.x + b.x, (v.y - mu) * rstd * g.y + b.y, (v.z - mu) * rstd * g.z + b.z, (v.w - mu) * rstd * g.w + b.w);
            }
            f32x4_t(&a4)[4] = acc[i & 3];
            a4[0] = mfma_16x16x4(w[i].x, v.x, a4[0]);   // weights first: a lane then holds four consecutive columns of one row
            a4[1] = mfma_16x16x4(w[i].y, v.y, a4[1]);
            a4[2] = mfma_16x16x4(w[i].z, v.z, a4[2]);
            a4[3] = mfma_16x16x4(w[i].w, v.w, a4[3]);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i][0] = (acc[i][0] + acc[i][1]) + (acc[i][2] + acc[i][3]);
    red[tid] = (acc[0][0] + acc[1][0]) + (acc[2][0] + acc[3][0]);
    __syncthreads();
    if (wave) return;
    const f32x4_t s = (red[lane] + red[64 + lane]) + (red[128 + lane] + red[192 + lane]);
    const int r = r0 + lc;
    if (r >= a.R) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = n0 + 4 * gq + j;
        if (n >= a.N) break;
        float v = s[j];
        if (a.bias) v += ((const float*)((const char*)a.bias + z * a.z_b))[n];
        switch (a.epi) {
        case EPI_GELU: ((float*)a.out)[(size_t)r * a.N + n] = gelu_f(v); break;
        case EPI_RESID: a.outf[(size_t)r * a.N + n] += v; break;
        case EPI_F32: a.outf[z * a.z_out + (size_t)r * a.N + n] = v; break;
        case EPI_SILU_RESID: ((float*)a.out)[z * a.z_out + (size_t)r * a.N + n] = X[(size_t)r * a.K + n] + silu_f(v); break;
        case EPI_QKV: {
            if (n < a.d) { ((float*)a.out)[(size_t)r * a.d + n] = v; break; }
            const int which = n / a.d - 1, c = n % a.d, head = c >> 6, dim = c & 63;
            const int b = r / a.M, pos = a.L[b] + r % a.M;
            if (pos < a.maxpos) {
                const size_t hb = ((size_t)b * a.nH + head) * kv_cap(a.maxpos) * 64;
                if (which) ((float*)a.Vc)[hb + vc_off(pos, dim)] = v;
                else ((float*)a.Kc)[hb + kc_off(pos, dim)] = v;
            }
            break;
        }
        }
    }
}

static void lin32(const GemmArgs& a, hipStream_t st, int nz = 1) {
    launch(k_lin32, dim3(cdiv(a.N, 16), cdiv(a.R, 16), nz), dim3(256), 0, st, a);
}

// ---------------------------------------------------------------------------
// Tree-masked attention (Sec. 2.1): one workgroup per (row, head).  A row sees cache positions [0, L) and, among the rows
// of this forward (stored at cache rows L + m), those whose bit is set in its mask row (table 1, a causal pass of the
// prompt: rows 0 .. n).  The four waves take 32-key blocks round-robin with a private online softmax: two lanes share a
// key's score (32 dimensions each, 16-byte loads), then a lane is a dimension and takes the block's 32 values as eight
// 16-byte loads; the four results merge through LDS.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_attn32(Dims D, DevState s, int layer, int table) {
    __shared__ float s_q[64], s_o[4][64], s_m[4], s_l[4];
    const int n = blockIdx.x, head = blockIdx.y, b = blockIdx.z, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const size_t r = (size_t)b * D.M + n;
    float* out = (float*)s.att + r * D.d + head * 64;
    if (n >= s.n_rows[b]) { if (wave == 0) out[lane] = 0.f; return; }
    const int L = s.L[b], T = min(table == 1 ? L + n + 1 : L + D.M, D.maxpos);   // (a causal row sees nothing behind itself)
    const size_t hb = ((((size_t)layer * D.Bmax + b) * D.nH + head) * kv_cap(D.maxpos)) * 64;
    const float *Kh = (const float*)s.Kc + hb, *Vh = (const float*)s.Vc + hb;
    // table 1 may have more rows than the mask table has entries: no mask words are read for it
    const uint32_t* mrow = s.t_mask[0] + (size_t)(table == 1 ? 0 : n) * MASK_WORDS;
    if (wave == 0) s_q[lane] = ((const float*)s.q)[r * D.d + head * 64 + lane] * 0.125f;
    __syncthreads();
    const int key = lane & 31, half = lane >> 5;
    float m = -INFINITY, l = 0.f, o = 0.f;
    for (int p0 = 32 * wave; p0 < T; p0 += 128) {
        float4 kv[8], vv[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {   // eight dimensions of the lane's key are 32 contiguous bytes
            const float* kp = Kh + kc_off(p0 + key, 32 * half + 8 * i);
            kv[2 * i] = ldgf4(kp);
            kv[2 * i + 1] = ldgf4(kp + 4);
            const float* vp = Vh + vc_off(p0 + 8 * i, lane);   // eight positions of the lane's dimension as well
            vv[2 * i] = ldgf4(vp);
            vv[2 * i + 1] = ldgf4(vp + 4);
        }
        float sc = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float* q = s_q + 32 * half + 4 * i;
            sc = fmaf(q[0], kv[i].x, sc); sc = fmaf(q[1], kv[i].y, sc); sc = fmaf(q[2], kv[i].z, sc); sc = fmaf(q[3], kv[i].w, sc);
        }
        sc = half_sum(sc);
        const int pos = p0 + key, mm = pos - L;
        bool see = pos < T;
        if (see && mm >= 0 && table != 1) see = (mrow[(mm >> 5) & (MASK_WORDS - 1)] >> (mm & 31)) & 1u;
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
    for (int l = 0; l < D.Ly; ++l) {
        const LayerW& w = layers[l];
        GemmArgs a = base;
        a.X = s.x; a.ln_g = w.ln1_g; a.ln_b = w.ln1_b; a.W = w.Wqkv; a.bias = w.bqkv; a.K = D.d; a.N = 3 * D.d; a.epi = EPI_QKV;
        a.out = s.q; a.Kc = (float*)s.Kc + l * kv_layer; a.Vc = (float*)s.Vc + l * kv_layer;
        lin32(a, st);
        launch(k_attn32, dim3(D.M, D.nH, D.B), dim3(256), 0, st, D, s, l, table);
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
