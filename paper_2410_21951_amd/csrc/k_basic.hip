// Element-wise kernels: embedding / tree expansion of the fp32 model, LayerNorm of all rows (inspection), and a few
// conversion helpers.  Templated on the storage type (float or bf16 bits); all arithmetic is fp32.
#include "common.h"

// ---------------------------------------------------------------------------
// Tree expansion + embedding (Sec. 2.1: the root is the base head's next token,
// depth D is filled from draft head D's top-k list; positions continue after
// the committed prefix).  In prefill mode the rows are consecutive prompt
// tokens: text ids are passed as -(id + 1), speech ids as they are.
// One block per row.
// ---------------------------------------------------------------------------
__global__ void k_embed32(Dims D, DevState s, int prefill_mode, int table) {
    const int r = blockIdx.x, b = r / D.M, n = r % D.M;
    float* x = s.x + (size_t)r * D.d;
    int rows;
    if (prefill_mode) rows = s.n_rows[b];
    else rows = s.finished[b] ? 0 : D.M;
    if (!prefill_mode && n == 0 && threadIdx.x == 0) s.n_rows[b] = rows;
    if (n >= rows) {
        for (int i = threadIdx.x; i < D.d; i += blockDim.x) x[i] = 0.f;
        if (threadIdx.x == 0) s.tok[r] = 0;
        return;
    }
    int tok, pos;
    const float* E;
    if (prefill_mode) {
        int t = s.chunk_tok[r];
        pos = s.L[b] + n;
        if (t < 0) { tok = -t - 1; E = (const float*)s.E_text; }
        else { tok = t; E = (const float*)s.E_speech; }
    } else {
        int dep = s.t_depth[table][n];
        pos = s.L[b] + dep;
        if (n == 0) tok = s.root[b];
        else tok = s.draft_topk[((size_t)b * D.Hh + (dep - 1)) * VADUSA_MAX_TOPK + s.t_rank[table][n]];
        if ((unsigned)tok >= (unsigned)D.V1) tok = 0;   // rows of NaN logits have no arg-max and no draft lists: stay inside the table
        E = (const float*)s.E_speech;
    }
    if (pos >= D.maxpos) pos = D.maxpos - 1;   // never reached: the host checks capacity first
    if (threadIdx.x == 0) s.tok[r] = tok;
    const float* e = E + (size_t)tok * D.d;
    const float* p = (const float*)s.P + (size_t)pos * D.d;
    for (int i = threadIdx.x; i < D.d; i += blockDim.x) x[i] = e[i] + p[i];
}

void launch_embed32(const Dims& D, const DevState& s, int prefill_mode, int table, hipStream_t st) {
    launch(k_embed32, dim3(D.B * D.M), dim3(256), 0, st, D, s, prefill_mode, table);
}

// ---------------------------------------------------------------------------
// LayerNorm over the last axis, one wave per row (biased variance, eps 1e-5).
// ---------------------------------------------------------------------------
template <class T>
__global__ void k_layernorm(const float* __restrict__ x, const float* __restrict__ g,
                            const float* __restrict__ bt, T* __restrict__ out, int R, int d) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int r = blockIdx.x * (blockDim.x >> 6) + wave;
    if (r >= R) return;
    const float* xr = x + (size_t)r * d;
    float sum = 0.f;
    for (int i = lane; i < d; i += 64) sum += xr[i];
    const float mu = wave_sum(sum) / d;
    float sq = 0.f;
    for (int i = lane; i < d; i += 64) { float t = xr[i] - mu; sq += t * t; }
    const float rstd = rsqrtf(wave_sum(sq) / d + LN_EPS);
    T* o = out + (size_t)r * d;
    for (int i = lane; i < d; i += 64) stf(o + i, (xr[i] - mu) * rstd * g[i] + bt[i]);
}

void launch_layernorm(const float* x, const float* g, const float* b, void* out, int R, int d, int dtype, hipStream_t st) {
    dim3 grid((R + 3) / 4), blk(256);
    if (dtype) launch(k_layernorm<bf16_t>, grid, blk, 0, st, x, g, b, (bf16_t*)out, R, d);
    else launch(k_layernorm<float>, grid, blk, 0, st, x, g, b, (float*)out, R, d);
}

// ---------------------------------------------------------------------------
// Helpers: fp32 -> storage conversion, storage -> fp32, prefill bookkeeping,
// KV read-back for inspection.
// ---------------------------------------------------------------------------
template <class T>
__global__ void k_convert(const float* __restrict__ src, T* __restrict__ dst, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) stf(dst + i, src[i]);
}
void launch_convert(const float* src, void* dst, size_t n, int dtype, hipStream_t st) {
    int blocks = (int)((n + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    if (dtype) launch(k_convert<bf16_t>, dim3(blocks), dim3(256), 0, st, src, (bf16_t*)dst, n);
    else launch(k_convert<float>, dim3(blocks), dim3(256), 0, st, src, (float*)dst, n);
}

template <class T>
__global__ void k_to_float(const T* __restrict__ src, float* __restrict__ dst, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) dst[i] = ldf(src + i);
}
void launch_to_float(const void* src, float* dst, size_t n, int dtype, hipStream_t st) {
    int blocks = (int)((n + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    if (dtype) launch(k_to_float<bf16_t>, dim3(blocks), dim3(256), 0, st, (const bf16_t*)src, dst, n);
    else launch(k_to_float<float>, dim3(blocks), dim3(256), 0, st, (const float*)src, dst, n);
}

__global__ void k_advance(DevState s, int B) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < B) s.L[b] += s.n_rows[b];
}
__global__ __launch_bounds__(256) void k_reset(DevState s, int B) {
    constexpr int W = VADUSA_MAX_DRAFT_HEADS + 2;
    for (int i = threadIdx.x; i < B * W; i += 256) {
        s.path[i] = 0;
        if (i < B) s.L[i] = s.finished[i] = s.n_out[i] = 0;
    }
}
void launch_reset(const DevState& s, int B, hipStream_t st) { launch(k_reset, dim3(1), dim3(256), 0, st, s, B); }
void launch_advance(const DevState& s, int B, hipStream_t st) {
    launch(k_advance, dim3((B + 63) / 64), dim3(64), 0, st, s, B);
}

__global__ __launch_bounds__(256) void k_gather(const int32_t* a, int na, const int32_t* b, int nb, const int32_t* c, int nc, int32_t* host) {
    for (int i = threadIdx.x; i < na + nb + nc; i += 256) host[i] = i < na ? a[i] : i < na + nb ? b[i - na] : c[i - na - nb];
}
void launch_gather(const int32_t* a, int na, const int32_t* b, int nb, const int32_t* c, int nc, int32_t* host, hipStream_t st) {
    launch(k_gather, dim3(1), dim3(256), 0, st, a, na, b, nb, c, nc, host);
}

// out[p][head*64 + dim] = K or V of (seq, head, position pos0 + p, dim)
template <class T>
__global__ void k_read_kv(Dims D, const T* __restrict__ cache, int seq, int which, int pos0, int npos, float* out) {
    const int p = blockIdx.x;
    for (int c = threadIdx.x; c < D.d; c += blockDim.x) {
        const int head = c >> 6, dim = c & 63;
        const size_t hb = ((size_t)seq * D.nH + head) * kv_cap(D.maxpos) * 64;
        out[(size_t)p * D.d + c] = which ? ldf(cache + hb + vc_off(pos0 + p, dim)) : ldf(cache + hb + kc_off(pos0 + p, dim));
    }
}
void launch_read_kv(const Dims& D, const void* cache_layer, int seq, int which, int pos0, int npos, float* out, int dtype, hipStream_t st) {
    if (dtype) launch(k_read_kv<bf16_t>, dim3(npos), dim3(256), 0, st, D, (const bf16_t*)cache_layer, seq, which, pos0, npos, out);
    else launch(k_read_kv<float>, dim3(npos), dim3(256), 0, st, D, (const float*)cache_layer, seq, which, pos0, npos, out);
}
