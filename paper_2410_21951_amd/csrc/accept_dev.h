// Device functions for verification with tolerance (Algorithm 1), choice of the
// accepted path (Sec. 2.3), continuation from the last accepted node (Sec. 2.1),
// KV compaction and the draft heads' top-k lists.  Each function is the body of
// one workgroup of 256 threads (64 for the compaction); the kernels of both models
// call them.
#pragma once
#include "common.h"

// Total order used everywhere a "largest logit" is needed: value descending,
// then token id ascending.  before(a, b) = a ranks strictly ahead of b.
__device__ __forceinline__ bool before(float va, int ia, float vb, int ib) {
    return va > vb || (va == vb && ia < ib);
}

// Best (value, id) pair of a wave under the order above; every lane gets it.  Inside a row of 16
// lanes by DPP permutations (after each step twice as many lanes agree, so the mirrored partners
// serve as well as the xor partners), across the four rows by the row-swap instructions.
template <int CTRL>
__device__ __forceinline__ void argbest_step(float& bv, int& bi) {
    const float ov = __int_as_float(dpp_perm<CTRL>(__float_as_int(bv)));
    const int oi = dpp_perm<CTRL>(bi);
    if (before(ov, oi, bv, bi)) { bv = ov; bi = oi; }
}
__device__ __forceinline__ void row16_argbest(float& bv, int& bi) {
    argbest_step<0xB1>(bv, bi);
    argbest_step<0x4E>(bv, bi);
    argbest_step<0x141>(bv, bi);
    argbest_step<0x140>(bv, bi);
}
__device__ __forceinline__ void wave_argbest(float& bv, int& bi) {
    row16_argbest(bv, bi);
    {
        const vadusa_u32x2 rv = __builtin_amdgcn_permlane16_swap(__float_as_uint(bv), __float_as_uint(bv), false, false);
        const vadusa_u32x2 ri = __builtin_amdgcn_permlane16_swap((unsigned)bi, (unsigned)bi, false, false);
        const bool x = before(__uint_as_float(rv.x), (int)ri.x, __uint_as_float(rv.y), (int)ri.y);
        bv = __uint_as_float(x ? rv.x : rv.y); bi = (int)(x ? ri.x : ri.y);
    }
    {
        const vadusa_u32x2 rv = __builtin_amdgcn_permlane32_swap(__float_as_uint(bv), __float_as_uint(bv), false, false);
        const vadusa_u32x2 ri = __builtin_amdgcn_permlane32_swap((unsigned)bi, (unsigned)bi, false, false);
        const bool x = before(__uint_as_float(rv.x), (int)ri.x, __uint_as_float(rv.y), (int)ri.y);
        bv = __uint_as_float(x ? rv.x : rv.y); bi = (int)(x ? ri.x : ri.y);
    }
}

// Block-wide arg-best under the order above, restricted to entries that come
// strictly after (pv, pi).  Every thread returns the winner.  64 NW threads, each with PER loads on their way at once: a round
// is one trip to the L2 (k_continue with four and with 16 loads per round, us per launch: 16 001 logits 12.3 -> 10.9; 1025 logits 6.4 either way).
// Loads are unconditional; an index beyond the row re-reads its last entry and does not count.
template <int NW, int PER>
__device__ inline void argbest_scan(const float* __restrict__ z, int n, float pv, int pi, float& bv, int& bi) {
    for (int v0 = threadIdx.x; v0 < n; v0 += 64 * NW * PER) {
        float zv[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) zv[j] = ldg(z + min(v0 + 64 * NW * j, n - 1));
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int v = v0 + 64 * NW * j;
            if (v < n && before(pv, pi, zv[j], v) && before(zv[j], v, bv, bi)) { bv = zv[j]; bi = v; }
        }
    }
}
template <int NW = 4>
__device__ inline int block_argbest(const float* __restrict__ z, int n, float pv, int pi, float* best_val) {
    __shared__ float sv[NW];
    __shared__ int si[NW];
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    if (n <= 64 * NW * 8) argbest_scan<NW, 8>(z, n, pv, pi, bv, bi);
    else argbest_scan<NW, 16>(z, n, pv, pi, bv, bi);
    wave_argbest(bv, bi);
    __syncthreads();   // protects sv/si against the previous call's readers
    if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = bv; si[threadIdx.x >> 6] = bi; }
    __syncthreads();
    bv = sv[0]; bi = si[0];
    for (int w = 1; w < NW; ++w) if (before(sv[w], si[w], bv, bi)) { bv = sv[w]; bi = si[w]; }
    if (bi == 0x7fffffff) bi = 0;   // no entry qualifies (a row of NaN): still an index of the row
    if (best_val) *best_val = bv;
    return bi;
}

// Algorithm 1, one edge: node n of sequence b is accepted iff fewer than tau entries of its
// parent's logit row rank before its token.  NW waves, of which this thread is number t0; returns this wave's count of such entries.
template <int NW>
__device__ inline int dev_edge_count(const Dims& D, const DevState& s, int b, int n, int t0) {
    const float* z = s.logits + ((size_t)b * D.M + s.t_parent[0][n]) * D.V1;
    const int t = s.tok[(size_t)b * D.M + n];
    const float zt = z[t];
    int cnt = 0;
    for (int v0 = t0; v0 < D.V1; v0 += 64 * NW * 17) {
        float zv[17];
#pragma unroll
        for (int q = 0; q < 17; ++q) zv[q] = v0 + 64 * NW * q < D.V1 ? z[v0 + 64 * NW * q] : -INFINITY;
#pragma unroll
        for (int q = 0; q < 17; ++q) cnt += (v0 + 64 * NW * q < D.V1 && before(zv[q], v0 + 64 * NW * q, zt, t)) ? 1 : 0;
    }
    return wave_sum_i_dpp(cnt);
}

// An accepted path in LDS: number of nodes, the nodes and their tokens.
struct PathLds { int cnt, node[VADUSA_MAX_DRAFT_HEADS + 1], tok[VADUSA_MAX_DRAFT_HEADS + 1]; };

// Sec. 2.3's choice for sequence b from the edge decisions in edge_ok (k_edges, k_edges_wide): a node is accepted iff every edge from the root to
// it is; the chosen one is the deepest, smallest index among equals (canonical order = leftmost).  Cut after the first EOS.
// Output: p, and path[b] = {count, node indices...} in memory for the compaction.  256 threads; everything it reads from memory is
// asked for at once, and what the walks need sits in LDS (a step's chain of dependent loads is what bounds it).
__device__ inline void dev_select(const Dims& D, const DevState& s, int b, int ignore_eos, PathLds& p) {
    __shared__ int s_par[VADUSA_MAX_TREE_NODES], s_edge[VADUSA_MAX_TREE_NODES], s_tok[VADUSA_MAX_TREE_NODES], s_key[2];
    const int n = threadIdx.x;
    const bool node = n < D.M;
    const int fin = ldg(s.finished + b);
    int par = 0, dep = 0, edge = 0, tok = 0;
    if (node) {
        par = ldg(s.t_parent[0] + n);
        dep = ldg(s.t_depth[0] + n);
        tok = ldg(s.tok + (size_t)b * D.M + n);
        edge = D.M > 1 ? ldg(s.edge_ok + (size_t)b * D.M + n) : !fin;   // (a tree of the root alone has no edge to test)
        if (D.M == 1) s.edge_ok[b] = edge;
        s_par[n] = par;
        s_edge[n] = edge;
        s_tok[n] = tok;
    }
    __syncthreads();
    int key = -1;   // deepest accepted node, smallest index among equals: largest depth * 256 + (255 - n)
    if (node) {
        int ok = 1, m = n;
        while (m > 0) { ok &= s_edge[m]; m = s_par[m]; }
        if (ok) key = dep * 256 + (255 - n);
    }
    if (n < VADUSA_MAX_TREE_NODES) {   // (two waves)
        key = max(key, dpp_perm<0xB1>(key));
        key = max(key, dpp_perm<0x4E>(key));
        key = max(key, dpp_perm<0x141>(key));
        key = max(key, dpp_perm<0x140>(key));
        key = max(max(__builtin_amdgcn_readlane(key, 0), __builtin_amdgcn_readlane(key, 16)), max(__builtin_amdgcn_readlane(key, 32), __builtin_amdgcn_readlane(key, 48)));
        if ((n & 63) == 0) s_key[n >> 6] = key;
    }
    __syncthreads();
    if (n == 0) {
        key = max(s_key[0], s_key[1]);
        int32_t* path = s.path + (size_t)b * (VADUSA_MAX_DRAFT_HEADS + 2);
        int cnt = fin ? 0 : (key < 0 ? 0 : key >> 8) + 1, m = key < 0 ? 0 : 255 - (key & 255);
        for (int j = cnt - 1; j >= 0; --j) { p.node[j] = m; p.tok[j] = s_tok[m]; m = s_par[m]; }
        if (!ignore_eos)
            for (int j = 0; j < cnt; ++j)
                if (p.tok[j] == D.V1 - 1) { cnt = j + 1; break; }
        for (int j = 0; j < cnt; ++j) path[1 + j] = p.node[j];
        path[0] = cnt;
        p.cnt = cnt;
    }
    __syncthreads();
}

// The path of sequence b that waits in memory (chosen earlier, or forced by the caller).
__device__ inline void dev_load_path(const Dims& D, const DevState& s, int b, PathLds& p) {
    const int32_t* path = s.path + (size_t)b * (VADUSA_MAX_DRAFT_HEADS + 2);
    const int j = threadIdx.x;
    if (j <= VADUSA_MAX_DRAFT_HEADS) {
        const int cnt = ldg(path), m = ldg(path + 1 + j);
        if (j < cnt) { p.node[j] = m; p.tok[j] = ldg(s.tok + (size_t)b * D.M + m); }
        if (j == 0) p.cnt = cnt;
    }
    __syncthreads();
}

// Continue from the last accepted node (Sec. 2.1): advance L, append the
// accepted tokens to the output, next root = best logit of that node's row, and
// its final-LayerNorm'd hidden state for the draft heads (operand tiles in the bf16 model).  acc_len[b] keeps the number
// of committed rows for the compaction that follows.  In prefill mode the
// "path" is the chunk's last row and nothing is emitted (p is not read).  host (or null): where the caller wants the results, laid out like
// the block that starts at kerr (after a prefill: the error word and the first roots).
template <class T>
__device__ inline void dev_finalize(const Dims& D, const DevState& s, int b, int prefill_mode, int ignore_eos, const PathLds& p, int32_t* host) {
    __shared__ float s_red[8];
    constexpr int W = VADUSA_MAX_DRAFT_HEADS + 1;
    const int cnt = prefill_mode ? ldg(s.n_rows + b) : p.cnt;
    const int L = ldg(s.L + b), no = prefill_mode ? 0 : ldg(s.n_out + b), old_root = ldg(s.root + b);
    if (host && b == 0 && threadIdx.x < 4) host[threadIdx.x] = ldg(s.kerr + threadIdx.x);
    if (threadIdx.x == 0) s.acc_len[b] = prefill_mode ? 0 : cnt;
    if (cnt <= 0) {
        if (host && !prefill_mode && threadIdx.x == 0) { host[4 + b] = 0; host[4 + D.Bmax + b] = L; host[4 + 2 * D.Bmax + b] = old_root; }
        return;
    }
    const int last = prefill_mode ? cnt - 1 : p.node[cnt - 1];
    const int r = prefill_mode && D.last_only ? b : (prefill_mode && s.row0 ? ldg(s.row0 + b) : b * D.M) + last;
    // final LayerNorm of the accepted node's residual row: read once, into registers (up to 16 values per
    // thread, d <= 4096; larger rows take the three-pass route below), ahead of the row of logits
    const float* xr = s.x + (size_t)r * D.d;
    float xv[16], gv[16], bv[16];
    if (D.d <= 4096) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = threadIdx.x * 2 + 512 * j;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                xv[2 * j + q] = i < D.d ? ldg(xr + i + q) : 0.f;
                gv[2 * j + q] = i < D.d ? ldg(s.lnf_g + i + q) : 0.f;
                bv[2 * j + q] = i < D.d ? ldg(s.lnf_b + i + q) : 0.f;
            }
        }
    }
    const int root = block_argbest(s.logits + (size_t)r * D.V1, D.V1, INFINITY, -1, nullptr);
    if (threadIdx.x == 0) {
        s.root[b] = root;
        s.L[b] = L + cnt;
        if (host && prefill_mode) host[4 + b] = root;
        if (!prefill_mode) {
            bool fin = false;
            for (int j = 0; j < cnt; ++j) {
                const int t = p.tok[j];
                s.acc_tok[b * W + j] = t;
                if (no + j < D.maxpos) s.out_tok[(size_t)b * D.maxpos + no + j] = t;
                if (t == D.V1 - 1) fin = true;
                if (host) host[4 + 3 * D.Bmax + b * W + j] = t;
            }
            s.n_out[b] = min(no + cnt, max(no, D.maxpos));
            s.path[(size_t)b * (VADUSA_MAX_DRAFT_HEADS + 2)] = 0;   // consumed
            if (fin && !ignore_eos) s.finished[b] = 1;
            if (host) { host[4 + b] = cnt; host[4 + D.Bmax + b] = L + cnt; host[4 + 2 * D.Bmax + b] = root; }
        }
    }
    auto store = [&](int i, float a, float c) {
        if constexpr (sizeof(T) == 4) *(float2*)((float*)s.hbest + (size_t)b * D.d + i) = make_float2(a, c);
        else *(uint32_t*)((bf16_t*)s.hbest + toff(b, i, D.d >> 5)) = pack_bf16(a, c);   // tiled for the draft maps
    };
    if (D.d <= 4096) {
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) sum += xv[2 * j] + xv[2 * j + 1];
        sum = wave_sum_dpp(sum);
        if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = sum;
        __syncthreads();
        const float mu = (s_red[0] + s_red[1] + s_red[2] + s_red[3]) / D.d;
        float sq = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = threadIdx.x * 2 + 512 * j;
            if (i < D.d) { const float t0 = xv[2 * j] - mu, t1 = xv[2 * j + 1] - mu; sq += t0 * t0 + t1 * t1; }
        }
        sq = wave_sum_dpp(sq);
        if ((threadIdx.x & 63) == 0) s_red[4 + (threadIdx.x >> 6)] = sq;
        __syncthreads();
        const float rstd = rsqrtf((s_red[4] + s_red[5] + s_red[6] + s_red[7]) / D.d + LN_EPS);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = threadIdx.x * 2 + 512 * j;
            if (i < D.d) store(i, (xv[2 * j] - mu) * rstd * gv[2 * j] + bv[2 * j], (xv[2 * j + 1] - mu) * rstd * gv[2 * j + 1] + bv[2 * j + 1]);
        }
    } else {
        float sum = 0.f;
        for (int i = threadIdx.x; i < D.d; i += 256) sum += ldg(xr + i);
        sum = wave_sum_dpp(sum);
        if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = sum;
        __syncthreads();
        const float mu = (s_red[0] + s_red[1] + s_red[2] + s_red[3]) / D.d;
        float sq = 0.f;
        for (int i = threadIdx.x; i < D.d; i += 256) { const float t = ldg(xr + i) - mu; sq += t * t; }
        sq = wave_sum_dpp(sq);
        if ((threadIdx.x & 63) == 0) s_red[4 + (threadIdx.x >> 6)] = sq;
        __syncthreads();
        const float rstd = rsqrtf((s_red[4] + s_red[5] + s_red[6] + s_red[7]) / D.d + LN_EPS);
        for (int i = threadIdx.x * 2; i < D.d; i += 512)
            store(i, (ldg(xr + i) - mu) * rstd * s.lnf_g[i] + s.lnf_b[i], (ldg(xr + i + 1) - mu) * rstd * s.lnf_g[i + 1] + s.lnf_b[i + 1]);
    }
}

// KV compaction after dev_finalize, nl consecutive layers from layer0 on: cache row L0 + j <- row L0 + path[j], where
// L0 = L - acc_len is the length before this step and acc_len the number of
// committed rows.  path[j] >= j, so a destination row can be the source of an
// earlier j: every thread owns one column of one head and reads all its sources
// before writing.  64 threads (one per head dimension).  The path is read once; four layers' rows are in flight
// together; a path whose rows already sit where they belong (the root alone, or nodes 0, 1, .. of the tree) moves nothing.
template <class T>
__device__ inline void dev_commit_kv_layers(const Dims& D, const DevState& s, int layer0, int nl, int b, int head, int dim) {
    constexpr int W = VADUSA_MAX_DRAFT_HEADS + 1, LB = 4;
    const int32_t* path = s.path + (size_t)b * (VADUSA_MAX_DRAFT_HEADS + 2);
    const int cnt = ldci(s.acc_len + b);
    if (cnt <= 0) return;
    const int L0 = ldci(s.L + b) - cnt;
    int src[W];
    bool moves = false;
#pragma unroll
    for (int j = 0; j < W; ++j) {
        src[j] = j < cnt ? ldci(path + 1 + j) : j;
        moves |= src[j] != j;
    }
    if (!moves) return;
    size_t so_k[W], so_v[W], do_k[W], do_v[W];
#pragma unroll
    for (int j = 0; j < W; ++j) {
        so_k[j] = kc_off(L0 + src[j], dim); so_v[j] = vc_off(L0 + src[j], dim);
        do_k[j] = kc_off(L0 + j, dim); do_v[j] = vc_off(L0 + j, dim);
    }
    const size_t lstride = (size_t)D.Bmax * D.nH * kv_cap(D.maxpos) * 64;
    const size_t hb0 = ((((size_t)layer0 * D.Bmax + b) * D.nH + head) * kv_cap(D.maxpos)) * 64;
    for (int l0 = 0; l0 < nl; l0 += LB) {
        T kr[LB][W], vr[LB][W];
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            const size_t hb = hb0 + (size_t)(l0 + i < nl ? l0 + i : nl - 1) * lstride;
            const T* Kh = (const T*)s.Kc + hb;
            const T* Vh = (const T*)s.Vc + hb;
#pragma unroll
            for (int j = 0; j < W; ++j)
                if (j < cnt) { kr[i][j] = Kh[so_k[j]]; vr[i][j] = Vh[so_v[j]]; }
        }
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            if (l0 + i >= nl) break;
            const size_t hb = hb0 + (size_t)(l0 + i) * lstride;
            T* Kh = (T*)s.Kc + hb;
            T* Vh = (T*)s.Vc + hb;
#pragma unroll
            for (int j = 0; j < W; ++j)
                if (j < cnt) { Kh[do_k[j]] = kr[i][j]; Vh[do_v[j]] = vr[i][j]; }
        }
    }
}

// Draft list of head i, sequence b: the VADUSA_MAX_TOPK best ids of its logits,
// descending, equal logits: lower id first (Sec. 2.1).
// Up to 4096 logits sit in registers (16 per thread).  The 256 threads form 64 quads; the 64
// quad maxima are distinct entries of the row, so the row's 16th best entry is not after the
// 16th best of them, T.  Every entry not after T is a candidate (two dozen for random logits);
// each candidate counts the candidates before it, which is its place in the list.
// More than 256 candidates (many equal or missing values): the list is built one entry per round by
// re-scanning (block_argbest).  Rows of more than 4096 logits are k_topk's.
__device__ inline void dev_topk(const Dims& D, const DevState& s, int i, int b) {
    __shared__ float c_v[256];
    __shared__ int c_i[256];
    __shared__ float g_v[64];
    __shared__ int g_i[64];
    __shared__ int c_n;
    __shared__ float t_v;
    __shared__ int t_i;
    const float* z = s.zdraft + ((size_t)i * D.Bmax + b) * D.V1;
    int32_t* out = s.draft_topk + ((size_t)b * D.Hh + i) * VADUSA_MAX_TOPK;
    const int kmax = D.V1 < VADUSA_MAX_TOPK ? D.V1 : VADUSA_MAX_TOPK;
    bool rescan = false;
    {
        float zr[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int v = threadIdx.x + 256 * j;
            zr[j] = v < D.V1 ? ldg(z + v) : -INFINITY;
        }
        float lv = -INFINITY;
        int li = 0x7fffffff;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int v = threadIdx.x + 256 * j;
            if (v < D.V1 && before(zr[j], v, lv, li)) { lv = zr[j]; li = v; }
        }
        // best of each quad: 64 group maxima (fewer for fewer than 253 logits; empty groups leave
        // (-inf, 0x7fffffff), which ranks after every real entry)
        argbest_step<0xB1>(lv, li);
        argbest_step<0x4E>(lv, li);
        if ((threadIdx.x & 3) == 0) { g_v[threadIdx.x >> 2] = lv; g_i[threadIdx.x >> 2] = li; }
        if (threadIdx.x == 0) { c_n = 0; t_v = -INFINITY; t_i = 0x7fffffff; }   // default T: keep everything
        __syncthreads();
        // T = the 16th best of the group maxima: an entry of the row with at least 15 others before
        // it, so the row's 16th best is not after T.  Wave 0 ranks the 64 maxima against each other
        // with lane broadcasts (no LDS traffic in the loop).  With fewer than 16 real maxima T stays
        // at its default.
        if (threadIdx.x < 64 && D.V1 >= 64) {
            const float gv = g_v[threadIdx.x];
            const int gi = g_i[threadIdx.x];
            int r = 0;
            for (int j = 0; j < 64; ++j) {
                const float bv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(gv), j));
                const int bi = __builtin_amdgcn_readlane(gi, j);
                r += before(bv, bi, gv, gi) ? 1 : 0;
            }
            if (r == 15) { t_v = gv; t_i = gi; }
        }
        __syncthreads();
        const float tv = t_v;
        const int ti = t_i;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int v = threadIdx.x + 256 * j;
            if (v < D.V1 && !before(tv, ti, zr[j], v)) {
                const int slot = atomicAdd(&c_n, 1);
                if (slot < 256) { c_v[slot] = zr[j]; c_i[slot] = v; }
            }
        }
        __syncthreads();
        const int n = c_n;
        if (n <= 64) {
            // the usual case (a few dozen candidates): wave 0 holds one candidate per lane and ranks
            // them against each other with lane broadcasts; a candidate's rank is its place in the list
            if (threadIdx.x < 64) {
                const bool have = (int)threadIdx.x < n;
                const float mv = have ? c_v[threadIdx.x] : -INFINITY;
                const int mi = have ? c_i[threadIdx.x] : 0x7fffffff;
                int r = 0;
                for (int j = 0; j < n; ++j) {
                    const float bv = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mv), j));
                    const int bi = __builtin_amdgcn_readlane(mi, j);
                    r += before(bv, bi, mv, mi) ? 1 : 0;
                }
                if (have && r < kmax) stwi(out + r, mi);
            }
        } else if (n <= 256) {
            if ((int)threadIdx.x < n) {
                const float mv = c_v[threadIdx.x];
                const int mi = c_i[threadIdx.x];
                int r = 0;
                for (int t0 = 0; t0 < n; t0 += 8) {   // eight candidates per round: LDS reads overlap
                    float cv[8];
                    int ci[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) { cv[q] = c_v[(t0 + q) & 255]; ci[q] = c_i[(t0 + q) & 255]; }
#pragma unroll
                    for (int q = 0; q < 8; ++q) r += (t0 + q < n && before(cv[q], ci[q], mv, mi)) ? 1 : 0;
                }
                if (r < kmax) stwi(out + r, mi);
            }
        } else {
            rescan = true;   // n is the same for every thread
        }
        __syncthreads();     // the LDS arrays are free again
    }
    if (rescan) {
        float pv = INFINITY;
        int pi = -1;
        for (int k = 0; k < kmax; ++k) {
            float bv;
            const int bi = block_argbest(z, D.V1, pv, pi, &bv);
            if (threadIdx.x == 0) stwi(out + k, bi);
            pv = bv; pi = bi;
        }
    }
}
