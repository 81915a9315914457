// Stand-alone top-k of the draft heads' logits for rows of more than 4096 (dev_topk has the shorter ones).
#include "accept_dev.h"

// The candidate scheme of dev_topk by 1024 threads of 16 logits: the best entries of the 64 groups of 256 logits are ranked by
// counting, T is the 16th of them, every entry not after T is a candidate (some twenty of them), and a candidate's rank is its place in the list.
// Rows of up to 16 384 logits are read once and stay in registers.  Longer ones, up to 65 536, go slice by slice (64 maxima each),
// and all slices but the last are read again for the candidates.  More than 256 candidates, or logits beyond that: one entry per
// round by re-scanning.
// What bounds it: one trip to memory and six barriers in the four or five workgroups that there are, nothing of the chip's rates
// (16 001 logits, 4 rows, per launch: 256 threads and slices of 4096, two passes, 36.6 us; this 8.8).
__global__ __launch_bounds__(1024) void k_topk(Dims D, DevState s, int seq0) {
    constexpr int PER = 16, SLICE = 1024 * PER, MAX_SLICES = 4, CAND = 256;
    __shared__ float c_v[CAND];
    __shared__ int c_i[CAND];
    __shared__ float t_v;
    __shared__ int t_i, c_n;
    static_assert(MAX_SLICES * 64 <= CAND, "the maxima share the candidates' arrays");
    const int tid = threadIdx.x, i = blockIdx.x, b = seq0 + blockIdx.y, V1 = D.V1;
    const float* z = s.zdraft + ((size_t)i * D.Bmax + b) * V1;
    int32_t* out = s.draft_topk + ((size_t)b * D.Hh + i) * VADUSA_MAX_TOPK;
    const int kmax = min(V1, VADUSA_MAX_TOPK), nsl = (V1 + SLICE - 1) / SLICE;
    // how many of the n entries in c_v, c_i rank before (v, id); eight LDS reads at a time
    auto rank = [&](int n, float v, int id) {
        int r = 0;
        for (int t0 = 0; t0 < n; t0 += 8) {
            float cv[8];
            int ci[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) { cv[q] = c_v[(t0 + q) & (CAND - 1)]; ci[q] = c_i[(t0 + q) & (CAND - 1)]; }
#pragma unroll
            for (int q = 0; q < 8; ++q) r += (t0 + q < n && before(cv[q], ci[q], v, id)) ? 1 : 0;
        }
        return r;
    };
    bool rescan = nsl > MAX_SLICES;
    if (!rescan) {
        float zr[PER];
        auto load = [&](int sl) {
#pragma unroll
            for (int j = 0; j < PER; ++j) zr[j] = ldg(z + min(sl * SLICE + tid + 1024 * j, V1 - 1));   // (an index beyond the row does not count)
        };
        if (tid == 0) { c_n = 0; t_v = -INFINITY; t_i = 0x7fffffff; }   // T without 16 maxima (missing values): keep everything
        for (int sl = 0; sl < nsl; ++sl) {
            load(sl);
            float lv = -INFINITY;
            int li = 0x7fffffff;   // (a group without entries ranks last)
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const int v = sl * SLICE + tid + 1024 * j;
                if (v < V1 && before(zr[j], v, lv, li)) { lv = zr[j]; li = v; }
            }
            row16_argbest(lv, li);
            if ((tid & 15) == 0) { c_v[sl * 64 + (tid >> 4)] = lv; c_i[sl * 64 + (tid >> 4)] = li; }
        }
        __syncthreads();
        // an entry of the row with 15 others before it: the row's 16th best is not after it
        if (tid < nsl * 64 && rank(nsl * 64, c_v[tid], c_i[tid]) == 15) { t_v = c_v[tid]; t_i = c_i[tid]; }
        __syncthreads();
        const float tv = t_v;
        const int ti = t_i;
        for (int sl = nsl - 1; sl >= 0; --sl) {   // the last slice is still in the registers
            if (sl < nsl - 1) load(sl);
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const int v = sl * SLICE + tid + 1024 * j;
                if (v < V1 && !before(tv, ti, zr[j], v)) {
                    const int slot = atomicAdd(&c_n, 1);
                    if (slot < CAND) { c_v[slot] = zr[j]; c_i[slot] = v; }
                }
            }
        }
        __syncthreads();
        const int n = c_n;   // the same for every thread
        rescan = n > CAND;
        if (tid < n && !rescan) {
            const int r = rank(n, c_v[tid], c_i[tid]);
            if (r < kmax) stwi(out + r, c_i[tid]);
        }
    }
    if (rescan) {
        float pv = INFINITY;
        int pi = -1;
        for (int k = 0; k < kmax; ++k) {
            float bv;
            const int bi = block_argbest<16>(z, V1, pv, pi, &bv);
            if (tid == 0) stwi(out + k, bi);
            pv = bv; pi = bi;
        }
    }
}
void launch_topk(const Dims& D, const DevState& s, int seq0, int nseq, hipStream_t st) {
    launch(k_topk, dim3(D.Hh, nseq), dim3(1024), 0, st, D, s, seq0);
}
