// Perturbed scores for the stochastic form of Algorithm 1 (tau tokens drawn per position from
// the nucleus of the temperature-scaled distribution, Sec. 3.1.2).
// For one logit row z and uniforms u: s = z / temperature; the nucleus keeps token v iff the
// tokens with a strictly larger s hold less than top_p of softmax(s), or fewer than tau tokens
// have a strictly larger s (so tau draws always exist); score = s - log(-log u) on kept tokens,
// -inf elsewhere.  Ordering a row's scores lists its tokens in the order successive draws
// without replacement would produce them, so the deterministic ranking kernels applied to the
// scores give Algorithm 1's "candidate is among the tau draws" and the first draw.
#include "common.h"

// Monotone map float -> uint32: a < b  <=>  key(a) < key(b) (no NaN expected).
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t b = __float_as_uint(f);
    return b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
}

// The kept set is {v : s_v >= s*}; s* is found by a search over the 32-bit keys of the predicate "the tokens above this key hold less
// than top_p, or are fewer than tau", which is monotone in the key and changes only at values that occur in the row.

// Rows of up to 4096 logits: one WAVE per row, the row in registers (values of lane l: l, l + 64, ...), no LDS
// and no workgroup barrier.  A plain bisection over the 32-bit keys: a round is a
// compare and two conditional adds per value and two wave sums by lane permutations.  The values are kept as their
// keys (key_value gives a value back), entries beyond the row have key 0 (below every key) and mass 0.
__device__ __forceinline__ float key_value(uint32_t k) { return __uint_as_float(k ^ ((k >> 31) ? 0x80000000u : 0xffffffffu)); }
__device__ __forceinline__ float wave_max_dpp(float v) {
    v = fmaxf(v, __int_as_float(dpp_perm<0xB1>(__float_as_int(v))));
    v = fmaxf(v, __int_as_float(dpp_perm<0x4E>(__float_as_int(v))));
    v = fmaxf(v, __int_as_float(dpp_perm<0x141>(__float_as_int(v))));
    v = fmaxf(v, __int_as_float(dpp_perm<0x140>(__float_as_int(v))));
    return fmaxf(fmaxf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0)), __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16))),
                 fmaxf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32)), __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48))));
}
__device__ __forceinline__ uint32_t wave_umax_dpp(uint32_t v) {
    v = max(v, (uint32_t)dpp_perm<0xB1>((int)v));
    v = max(v, (uint32_t)dpp_perm<0x4E>((int)v));
    v = max(v, (uint32_t)dpp_perm<0x141>((int)v));
    v = max(v, (uint32_t)dpp_perm<0x140>((int)v));
    return max(max((uint32_t)__builtin_amdgcn_readlane((int)v, 0), (uint32_t)__builtin_amdgcn_readlane((int)v, 16)),
               max((uint32_t)__builtin_amdgcn_readlane((int)v, 32), (uint32_t)__builtin_amdgcn_readlane((int)v, 48)));
}
template <int GROUPS>   // groups of four 64-value chunks the row may have: GROUPS * 256 >= V1
__global__ __launch_bounds__(64) void k_perturb_wave(const float* __restrict__ logits, const float* __restrict__ u,
                                                     float* __restrict__ scores, int V1, float temperature, float top_p, int tau) {
    const size_t row = blockIdx.x;
    const int lane = threadIdx.x;
    const float* z = logits + row * V1;
    const float* ur = u + row * V1;
    float* y = scores + row * V1;
    float e[GROUPS][4];
    uint32_t key[GROUPS][4];
    float zv[GROUPS][4], gum[GROUPS][4];
    // logits and uniforms are asked for together (one memory latency, not one before and one after the search)
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int v = g * 256 + q * 64 + lane;
            zv[g][q] = v < V1 ? z[v] : 0.f;
            gum[g][q] = v < V1 ? ur[v] : 0.5f;
        }
    float m = -INFINITY, mn = INFINITY;
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int v = g * 256 + q * 64 + lane;
            const float sv = v < V1 ? zv[g][q] / temperature + 0.f : -INFINITY;   // -0 becomes +0: equal values, equal keys
            gum[g][q] = logf(-logf(gum[g][q]));
            key[g][q] = v < V1 ? order_key(sv) : 0u;
            m = fmaxf(m, sv);
            mn = fminf(mn, v < V1 ? sv : INFINITY);
        }
    m = wave_max_dpp(m);
    uint32_t kmin = 0;   // keep everything
    if (top_p < 1.f) {
        float zsum = 0.f;
#pragma unroll
        for (int g = 0; g < GROUPS; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                e[g][q] = g * 256 + q * 64 + lane < V1 ? expf(key_value(key[g][q]) - m) : 0.f;
                zsum += e[g][q];
            }
        const float target = top_p * wave_sum_dpp(zsum);
        // The search runs between the row's smallest and largest key: the predicate holds at the largest (nothing
        // lies above it), and below the smallest it is what it is at the smallest minus one (everything above), so a
        // result below the smallest key would keep the same tokens as the smallest key itself.  The answer is a key
        // of the row whenever the predicate fails just below the interval (it changes only at keys that occur), so
        // once the predicate has failed somewhere (lo has moved) and a single entry of the row is left in [lo, hi],
        // that entry's key is the answer: with ~1000 logits some 15 rounds instead of 32.
        uint32_t lo = order_key(-wave_max_dpp(-mn)), hi = order_key(m);
        // entries at or above lo and entries above hi, known from the rounds that set lo and hi: their difference is
        // the number of entries left in [lo, hi] (no count of its own per round)
        int c_lo = V1, c_hi = 0;
        bool failed = false;
        while (lo < hi) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            float a4[4] = {0.f, 0.f, 0.f, 0.f};   // four independent partial sums: no chain of dependent additions
            int c4[4] = {0, 0, 0, 0};
#pragma unroll
            for (int g = 0; g < GROUPS; ++g)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool above = key[g][q] > mid;
                    a4[q] += above ? e[g][q] : 0.f;
                    c4[q] += above ? 1 : 0;
                }
            const float A = wave_sum_dpp((a4[0] + a4[1]) + (a4[2] + a4[3]));
            const int C = wave_sum_i_dpp((c4[0] + c4[1]) + (c4[2] + c4[3]));
            if (A < target || C < tau) { hi = mid; c_hi = C; }
            else { lo = mid + 1; c_lo = C; failed = true; }
            if (failed && c_lo - c_hi == 1) {   // one entry left: its key (every other lane contributes 0)
                uint32_t kin = 0;
#pragma unroll
                for (int g = 0; g < GROUPS; ++g)
#pragma unroll
                    for (int q = 0; q < 4; ++q) kin = (key[g][q] >= lo && key[g][q] <= hi) ? key[g][q] : kin;
                hi = (uint32_t)wave_sum_i_dpp((int)kin);
                break;
            }
        }
        kmin = hi;
    }
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int v = g * 256 + q * 64 + lane;
            if (v < V1) y[v] = key[g][q] >= kmin ? key_value(key[g][q]) - gum[g][q] : -INFINITY;
        }
}

// Rows of more than 4096 logits: the same by a workgroup of 1024 threads per row, the row in registers (entries of thread t: t, t + 1024, ...;
// PER of them), so up to 16 384 logits.  A round of the bisection is three instructions per value, a wave's two sums by lane
// permutations, 16 pairs through LDS (two sets in turn: one barrier) and their sum in the same order by every thread, so that lo and
// hi are the same everywhere.  The smallest and the largest key are taken as keys: with missing values among the logits the interval still
// holds every key of the row.
// What bounds it: some 17 rounds one after the other, each a reduction and a barrier, behind one trip to memory (64 rows of
// 16 001, us per launch: 256 threads, the row in LDS, 15 keys per round and the exponentials anew in each 171; this 34).
template <int PER>
__global__ __launch_bounds__(1024) void k_perturb_block(const float* __restrict__ logits, const float* __restrict__ u,
                                                        float* __restrict__ scores, int V1, float temperature, float top_p, int tau) {
    constexpr int NW = 16;
    __shared__ float s_f[2][NW];
    __shared__ int s_i[2][NW];
    __shared__ uint32_t s_lo[NW], s_hi[NW], s_last;
    const size_t row = blockIdx.x;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const float* z = logits + row * V1;
    const float* ur = u + row * V1;
    float* y = scores + row * V1;
    float gum[PER], e[PER];
    uint32_t key[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {   // logits and uniforms together; an index beyond the row re-reads its last entry
        e[j] = ldg(z + min(tid + 1024 * j, V1 - 1));
        gum[j] = ldg(ur + min(tid + 1024 * j, V1 - 1));
    }
    float m = -INFINITY;
    uint32_t lo = 0xffffffffu, hi = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const bool have = tid + 1024 * j < V1;
        const float sv = have ? e[j] / temperature + 0.f : -INFINITY;   // -0 becomes +0: equal values, equal keys
        gum[j] = logf(-logf(gum[j]));
        key[j] = have ? order_key(sv) : 0u;   // (below every key, and no mass)
        m = fmaxf(m, sv);
        lo = min(lo, have ? key[j] : 0xffffffffu);
        hi = max(hi, key[j]);
    }
    uint32_t kmin = 0;   // keep everything
    if (top_p < 1.f) {
        m = wave_max_dpp(m);
        hi = wave_umax_dpp(hi);
        lo = ~wave_umax_dpp(~lo);
        if (lane == 0) { s_f[0][wave] = m; s_lo[wave] = lo; s_hi[wave] = hi; }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) { m = fmaxf(m, s_f[0][w]); lo = min(lo, s_lo[w]); hi = max(hi, s_hi[w]); }
        // sums over the row by every thread; `set` is not the one of the call before
        auto block_sums = [&](int set, float a, int c, float& A, int& C) {
            a = wave_sum_dpp(a);
            c = wave_sum_i_dpp(c);
            if (lane == 0) { s_f[set][wave] = a; s_i[set][wave] = c; }
            __syncthreads();
            float av[NW];
            C = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) { av[w] = s_f[set][w]; C += s_i[set][w]; }
#pragma unroll
            for (int n = NW / 2; n; n >>= 1)
#pragma unroll
                for (int w = 0; w < n; ++w) av[w] += av[w + n];
            A = av[0];
        };
        float zs[4] = {0.f, 0.f, 0.f, 0.f}, zsum;
        int none;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            e[j] = tid + 1024 * j < V1 ? expf(key_value(key[j]) - m) : 0.f;
            zs[j & 3] += e[j];
        }
        block_sums(1, (zs[0] + zs[1]) + (zs[2] + zs[3]), 0, zsum, none);
        const float target = top_p * zsum;
        // (the search and its early end: as in k_perturb_wave)
        int c_lo = V1, c_hi = 0, set = 0;
        bool failed = false;
        while (lo < hi) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            float a4[4] = {0.f, 0.f, 0.f, 0.f}, A;
            int c4[4] = {0, 0, 0, 0}, C;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const bool above = key[j] > mid;
                a4[j & 3] += above ? e[j] : 0.f;
                c4[j & 3] += above ? 1 : 0;
            }
            block_sums(set, (a4[0] + a4[1]) + (a4[2] + a4[3]), (c4[0] + c4[1]) + (c4[2] + c4[3]), A, C);
            set ^= 1;
            if (A < target || C < tau) { hi = mid; c_hi = C; }
            else { lo = mid + 1; c_lo = C; failed = true; }
            if (failed && c_lo - c_hi == 1) {   // one entry left: its key
#pragma unroll
                for (int j = 0; j < PER; ++j)
                    if (tid + 1024 * j < V1 && key[j] >= lo && key[j] <= hi) s_last = key[j];
                __syncthreads();
                hi = s_last;
                break;
            }
        }
        kmin = hi;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int v = tid + 1024 * j;
        if (v < V1) y[v] = key[j] >= kmin ? key_value(key[j]) - gum[j] : -INFINITY;
    }
}

// (V1 <= 16 384: vadusa_step and vadusa_verify refuse the stochastic rule for larger vocabularies)
void launch_perturb(const float* logits, const float* u, float* scores, int rows, int V1, float temperature,
                    float top_p, int tau, hipStream_t st) {
    if (V1 <= 1280) launch(k_perturb_wave<5>, dim3(rows), dim3(64), 0, st, logits, u, scores, V1, temperature, top_p, tau);
    else if (V1 <= 2304) launch(k_perturb_wave<9>, dim3(rows), dim3(64), 0, st, logits, u, scores, V1, temperature, top_p, tau);
    else if (V1 <= 4096) launch(k_perturb_wave<16>, dim3(rows), dim3(64), 0, st, logits, u, scores, V1, temperature, top_p, tau);
    else if (V1 <= 8192) launch(k_perturb_block<8>, dim3(rows), dim3(1024), 0, st, logits, u, scores, V1, temperature, top_p, tau);
    else launch(k_perturb_block<16>, dim3(rows), dim3(1024), 0, st, logits, u, scores, V1, temperature, top_p, tau);
}
