// The decoder layers of the bf16 model, one launch per map: embedding, then per layer QKV, attention,
// out-projection, FFN1 and FFN2, and the vocabulary map at the end (Sec. 2.1's tree-verify forward).
//
// Why launches and not one persistent kernel: on this GPU a launch that waits for the one before it costs 2.3 to
// 2.8 us from end to end (chain of 256-workgroup kernels that read what the previous one wrote; host side 2.6 us,
// less than a map takes), which is what a grid barrier with the write-through stores it needs cost inside one kernel
// (1.6 us + 0.9 us of acknowledgement).  Between launches the caches are made coherent by the hardware, so results
// are stored and read as ordinary memory, every map has a kernel with the registers and workgroups per compute unit
// that suit it, and operand addresses come straight from the kernel arguments.
//
// LayerNorm is folded into the map that follows it:
//   LN(x) W^T = rstd * (x (g*W)^T - mu * colsum(g*W)) + (beta W^T + bias),
// so a map reads the bf16 copy of the raw residual stream and applies the row statistics in its epilogue.  The
// statistics come from whoever wrote the residual stream (exact fp32 values, per group of 16, 32 or 64 columns,
// [row][group]) and are merged by the consumer: mean of the group means; squared deviations = the groups' own plus
// their columns x the spread of the group means, summed as distances from the row's first group mean.  No atomics
// combine data: results are bit-reproducible.
#include <algorithm>
#include <type_traits>

#include "accept_dev.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// The compiler moves no instruction across a fence, and waits for a value at the place where it is declared arrived.
#if defined(__HIP_DEVICE_COMPILE__)
#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
#define ARRIVED(v) asm volatile("" : "+v"(v))
#else
#define SCHED_FENCE() ((void)0)
#define ARRIVED(v) ((void)0)
#endif

enum { LE_QKV = 0, LE_GELU, LE_LOGITS, LE_RESID, LE_SILU, LE_F32 };   // LE_SILU, LE_F32: first and second map of the draft heads

__device__ __forceinline__ uint32_t mulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }

// Lines of weights that a later launch will read, brought into the L2s ahead of it by workgroups of a launch that leaves compute units idle: of each
// group of column tiles, which workgroups of XCD (group mod 8) read, `take` pieces of 64 lines.  Lines that have only been read stay in the L2 from
// launch to launch (32 KiB by one wave per compute unit: 1060 clocks from the own L2, 2880 from the memory-side cache or where another XCD has
// read them, 3440 from HBM); without this the memory has nothing to do between two maps' loads: while a launch ends and the next starts (1.3 us),
// while it finds its operands, adds and stores.  us per step, without and with it: 1 node 279 -> 261, 16 nodes 306 -> 274, 64 nodes 331 -> 319, 128 nodes
// and 2000 keys 449 -> 429, 5 sequences of 27 nodes 437 -> 424, 8 of 64 674 -> 676 (d = 1024); d = 768: 226 -> 224, 244 -> 238, 278 -> 275, 389 -> 375, 333 -> 327; d = 640,
// 512 and 256: within 1.5 % either way.  Idle is a compute unit that this launch leaves so: work of other streams and contexts on the GPU shares the memory with these loads.
struct Touch {
    const char* p;          // first piece of the first group
    uint32_t stride, last;  // bytes from a group to the next; from a group's first piece to its last line
    uint32_t take, magic;   // ceil(2^32 / take)
    int groups;
};
template <int N> struct TouchList { Touch map[N]; };
__device__ __forceinline__ int touch_pieces(const Touch& m, int xcd) { return ((m.groups - xcd + 7) >> 3) * (int)m.take; }   // of each map, for this XCD
__device__ __forceinline__ const char* touch_line(const Touch& m, int xcd, int piece, int lane) {
    const uint32_t g = m.take == 1 ? (uint32_t)piece : mulhi((uint32_t)piece, m.magic), part = (uint32_t)piece - g * m.take;
    return m.p + (size_t)(g * 8 + xcd) * m.stride + min(part * 8192u + (uint32_t)lane * 128u, m.last);
}
// By the workgroups from column `first` on of a grid whose columns are whole groups of eight behind it, NW waves each, one lane per line.  (One load of a
// wave on its way at a time: four are no faster.)  nz maps of each shape, z_w[i] bytes from one to the next.
template <int NW, int N>
__device__ __forceinline__ void touch(const TouchList<N>& t, int first, int nz, const size_t* z_w) {
    const int xcd = blockIdx.x & 7, lane = threadIdx.x & 63, each = ((int)gridDim.x - first) >> 3, nw = each * gridDim.y * NW;
    const int w = (int)(blockIdx.y * each + ((blockIdx.x - first) >> 3)) * NW + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#pragma unroll
    for (int m = 0; m < N; ++m) {
        const int n = touch_pieces(t.map[m], xcd);
        for (int z = 0, i = w; z < nz; ++z, i -= n)
            for (; i < n; i += nw) {
                uint32_t v = ldg((const uint32_t*)(touch_line(t.map[m], xcd, i, lane) + (z_w ? z * z_w[m] : 0)));
                ARRIVED(v);
            }
    }
}

struct LinArgs {
    const bf16_t* X;        // [R][K] operand tiles
    const uint4* W;         // [N][K] operand tiles
    const float *bias, *colsum;
    const float2* stats;    // [R][K >> sg] statistics of X's rows (LayerNorm-folded maps)
    int nks, NT, R, N;      // K / 32, column tiles, rows, columns
    int sg, sg_out;         // log2 of the columns that an entry of stats (stats_out) describes: 4 to 6; a row's entries are an even number
    bf16_t* out;            // operand tiles of the next map: q, hidden layer or the residual stream's bf16 copy
    float* outf;            // logits, or the new residual stream (LE_RESID)
    float2* stats_out;      // [R][N >> sg_out] (LE_RESID)
    bf16_t *Kc, *Vc;        // LE_QKV: this layer's cache
    const int32_t *L, *n_rows, *row_seq, *row0;   // row_seq, row0: of a ragged prompt pass (null: sequence b has rows b * M ..)
    uint32_t m_magic;       // ceil(2^32 / M): r / M of a step's rows (0: M = 1)
    const float* resid;     // LE_RESID: what the map's result is added to
    int M, nH, maxpos, d;
    size_t z_w, z_b, z_x, z_out;   // LE_SILU, LE_F32: what a draft head's weights, bias (bytes), X and result (elements) are ahead of the previous head's
};

// Workgroup i runs on XCD i mod 8.  The first grid dimension counts column groups, padded to a multiple of 8, so that
// the row blocks that share a weight tile share an XCD and its L2 and the tile leaves HBM once.
__host__ __device__ inline int pad8(int a) { return (a + 7) & ~7; }

// Row statistics of the LayerNorm folded into a map, for the ROWS rows of a workgroup, in two steps: request (k_lin: behind its first
// operands, k_big: ahead of them) and merge (k_lin: behind the products, k_big: while the operands are on their way).  Eight (sixteen)
// neighbouring lanes share a row and read its tile statistics two at a time, 128 (256) contiguous bytes per load.
template <int ROWS, int OTHER>
struct RowStats {
    static constexpr int TPR = ROWS >= 32 ? 8 : 16, PASS = ROWS * TPR / 256, NV = 32 / TPR;   // NV loads: the 64 tiles of K = 1024
    const float2* sp[PASS];
    float c0[PASS];
    uint4 v[PASS][NV];
    __device__ __forceinline__ void request(const LinArgs& a, const float2* stats, int nks, int R, int row0) {
        const int tiles = nks * 32 >> a.sg, part = threadIdx.x % TPR;
#pragma unroll
        for (int p = 0; p < PASS; ++p) {
            sp[p] = stats + (size_t)min(row0 + p * (256 / TPR) + (int)threadIdx.x / TPR, R - 1) * tiles;
            c0[p] = ldg(&sp[p]->x);
#pragma unroll
            for (int j = 0; j < NV; ++j)
                if (j == 0 || 2 * j * TPR < tiles) v[p][j] = ldg4(sp[p] + (2 * (part + j * TPR) < tiles ? 2 * (part + j * TPR) : 0));
        }
    }
    __device__ __forceinline__ void merge(const LinArgs& a, float* s_mean, float* s_rstd) {
        const int tiles = a.nks * 32 >> a.sg, part = threadIdx.x % TPR;
#pragma unroll
        for (int p = 0; p < PASS; ++p) {
            float s1 = 0.f, s2 = 0.f, s3 = 0.f;   // sums of the tile means' distances from c0, of the tiles' squared deviations, of the squared distances
            // Which of two squares enters their sum without having been rounded is said here.  Left to the compiler it changes with the code around it, and
            // with it the last bit of a row's variance (OTHER: the pieces of the first of two passes in which it has always been the second one).
            auto add = [&](const uint4& w, bool second = false) {
                const float d0 = __uint_as_float(w.x) - c0[p], d1 = __uint_as_float(w.z) - c0[p];
                s1 += d0 + d1;
                s2 += __uint_as_float(w.y) + __uint_as_float(w.w);
                s3 += second ? __builtin_fmaf(d1, d1, d0 * d0) : __builtin_fmaf(d0, d0, d1 * d1);
            };
#pragma unroll
            for (int j = 0; j < NV; ++j)
                if (2 * (part + j * TPR) < tiles) add(v[p][j], PASS == 2 && p == 0 && j > 0 && j <= OTHER);
            for (int t = 2 * (part + NV * TPR); t < tiles; t += 2 * TPR) add(ldg4(sp[p] + t));
            auto sum = [](float x) {
                x = quad_sum(x);
                x += __int_as_float(dpp_perm<0x141>(__float_as_int(x)));
                if (TPR == 16) x += __int_as_float(dpp_perm<0x140>(__float_as_int(x)));
                return x;
            };
            s1 = sum(s1);
            s2 = sum(s2);
            s3 = sum(s3);
            if (part == 0) {
                const int r = p * (256 / TPR) + (int)threadIdx.x / TPR;
                const float m2 = s2 + (float)(1 << a.sg) * fmaxf(s3 - s1 * s1 / tiles, 0.f);
                s_mean[r] = c0[p] + s1 / tiles;
                s_rstd[r] = rsqrtf(m2 / (a.nks * 32) + LN_EPS);
            }
        }
    }
};

// Where row r of the QKV map goes in the cache: element offset of its sequence and position, or a negative position
// if it has none (a finished sequence, or beyond the cache).
struct KvRow { size_t base; int pos; };
__device__ __forceinline__ KvRow kv_row(const LinArgs& a, int r) {
    KvRow k{0, -1};
    if (r >= a.R) return k;
    const int b = a.row_seq ? ldg(a.row_seq + r) : r / a.M, pos = ldg(a.L + b) + (r - (a.row_seq ? ldg(a.row0 + b) : b * a.M));
    k.base = (size_t)b * a.nH * kv_cap(a.maxpos) * 64;
    if (pos < a.maxpos && ldg(a.n_rows + b) > 0) k.pos = pos;
    return k;
}

// Stores four consecutive outputs of one row (columns n0 .. n0 + 3); LE_RESID: the new values of the residual stream.
template <int EPI>
__device__ __forceinline__ void store4(const LinArgs& a, int r, int n0, bool live, const float (&v)[4], const KvRow& kv) {
    if constexpr (EPI == LE_LOGITS || EPI == LE_F32) {
        if (live)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (n0 + j < a.N) a.outf[(size_t)r * a.N + n0 + j] = v[j];
    } else if constexpr (EPI == LE_GELU) {
        const uint2 pk = make_uint2(pack_bf16(gelu_s(v[0]), gelu_s(v[1])), pack_bf16(gelu_s(v[2]), gelu_s(v[3])));
        if (live) *(uint2*)(a.out + toff(r, n0, a.N >> 5)) = pk;
    } else if constexpr (EPI == LE_SILU) {
        if (live) *(uint2*)(a.out + toff(r, n0, a.N >> 5)) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
    } else if constexpr (EPI == LE_RESID) {
        if (live) {
            *(float4*)(a.outf + (size_t)r * a.N + n0) = make_float4(v[0], v[1], v[2], v[3]);
            *(uint2*)(a.out + toff(r, n0, a.N >> 5)) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
        }
    } else {
        const uint2 pk = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
        if (n0 < a.d) {
            if (live) *(uint2*)(a.out + toff(r, n0, a.d >> 5)) = pk;
        } else if (kv.pos >= 0) {
            const int which = n0 >= 2 * a.d, cc = n0 - (which + 1) * a.d, head = cc >> 6, dim = cc & 63;
            const size_t hb = kv.base + (size_t)head * kv_cap(a.maxpos) * 64;
            if (which) {   // four dimensions of one position: four lanes of a value tile
                bf16_t* vp = a.Vc + hb + vc_off(kv.pos, dim);
                vp[0] = (bf16_t)pk.x; vp[8] = (bf16_t)(pk.x >> 16); vp[16] = (bf16_t)pk.y; vp[24] = (bf16_t)(pk.y >> 16);
            } else {
                *(uint2*)(a.Kc + hb + kc_off(kv.pos, dim)) = pk;   // four dimensions of one key: half of a lane's piece
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Linear map, one workgroup per 16 RT rows x 16 CT columns.  The four waves split the reduction; each loads its
// operands (weights from HBM, activations from L2, both already in MFMA operand tiles: one contiguous KiB per wave
// load) straight into registers, CH k-steps at a time with the next chunk's loads ahead of the current chunk's MFMAs;
// the four partial sums are added in wave order through LDS.
// What bounds it with few rows: the chain from the launch to the first product.  A wave issues an instruction every five clocks, every eight where one
// needs the one before, and arguments in memory take some 500 to 850 clocks, so what the operands' addresses need comes as leading
// arguments, which arrive in registers with the wave (build.py), the operands are asked for before everything else, from scalar bases with the
// distance in the instruction (WHOLE), and nothing waits ahead of them.  Statistics and the epilogue's inputs requested first, with the wait that this
// put before the operands, and arguments as one struct: steps of 1 | 16 | 64 | 128 | 5 x 27 nodes, us 310 | 340 | 358 | 475 | 464, with this change alone
// 288 | 315 | 341 | 465 | 449.  At d = 256 to 768, together with the attention's early keys and the touched weights, 64 nodes: 232 -> 221 (256), 254 -> 247, 258 -> 250, 293 -> 275 (768).
// ---------------------------------------------------------------------------
template <int RT, int CT, int CH, int EPI, int NW, bool WHOLE>   // WHOLE: every wave's k-steps are whole chunks (no load is clamped)
__global__ __launch_bounds__(64 * NW) void k_lin(const bf16_t* X, const uint4* W, int nks, int NT, int R, int per_block, size_t z_w, size_t z_x, LinArgs a, TouchList<2> ahead) {   // ahead: for the workgroups behind the map's own
    constexpr bool LN = EPI <= LE_LOGITS;
    constexpr int T = RT * CT, NPW = (T + NW - 1) / NW;   // output tiles, tiles per wave in the epilogue
    static_assert(!LN || NW == 4, "the row statistics are merged by 256 threads");
    constexpr int ROWS = RT == 3 ? 64 : RT * 16;   // rows whose statistics are merged
    __shared__ f32x4_t red[NW * T * 64];
    __shared__ float s_mean[ROWS], s_rstd[ROWS];
    const int g = blockIdx.x, rb = blockIdx.y;
    if (__builtin_expect(g * CT >= NT, 0)) {   // padding of the XCD-aware numbering
        const int first = (NT + CT * 8 - 1) / (CT * 8) * 8;
        if (g >= first) touch<NW>(ahead, first, 1, nullptr);
        return;
    }
    if constexpr (EPI == LE_SILU || EPI == LE_F32) {
        W = (const uint4*)((const char*)W + blockIdx.z * z_w);
        X += blockIdx.z * z_x;
    }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int lc = lane & 15, gq = lane >> 4, row0 = rb * RT * 16, last_rt = (R - 1) >> 4;
    const int ks_lo = (uint32_t)(nks * wave) / NW, ks_hi = (uint32_t)(nks * (wave + 1)) / NW, nk = ks_hi - ks_lo;
    // (one row tile: rows beyond the map's last read the last one's pieces, which are fewer lines: one row, QKV 4.3 -> 3.9 us, FFN2 6.8 -> 5.9)
    const uint32_t wl = (uint32_t)lane * 16u, xl = RT > 1 ? wl : (uint32_t)(min(lc, R - 1 - min(rb, last_rt) * 16) + 16 * gq) * 16u;
    const char *Wp[CT], *Xp[RT];
#pragma unroll
    for (int c = 0; c < CT; ++c) Wp[c] = (const char*)W + (size_t)(uint32_t)min(g * CT + c, NT - 1) * (uint32_t)(nks * 1024);
#pragma unroll
    for (int r = 0; r < RT; ++r) Xp[r] = (const char*)X + (size_t)(uint32_t)min(rb * RT + r, last_rt) * (uint32_t)(nks * 1024);
    f32x4_t acc[CT][RT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[c][r] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    // Workgroups on the same columns start at different k-steps: side by side they would all wait for the same lines from HBM, and a
    // compute unit has no more than some 64 KB of misses on their way; so each brings in a part that the others find in the L2.
    // (FFN2, K = 4096, us: 128 rows 8.6 -> 7.0, 135 rows 9.3 -> 8.7, 320 rows 12.8 -> 11.7; beyond what an L2 holds they
    // drive each other out of it: 1024 rows 18.4 -> 20.3, k_tile and k_big likewise.  Not the LayerNorm-folded maps of K = 1024,
    // whose operands are all on their way at once: 64 rows FFN1 5.0 -> 5.4.  Steps with and without it, us: d = 512, 128 nodes 265 | 271, d = 640 279 | 284, d = 768,
    // 64 nodes 275 | 282; d = 512, 64 nodes, where a wave's k-steps are one chunk, 247 | 242.)
    const int nch = (nk + CH - 1) / CH, turn = EPI == LE_RESID ? nk * rb * per_block >> 16 : 0;
    // Chunk j of the wave.  Loads are unconditional: a tile beyond the map's last row or column re-reads a valid one and only reaches
    // accumulators that are never stored; a k-step beyond the last re-reads a valid one and is not multiplied.
    auto load = [&](int j, uint4 (&w)[CH][CT], uint4 (&x)[CH][RT]) {
        if constexpr (WHOLE && EPI != LE_RESID) {   // distances from a scalar base per tile and four k-steps, as part of the instruction
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const uint32_t off = (uint32_t)(ks_lo + j * CH + (i & ~3)) * 1024u;
#pragma unroll
                for (int c = 0; c < CT; ++c) w[i][c] = ldg4(Wp[c] + off + wl + (i & 3) * 1024);
#pragma unroll
                for (int r = 0; r < RT; ++r) x[i][r] = ldg4(Xp[r] + off + xl + (i & 3) * 1024);
            }
        } else {
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                const int q = j * CH + i + turn, k = ks_lo + (EPI == LE_RESID && q >= nk ? q - nk : q);
                const uint32_t off = (uint32_t)(WHOLE ? k : min(k, nks - 1)) * 1024u;
#pragma unroll
                for (int c = 0; c < CT; ++c) w[i][c] = ldg4(Wp[c] + (off + wl));
#pragma unroll
                for (int r = 0; r < RT; ++r) x[i][r] = ldg4(Xp[r] + (off + xl));
            }
        }
    };
    auto mul = [&](int n, const uint4 (&w)[CH][CT], const uint4 (&x)[CH][RT]) {
#pragma unroll
        for (int i = 0; i < CH; ++i)
            if (i < n)
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int r = 0; r < RT; ++r)   // weights first: a lane then holds four consecutive columns of one row
                        acc[c][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[i][c]), __builtin_bit_cast(bf16x8_t, x[i][r]), acc[c][r], 0, 0, 0);
    };
    uint4 wA[CH][CT], xA[CH][RT], wB[CH][CT], xB[CH][RT];
    load(0, wA, xA);
    SCHED_FENCE();
    // row statistics and what the epilogue of this thread's tiles adds
    if constexpr (EPI == LE_SILU || EPI == LE_F32) {
        a.bias = (const float*)((const char*)a.bias + blockIdx.z * a.z_b);
        a.out += blockIdx.z * a.z_out;
        a.outf += blockIdx.z * a.z_out;
    }
    float bias[NPW][4], cs[NPW][4], xr[NPW][4];
    int seq[NPW], len[NPW], first[NPW], rows[NPW];   // LE_QKV: the row's sequence, its committed length, first row and rows
    RowStats<ROWS, EPI == LE_QKV ? 1 : 2> st;
    if constexpr (LN) st.request(a, a.stats, nks, R, row0);
#pragma unroll
    for (int p = 0; p < NPW; ++p) {
        const int t = wave + NW * p, n0 = (g * CT + t % CT) * 16 + 4 * gq, r = row0 + (t / CT) * 16 + lc;
        const bool have = t < T && g * CT + t % CT < NT;
        uint4 b4 = make_uint4(0, 0, 0, 0), c4 = b4, x4 = b4;
        if (have) {
            if (EPI != LE_F32) b4 = ldg4(a.bias + n0);
            if (LN) c4 = ldg4(a.colsum + n0);
            if (EPI == LE_RESID) x4 = ldg4(a.resid + (size_t)(r < R ? r : 0) * a.N + n0);
        }
        if constexpr (EPI == LE_QKV) {
            const int rr = min(r, R - 1);
            seq[p] = a.row_seq ? ldg(a.row_seq + rr) : a.m_magic ? (int)mulhi((uint32_t)rr, a.m_magic) : rr;
            len[p] = ldg(a.L + seq[p]);
            first[p] = a.row_seq ? ldg(a.row0 + seq[p]) : seq[p] * a.M;
            rows[p] = ldg(a.n_rows + seq[p]);
        }
        bias[p][0] = __uint_as_float(b4.x); bias[p][1] = __uint_as_float(b4.y); bias[p][2] = __uint_as_float(b4.z); bias[p][3] = __uint_as_float(b4.w);
        cs[p][0] = __uint_as_float(c4.x); cs[p][1] = __uint_as_float(c4.y); cs[p][2] = __uint_as_float(c4.z); cs[p][3] = __uint_as_float(c4.w);
        xr[p][0] = __uint_as_float(x4.x); xr[p][1] = __uint_as_float(x4.y); xr[p][2] = __uint_as_float(x4.z); xr[p][3] = __uint_as_float(x4.w);
        if (EPI == LE_SILU && have) {   // the map's own input at the output's place (N = K)
            const uint2 h = ldg2(X + toff(min(r, R - 1), n0, nks));
            xr[p][0] = bf2f((bf16_t)h.x); xr[p][1] = bf2f((bf16_t)(h.x >> 16)); xr[p][2] = bf2f((bf16_t)h.y); xr[p][3] = bf2f((bf16_t)(h.y >> 16));
        }
    }
    SCHED_FENCE();
    int j = 0;
    for (; j + 2 < nch; j += 2) {
        load(j + 1, wB, xB);
        SCHED_FENCE();   // (the scheduler would put a chunk's loads between the products)
        mul(CH, wA, xA);
        SCHED_FENCE();
        load(j + 2, wA, xA);
        SCHED_FENCE();
        mul(CH, wB, xB);
        SCHED_FENCE();
    }
    if (j + 1 < nch) {
        load(j + 1, wB, xB);
        SCHED_FENCE();
        mul(CH, wA, xA);
        mul(WHOLE ? CH : nk - (j + 1) * CH, wB, xB);
    } else {
        mul(WHOLE ? CH : nk - j * CH, wA, xA);
    }
    if constexpr (LN) st.merge(a, s_mean, s_rstd);
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int r = 0; r < RT; ++r) red[(wave * T + r * CT + c) * 64 + lane] = acc[c][r];
    __syncthreads();
#pragma unroll
    for (int p = 0; p < NPW; ++p) {
        const int t = wave + NW * p;
        if (t >= T) break;
        const int c = t % CT, rl = (t / CT) * 16 + lc, r = row0 + rl, tile = g * CT + c, n0 = tile * 16 + 4 * gq;
        if (tile >= NT) continue;
        f32x4_t s = red[t * 64 + lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) s += red[(w * T + t) * 64 + lane];
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float y = s[j];
            if (LN) y = s_rstd[rl] * (y - s_mean[rl] * cs[p][j]);
            v[j] = y + bias[p][j];
            if (EPI == LE_RESID) v[j] += xr[p][j];
            if (EPI == LE_SILU) v[j] = xr[p][j] + v[j] / (1.f + __expf(-v[j]));
        }
        if constexpr (EPI == LE_RESID) {   // statistics of the tile's 16 columns: four here, twelve in the lanes 16, 32 and 48 further on
            const float mean = rows_sum(v[0] + v[1] + v[2] + v[3]) * (1.f / 16.f);
            const float m2 = rows_sum((v[0] - mean) * (v[0] - mean) + (v[1] - mean) * (v[1] - mean) + (v[2] - mean) * (v[2] - mean) + (v[3] - mean) * (v[3] - mean));
            if (r < R && gq == 0) a.stats_out[(size_t)r * (a.N >> 4) + tile] = make_float2(mean, m2);
        }
        KvRow kv{0, -1};
        if constexpr (EPI == LE_QKV) {
            kv.base = (size_t)seq[p] * a.nH * kv_cap(a.maxpos) * 64;
            const int pos = len[p] + r - first[p];
            if (r < R && pos < a.maxpos && rows[p] > 0) kv.pos = pos;
        }
        store4<EPI>(a, r, n0, r < R, v, kv);
    }
}

// ---------------------------------------------------------------------------
// Linear map of many rows: one workgroup per 64 rows x 128 columns, wave w taking all rows and the columns 32 w .. 32 w + 31
// of them.  Activations pass through LDS (all four waves need all of them), weights go straight into the
// registers of the one wave that needs them.  v_mfma_f32_32x32x16_bf16: with one wave per SIMD it reaches 2.26 PFLOP/s
// where the 16 x 16 x 32 form reaches 1.4 (register operands, 256 workgroups); two row tiles (column tiles) and half
// of their k-step make one operand, which is a permutation of the 16-byte pieces of the stored tiles.
// The reduction runs in stages of two k-steps of 32.  A stage's activation tiles are fetched into registers by the four
// waves (two tiles each) four stages before they are multiplied and written to LDS two stages before; weights are
// fetched two stages ahead.  Two stages in registers and 144 vector registers let three workgroups share a compute unit;
// tile, depth and occupancy were measured together (FFN1 at 2048 rows, K = 1024, us): 128 x 256, one workgroup per compute
// unit 28.7; 128 x 128, two, 24.7; 64 x 256, two, 25.3; 64 x 128 with four stages, two, 27.5, with two stages, three, 26.0, four,
// 31.  64 x 128 is the best of them at 1024 rows and for narrow maps (QKV 14.1 against 16.2 for 128 x 128, FFN1 15.7 against 16.5).
// What bounds it: no single unit.  FFN1 of 1024 rows takes 17 us in a step; its products keep a SIMD's matrix core busy
// for 3.4 us of them, and a compute unit pulls 0.8 MB through L2.  512 workgroups are 0.67 rounds of the 768 that fit, each with its
// statistics, 16 stages with a barrier, GELU and stores one behind the other.
// Residual maps: tiles numbered in blocks per XCD (with a column of tiles per XCD all activations go into every L2), statistics per
// 32 columns (us, before and after, weights from HBM): out-projection of 2048 rows 15.0 -> 13.2, FFN2 of 3200 rows 46.4 -> 42.5, of 4352 rows
// 68.6 -> 62.4.  The other maps keep the column numbering: their activations fit an L2, and finding the block costs more than it gives (QKV
// of 1024 rows 16.8 against 17.6).  FFN1 stores its results as whole 16-byte pieces (640 rows 15.4 -> 14.3, 1024 rows 18.2 -> 17.4).
// ---------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
// D = A B + C, A 32 x 16 (lane: row lane & 31, k 8 (lane >> 5) ..), B 16 x 32 alike; lane l, element i of D: column
// l & 31, row (i & 3) + 8 (i >> 2) + 4 (l >> 5).
__device__ __forceinline__ f32x16_t mfma_32x32(uint4 a, uint4 b, f32x16_t c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
#else   // host emulation of the kernels: the wave's operands meet in an array, between two lane exchanges
    __shared__ uint4 ops[8][2][64];
    const int w = (int)(threadIdx.x >> 6), l = (int)(threadIdx.x & 63);
    ops[w][0][l] = a;
    ops[w][1][l] = b;
    (void)__shfl(0u, 0, 64);
    for (int i = 0; i < 16; ++i)
        for (int k = 0; k < 16; ++k) {
            auto value = [&](int op, int row) { return bf2f(((const bf16_t*)&ops[w][op][row + 32 * (k >> 3)])[k & 7]); };
            c[i] += value(0, (i & 3) + 8 * (i >> 2) + 4 * (l >> 5)) * value(1, l & 31);
        }
    (void)__shfl(0u, 0, 64);
    return c;
#endif
}

// Stores 16 outputs of one row, columns n0 .. n0 + 15, held by lanes l and l + 32 (hi): columns 4 hi .. + 3 and 8 + 4 hi .. + 3.
// bf16 results change places between the two lanes first, so that each has eight consecutive columns, a whole piece of an
// operand tile: with half pieces every cache line is written in two parts.
template <int EPI>
__device__ __forceinline__ void store16(const LinArgs& a, int r, int n0, int hi, float (&v)[8], const KvRow& kv) {
    const bool live = r < a.R;
    if constexpr (EPI == LE_LOGITS) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int n = n0 + 4 * hi + (j & 3) + 2 * (j & 4);
            if (live && n < a.N) a.outf[(size_t)r * a.N + n] = v[j];
        }
        return;
    }
    if constexpr (EPI == LE_RESID) {
        if (live) {
            *(float4*)(a.outf + (size_t)r * a.N + n0 + 4 * hi) = make_float4(v[0], v[1], v[2], v[3]);
            *(float4*)(a.outf + (size_t)r * a.N + n0 + 8 + 4 * hi) = make_float4(v[4], v[5], v[6], v[7]);
        }
    }
    if constexpr (EPI == LE_GELU)
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = gelu_s(v[j]);
    if constexpr (EPI == LE_QKV) {
        // (half pieces: a store of values wants the two lanes' dimensions four apart, in the same line; through LDS into whole pieces of eight
        // positions it took 1 to 2 us more)
        const float lo[4] = {v[0], v[1], v[2], v[3]}, up[4] = {v[4], v[5], v[6], v[7]};
        store4<EPI>(a, r, n0 + 4 * hi, live, lo, kv);
        store4<EPI>(a, r, n0 + 8 + 4 * hi, live, up, kv);
        return;
    }
    const vadusa_u32x2 p = __builtin_amdgcn_permlane32_swap(pack_bf16(v[0], v[1]), pack_bf16(v[4], v[5]), false, false);
    const vadusa_u32x2 q = __builtin_amdgcn_permlane32_swap(pack_bf16(v[2], v[3]), pack_bf16(v[6], v[7]), false, false);
    const uint4 pk = make_uint4(p.x, q.x, p.y, q.y);   // columns n .. n + 7
    const int n = n0 + 8 * hi;
    if (live) *(uint4*)(a.out + toff(r, n, a.N >> 5)) = pk;
}

// Which tile a workgroup takes.  Workgroup i runs on XCD i mod 8: every XCD gets an eighth of the tiles, consecutive in
// strips of `strip` column tiles, so that the rows and columns which its L2 fetches are about the same number.
// (n: tiles; gs: those of a strip; magics: ceil(2^32 / gs), ceil(2^32 / strip), or 0 where a quotient by them is not exact for every tile.)
struct TileGrid { int gr, gc, strip, n, gs; uint32_t gs_magic, strip_magic; };
__device__ __forceinline__ uint32_t div_magic(uint32_t a, uint32_t by, uint32_t magic) { return magic ? mulhi(a, magic) : a / by; }
// Row and column tile of this workgroup, or false.  What every workgroup needs comes first, as arguments that arrive with the wave, and is found without a
// division (64 x 32 nodes 1499 -> 1487 us per step, its prompts 12 350 -> 12 180, 5 x 27 nodes 439 -> 433); a last strip that is narrower than the
// others is found from the rest.
__device__ __forceinline__ bool tile_of(int n, int gs, uint32_t gs_magic, int strip, uint32_t strip_magic, const TileGrid& g, int* row, int* col) {
    const int xcd = blockIdx.x & 7, lo = (n * xcd) >> 3, i = lo + (int)(blockIdx.x >> 3);
    if (i >= (n * (xcd + 1)) >> 3) return false;
    const int s = (int)div_magic((uint32_t)i, (uint32_t)gs, gs_magic), in = i - s * gs;
    int w = strip;
    if (n - s * gs >= gs) {
        *row = (int)div_magic((uint32_t)in, (uint32_t)strip, strip_magic);
    } else {
        w = g.gc - s * strip;
        *row = in / w;
    }
    *col = s * strip + in - *row * w;
    return true;
}

constexpr int BIG_RT = 4, BIG_CT = 2;   // row tiles of a workgroup, column tiles of a wave
template <int EPI>
__global__ __launch_bounds__(256, 3) void k_big(const bf16_t* X, const uint4* Wt, const float2* stats, int nks, int NT, int R, int n, int gs, uint32_t gs_magic, int strip, LinArgs a, TileGrid g) {
    constexpr bool LN = EPI <= LE_LOGITS;
    constexpr int NRT = BIG_RT, NCT = BIG_CT, DEPTH = 2;   // DEPTH: stages in registers
    static_assert(4 % DEPTH == 0, "stage c uses register set c mod DEPTH by c mod 4");
    constexpr int ROWS = NRT * 16, NA = NRT / 2, NR2 = NRT / 2, NC2 = NCT / 2;   // NA: activation tiles a wave fetches per stage
    __shared__ uint4 sA[4][NRT * 2 * 64];
    __shared__ float s_mean[ROWS], s_rstd[ROWS];
    int rb, ct0;   // row tile of 64, first column tile
    if constexpr (EPI != LE_RESID) {
        // Workgroup i runs on XCD i mod 8: the XCD has an eighth of the columns, whose weights leave HBM once.
        rb = blockIdx.y;
        ct0 = blockIdx.x * 4 * NCT;
        if (ct0 >= NT) return;   // padding of that numbering
    } else {
        if (!tile_of(n, gs, gs_magic, strip, g.strip_magic, g, &rb, &ct0)) return;
        ct0 *= 4 * NCT;
    }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int row0 = rb * ROWS, last_rt = (R - 1) >> 4;
    const int wt0 = ct0 + wave * NCT;      // this wave's first column tile
    const int nst = nks >> 1;            // stages (K is a multiple of 64)
    RowStats<ROWS, 1> st;
    if constexpr (LN) st.request(a, stats, nks, R, row0);
    // Tiles beyond the map's last row or column re-read a valid one and only reach accumulators that are never stored.
    const char* Xp[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) {         // the wave's tiles of a stage: T = wave + 4 j is row tile T >> 1, k-step T & 1
        const int T = wave + 4 * j;
        Xp[j] = (const char*)((const uint4*)X + ((size_t)min(rb * NRT + (T >> 1), last_rt) * nks + (T & 1)) * 64);
    }
    const int second = (lane >> 4) & 1, piece = (lane & 15) + 16 * (lane >> 5);   // operand lane -> tile of the pair, piece of the tile's first half
    // Tiles by a 64-bit base of the wave and a 32-bit distance from it: a map may hold more than 4 GiB.
    const int wt_first = min(wt0, NT - 1);
    const char* Wp = (const char*)Wt + (size_t)wt_first * nks * 1024;
    uint32_t woff[NC2];
#pragma unroll
    for (int c = 0; c < NC2; ++c) woff[c] = (uint32_t)(min(wt0 + 2 * c + second, NT - 1) - wt_first) * (uint32_t)nks * 1024u + (uint32_t)piece * 16u;
    auto loadA = [&](int c, uint4 (&x)[NA]) {
        const uint32_t off = (uint32_t)min(c, nst - 1) * 2048u + (uint32_t)lane * 16u;
#pragma unroll
        for (int j = 0; j < NA; ++j) x[j] = ldg4(Xp[j] + off);
    };
    auto loadW = [&](int c, uint4 (&w)[4][NC2]) {   // the four operand halves (k-step, half) of the stage
        const char* base = Wp + (uint32_t)min(c, nst - 1) * 2048u;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < NC2; ++i) w[q][i] = ldg4(base + q * 512 + woff[i]);
    };
    auto writeA = [&](int buf, const uint4 (&x)[NA]) {
#pragma unroll
        for (int j = 0; j < NA; ++j) sA[buf][(wave + 4 * j) * 64 + lane] = x[j];
    };
    f32x16_t acc[NC2][NR2];
#pragma unroll
    for (int c = 0; c < NC2; ++c)
#pragma unroll
        for (int r = 0; r < NR2; ++r)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[c][r][i] = 0.f;
    auto readA = [&](int buf, int k, uint4 (&x)[2][NR2]) {   // both halves of k-step k
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < NR2; ++r) x[h][r] = sA[buf][((2 * r + second) * 2 + k) * 64 + 32 * h + piece];
    };
    auto mul = [&](const uint4 (&x)[2][NR2], const uint4 (&w0)[NC2], const uint4 (&w1)[NC2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < NR2; ++r)
#pragma unroll
                for (int c = 0; c < NC2; ++c)   // weights first: a lane then holds groups of four consecutive columns of one row
                    acc[c][r] = mfma_32x32(h ? w1[c] : w0[c], x[h][r], acc[c][r]);
    };
    // Stage c reads LDS buffer c mod 4 and weight set c mod 2; set c mod 2 of the activation registers holds stage
    // c + 2, which goes into buffer (c + 2) mod 4, last read in stage c - 2, and then takes stage c + 4.  The first k-step's operands of stage c are
    // read at the end of stage c - 1, so that no multiplication waits for LDS; the scheduling fences keep the compiler
    // from moving the reads next to their uses.  Every load, copy and read is unconditional, so that the waits count exactly
    // the loads issued since: past the end the last stage is fetched again (from L2) and never multiplied.
    uint4 A[DEPTH][NA], W[DEPTH][4][NC2], x0[2][NR2], x1[2][NR2];
    loadA(0, A[0]);
    loadA(1, A[1]);
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) {
        loadW(i, W[i]);
        if (i >= 2) loadA(i, A[i]);
    }
    if constexpr (LN) st.merge(a, s_mean, s_rstd);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        writeA(i, A[i]);
        loadA(DEPTH + i, A[i]);
    }
    __syncthreads();
    readA(0, 0, x0);
    auto stage = [&](int c, auto bc) {
        constexpr int b = decltype(bc)::value;   // c mod 4
        readA(b, 1, x1);
        writeA((b + 2) & 3, A[(b + 2) % DEPTH]);
        loadA(c + 2 + DEPTH, A[(b + 2) % DEPTH]);
        SCHED_FENCE();
        mul(x0, W[b % DEPTH][0], W[b % DEPTH][1]);
        __syncthreads();
        readA((b + 1) & 3, 0, x0);
        SCHED_FENCE();
        mul(x1, W[b % DEPTH][2], W[b % DEPTH][3]);
        loadW(c + DEPTH, W[b % DEPTH]);
        SCHED_FENCE();
    };
    constexpr std::integral_constant<int, 0> b0{};
    constexpr std::integral_constant<int, 1> b1{};
    constexpr std::integral_constant<int, 2> b2{};
    constexpr std::integral_constant<int, 3> b3{};
    int c = 0;
    for (; c + 4 <= nst; c += 4) {
        stage(c, b0);
        stage(c + 1, b1);
        stage(c + 2, b2);
        stage(c + 3, b3);
    }
    if (c < nst) {
        stage(c, b0);
        if (c + 1 < nst) {
            stage(c + 1, b1);
            if (c + 2 < nst) stage(c + 2, b2);
        }
    }
    // Everything the epilogue reads arrives before its first store: a wait between the stores would wait for them too
    // (loads and stores share one counter).
    const int lr = lane & 31, hi = lane >> 5;   // the lane's row of a 32-row block; its columns of a block: 8 q + 4 hi .. + 3, q = 0 .. 3
    KvRow kv[NR2];
    float mean[NR2], rstd[NR2];
#pragma unroll
    for (int ri = 0; ri < NR2; ++ri) {
        kv[ri] = KvRow{0, -1};
        if (EPI == LE_QKV && wt0 * 16 + 16 * NCT > a.d) kv[ri] = kv_row(a, row0 + ri * 32 + lr);
        mean[ri] = LN ? s_mean[ri * 32 + lr] : 0.f;
        rstd[ri] = LN ? s_rstd[ri * 32 + lr] : 1.f;
    }
#pragma unroll
    for (int ci = 0; ci < NC2; ++ci) {
        float bias[4][4], cs[4][4], xr[NR2][4][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int tile = min(wt0 + 2 * ci + (q >> 1), NT - 1), n0 = tile * 16 + 8 * (q & 1) + 4 * hi;
            const uint4 b4 = ldg4(a.bias + n0), c4 = LN ? ldg4(a.colsum + n0) : make_uint4(0, 0, 0, 0);
            bias[q][0] = __uint_as_float(b4.x); bias[q][1] = __uint_as_float(b4.y); bias[q][2] = __uint_as_float(b4.z); bias[q][3] = __uint_as_float(b4.w);
            cs[q][0] = __uint_as_float(c4.x); cs[q][1] = __uint_as_float(c4.y); cs[q][2] = __uint_as_float(c4.z); cs[q][3] = __uint_as_float(c4.w);
            if constexpr (EPI == LE_RESID)
#pragma unroll
                for (int ri = 0; ri < NR2; ++ri) {
                    const uint4 x4 = ldg4(a.resid + (size_t)min(row0 + ri * 32 + lr, R - 1) * a.N + n0);
                    xr[ri][q][0] = __uint_as_float(x4.x); xr[ri][q][1] = __uint_as_float(x4.y); xr[ri][q][2] = __uint_as_float(x4.z); xr[ri][q][3] = __uint_as_float(x4.w);
                }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            ARRIVED(bias[q][0]); ARRIVED(cs[q][0]);
            if constexpr (EPI == LE_RESID)
#pragma unroll
                for (int ri = 0; ri < NR2; ++ri) ARRIVED(xr[ri][q][0]);
        }
        if (EPI == LE_QKV)
#pragma unroll
            for (int ri = 0; ri < NR2; ++ri) ARRIVED(kv[ri].pos);
#pragma unroll
        for (int ri = 0; ri < NR2; ++ri) {
            const int r = row0 + ri * 32 + lr;
            float v[2][8];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int q = 2 * t + (e >> 2), j = e & 3;
                    float y = acc[ci][ri][8 * t + e];
                    if (LN) y = rstd[ri] * (y - mean[ri] * cs[q][j]);
                    v[t][e] = y + bias[q][j];
                    if (EPI == LE_RESID) v[t][e] += xr[ri][q][j];
                }
            if constexpr (EPI == LE_RESID) {
                // statistics of 32 columns: sixteen here, sixteen in the lane 32 further on
                float sum = 0.f, sq = 0.f;
#pragma unroll
                for (int t = 0; t < 2; ++t) sum += ((v[t][0] + v[t][1]) + (v[t][2] + v[t][3])) + ((v[t][4] + v[t][5]) + (v[t][6] + v[t][7]));
                const float mu = half_sum(sum) * (1.f / 32.f);
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 8; ++e) sq += (v[t][e] - mu) * (v[t][e] - mu);
                sq = half_sum(sq);
                if (r < R && hi == 0 && wt0 + 2 * ci < NT) a.stats_out[(size_t)r * (a.N >> 5) + ((wt0 + 2 * ci) >> 1)] = make_float2(mu, sq);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)
                if (wt0 + 2 * ci + t < NT) store16<EPI>(a, r, (wt0 + 2 * ci + t) * 16, hi, v[t], kv[ri]);
        }
    }
}

// ---------------------------------------------------------------------------
// Linear map of many rows where its rounds of workgroups are nearly full: one workgroup per 64 RG rows x 64 CG columns and compute
// unit, eight waves of 64 x 64 outputs each; where the workgroup has fewer than eight such blocks the waves share a block's reduction
// (KSP waves per block).  Both operands pass through a ring of LDS stages, filled by loads that go straight into LDS (a stored operand
// tile is the contiguous KiB that such a load writes): up to 144 KiB are in flight per compute unit and cost no registers.  Half the bytes of
// k_big per product cross from L2.
// What bounds it (2048 rows, FFN1, 256 x 128 outputs, 24.8 us in a step): launch 2.5 us, the first stage 2.5, products 13 (LDS: 128 KB of
// operand reads and 48 KB of arrivals per stage at 128 B per clock against 1024 clocks of matrix instructions; and the clock, which
// falls from 2.4 to 1.6 GHz while every matrix core is busy), epilogue 5 (GELU: 70 clocks per value and SIMD) with nothing beside it.  Measured
// and not kept: 128 x 64 outputs per wave and four waves, which reads a quarter less from LDS but leaves one wave per SIMD (27.8 instead of 24.2 us);
// a stage's loads in one piece behind the barrier (24.9); the row statistics asked for in the middle of the reduction (+1.5); a ninth wave
// that reads the weights' lines ahead of the ring (K = 4096: products 21.5 -> 20.2 us and a clock 0.3 GHz lower, 29.1 -> 30.6).
// ---------------------------------------------------------------------------
// One KiB from memory into LDS, 16 bytes per lane; counts as one load of the wave.  No register receives it and the
// compiler does not know of it: landed() is what says that it has arrived.
__device__ __forceinline__ void fill_lds(uint4* lds, const char* src, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"((uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint4*)lds), "v"(lane * 16), "s"(src) : "memory");
#else
    lds[lane] = ldg4(src + lane * 16);
#endif
}
// All but the wave's N youngest loads have arrived and its LDS reads are done; then every wave of the workgroup is here.
template <int N>
__device__ __forceinline__ void landed() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
#else
    __syncthreads();
#endif
}

template <int RG, int CG> struct TileShape {
    static constexpr int NB = RG * CG, KSP = 8 / NB;              // blocks of 64 x 64, waves per block
    static constexpr int KB = KSP == 1 ? 2 : 4;                   // k-steps of 32 per stage
    static constexpr int TILES = 4 * (RG + CG), KIB = TILES * KB; // operand tiles, KiB of a stage
    static constexpr int NS = 144 / KIB;                          // stages in the ring
    static_assert((KSP == 1 || KSP == 4) && NS == 3, "the waits and the epilogue are written for 256 x 128 and 128 x 64 outputs");
    static constexpr int LPW = KIB / 8, SPW = 2 * KB / KSP;       // loads and half k-steps of a wave per stage
};

template <int RG, int CG, int EPI>
__global__ __launch_bounds__(512) void k_tile(const bf16_t* X, const uint4* W, const float2* stats, int nks, int NT, int R, int n, int gs, uint32_t gs_magic, int strip, LinArgs a, TileGrid t) {
    using S = TileShape<RG, CG>;
    constexpr bool LN = EPI <= LE_LOGITS;
    constexpr int NB = S::NB, KSP = S::KSP, KB = S::KB, NS = S::NS, LPW = S::LPW, SPW = S::SPW, ROWS = 64 * RG;
    static_assert(SPW % 2 == 0, "a stage starts with the first of the two operand sets");
    __shared__ uint4 ring[NS * S::KIB * 64];
    __shared__ float s_mean[ROWS], s_rstd[ROWS];
    __shared__ float4 s_bias[16 * CG], s_cs[16 * CG];
    int row0, ct0;   // first row and column tile
    {
        if (!tile_of(n, gs, gs_magic, strip, t.strip_magic, t, &row0, &ct0)) return;
        row0 *= ROWS;
        ct0 *= 4 * CG;
    }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int rg = wave / CG % RG, cg = wave % CG, kq = wave / NB;   // the wave's block and its share of the reduction
    const int nst = (nks + KB - 1) / KB;
    // row statistics: TPR threads of a row read two groups at a time, NV such pieces asked for here
    constexpr int TPR = 512 / ROWS, NV = TPR < 8 ? 8 : 4;
    const int groups = (nks * 32) >> a.sg;
    const float2* sp = nullptr;
    float c0 = 0.f;
    uint4 sv[NV];
    if constexpr (LN) {
        sp = stats + (size_t)min(row0 + tid / TPR, R - 1) * groups;
        c0 = ldg(&sp->x);
#pragma unroll
        for (int j = 0; j < NV; ++j) sv[j] = ldg4(sp + (2 * (tid % TPR + j * TPR) < groups ? 2 * (tid % TPR + j * TPR) : 0));
    }
    float bias_in = 0.f, cs_in = 0.f;   // one column's per thread of the first waves
    if (tid < 64 * CG) {
        const int n = min(ct0 * 16 + tid, NT * 16 - 1);
        bias_in = ldg(a.bias + n);
        if constexpr (LN) cs_in = ldg(a.colsum + n);
    }
    SCHED_FENCE();
    // Tiles beyond the map's last row or column re-read a valid one and only reach accumulators that are never stored; k-steps
    // beyond the last re-read the last and are not multiplied.
    const char* base[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int T = (wave + 8 * i) / KB;
        base[i] = T < 4 * RG ? (const char*)X + (size_t)min((row0 >> 4) + T, (R - 1) >> 4) * nks * 1024
                             : (const char*)W + (size_t)min(ct0 + T - 4 * RG, NT - 1) * nks * 1024;
    }
    auto fetch = [&](int s, int buf, int i0, int i1) {   // loads i0 .. i1 - 1 of stage s
#pragma unroll
        for (int i = 0; i < LPW; ++i)
            if (i >= i0 && i < i1) {
                const int j = wave + 8 * i;
                fill_lds(ring + (buf * S::KIB + j) * 64, base[i] + (uint32_t)min(s * KB + j % KB, nks - 1) * 1024u, lane);
            }
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < nst) fetch(s, s, 0, LPW);
    f32x16_t acc[2][2];   // [block of 32 columns][block of 32 rows]
#pragma unroll
    for (int i = 0; i < 64; ++i) acc[i >> 5][(i >> 4) & 1][i & 15] = 0.f;
    // an operand: two tiles' rows, one half of their k-step
    const int second = (lane >> 4) & 1, piece = (lane & 15) + 16 * (lane >> 5);
    const uint4* xl = ring + (rg * 4 + second) * KB * 64 + piece;
    const uint4* wl = ring + ((RG + cg) * 4 + second) * KB * 64 + piece;
    uint4 x[2][2], w[2][2];
    auto read = [&](int buf, int sl, uint4 (&x)[2], uint4 (&w)[2]) {
        const int q = kq * SPW + sl, at = buf * S::KIB * 64 + (q >> 1) * 64 + (q & 1) * 32;
#pragma unroll
        for (int i = 0; i < 2; ++i) { x[i] = xl[at + 2 * i * KB * 64]; w[i] = wl[at + 2 * i * KB * 64]; }
    };
    auto mul = [&](const uint4 (&x)[2], const uint4 (&w)[2]) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int r = 0; r < 2; ++r) acc[c][r] = mfma_32x32(w[c], x[r], acc[c][r]);   // weights first: a lane then holds groups of four consecutive columns of one row
    };
    // Stage s is multiplied while the stages behind it arrive; behind it, one slice after the other, go the loads of stage
    // s + NS - 1 into the place that stage s - 1 left.
    int buf = 0;
    if (nst >= NS - 1) landed<(NS - 2) * LPW>();
    else landed<0>();
    read(0, 0, x[0], w[0]);
    auto stage = [&](int s, auto final) {
        const int next = buf + 1 == NS ? 0 : buf + 1, left = buf ? buf - 1 : NS - 1;
#pragma unroll
        for (int sl = 0; sl < SPW; ++sl) {
            if (sl + 1 < SPW) read(buf, sl + 1, x[(sl + 1) & 1], w[(sl + 1) & 1]);
            if constexpr (!decltype(final)::value) {
                if (sl + 1 < SPW) {
                    if (s + NS - 1 < nst) fetch(s + NS - 1, left, LPW * sl / (SPW - 1), LPW * (sl + 1) / (SPW - 1));
                } else {
                    if (s + NS <= nst) landed<(NS - 2) * LPW>();      // stages s + 2 .. s + NS - 1 may be on their way
                    else landed<0>();
                    read(next, 0, x[0], w[0]);
                }
            }
            SCHED_FENCE();
            if (KB == 2 || s * KB + (kq * SPW + sl) / 2 < nks) mul(x[sl & 1], w[sl & 1]);
            SCHED_FENCE();
        }
        buf = next;
    };
    for (int s = 0; s + 1 < nst; ++s) stage(s, std::false_type{});
    // What the epilogue adds is asked for ahead of the last stage's products.
    constexpr int RB = KSP == 1 ? 2 : 1, TB = KSP == 1 ? 4 : 2;
    const int lr = lane & 31, hi = lane >> 5, rb0 = KSP == 1 ? 0 : kq >> 1, tb0 = KSP == 1 ? 0 : 2 * (kq & 1), tile0 = ct0 + 4 * cg + tb0;
    int r[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) r[i] = row0 + (rg * 2 + rb0 + i) * 32 + lr;
    uint4 xr[RB][TB][2];
    if constexpr (EPI == LE_RESID)
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int tt = 0; tt < TB; ++tt)
#pragma unroll
                for (int h = 0; h < 2; ++h) xr[i][tt][h] = ldg4(a.resid + (size_t)min(r[i], R - 1) * a.N + min(tile0 + tt, NT - 1) * 16 + 8 * h + 4 * hi);
    KvRow kv[RB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        kv[i] = KvRow{0, -1};
        if (EPI == LE_QKV && (tile0 + TB) * 16 > a.d) kv[i] = kv_row(a, r[i]);
    }
    SCHED_FENCE();
    stage(nst - 1, std::true_type{});
    if constexpr (LN) {
        float s1 = 0.f, s2 = 0.f, s3 = 0.f;   // sums of the group means' distances from c0, of the groups' squared deviations, of the squared distances
        auto add = [&](const uint4& g) {
            const float d0 = __uint_as_float(g.x) - c0, d1 = __uint_as_float(g.z) - c0;
            s1 += d0 + d1;
            s2 += __uint_as_float(g.y) + __uint_as_float(g.w);
            s3 += d0 * d0 + d1 * d1;
        };
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            ARRIVED(sv[j].x);
            if (2 * (tid % TPR + j * TPR) < groups) add(sv[j]);
        }
        for (int g = 2 * (tid % TPR + NV * TPR); g < groups; g += 2 * TPR) add(ldg4(sp + g));
        auto sum = [](float v) {
            if (TPR >= 2) v += __int_as_float(dpp_perm<0xB1>(__float_as_int(v)));
            if (TPR >= 4) v += __int_as_float(dpp_perm<0x4E>(__float_as_int(v)));
            if (TPR >= 8) v += __int_as_float(dpp_perm<0x141>(__float_as_int(v)));
            return v;
        };
        s1 = sum(s1);
        s2 = sum(s2);
        s3 = sum(s3);
        if (tid % TPR == 0) {
            const float m2 = s2 + (float)(1 << a.sg) * fmaxf(s3 - s1 * s1 / groups, 0.f);
            s_mean[tid / TPR] = c0 + s1 / groups;
            s_rstd[tid / TPR] = rsqrtf(m2 / (nks * 32) + LN_EPS);
        }
    }
    // The block's outputs: piece u of 32 rows x 16 columns, u = 4 (row block) + column tile; a lane holds eight values of one
    // row, columns 4 hi .. + 3 of each eight.  Waves that share a block add their sums through LDS and take 8 / KSP pieces each.
    float y[RB][TB][8];
    ARRIVED(bias_in);
    if (tid < 64 * CG) {
        ((float*)s_bias)[tid] = bias_in;
        if constexpr (LN) ((float*)s_cs)[tid] = cs_in;
    }
    if constexpr (KSP == 1) {
#pragma unroll
        for (int i = 0; i < 64; ++i) y[i >> 5][(i >> 3) & 3][i & 7] = acc[(i >> 4) & 1][i >> 5][8 * ((i >> 3) & 1) + (i & 7)];
        __syncthreads();
    } else {
        float4* part = (float4*)ring;   // [wave][piece][half][lane]; 
        __syncthreads();                // (the last stage has been read)
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x16_t& v = acc[(u >> 1) & 1][u >> 2];
                const int e = 8 * (u & 1) + 4 * h;
                part[((wave * 8 + u) * 2 + h) * 64 + lane] = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
            }
        __syncthreads();
#pragma unroll
        for (int tt = 0; tt < TB; ++tt)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int k = 0; k < KSP; ++k) {
                    const float4 p = part[(((k * NB + rg * CG + cg) * 8 + rb0 * 4 + tb0 + tt) * 2 + h) * 64 + lane];
                    v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
                }
                y[0][tt][4 * h] = v.x; y[0][tt][4 * h + 1] = v.y; y[0][tt][4 * h + 2] = v.z; y[0][tt][4 * h + 3] = v.w;
            }
    }
    // Everything the epilogue reads has arrived before its first store: a wait between the stores would wait for them too
    // (loads and stores share one counter).
    if (tile0 >= NT) return;
    if constexpr (EPI == LE_RESID)
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int tt = 0; tt < TB; ++tt) { ARRIVED(xr[i][tt][0].x); ARRIVED(xr[i][tt][1].x); }
    if constexpr (EPI == LE_QKV)
#pragma unroll
        for (int i = 0; i < RB; ++i) ARRIVED(kv[i].pos);
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int rl = (rg * 2 + rb0 + i) * 32 + lr;
        const float mean = LN ? s_mean[rl] : 0.f, rstd = LN ? s_rstd[rl] : 1.f;
#pragma unroll
        for (int tt = 0; tt < TB; ++tt)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int at = (4 * cg + tb0 + tt) * 4 + 2 * h + hi;
                const float4 b4 = s_bias[at], c4 = LN ? s_cs[at] : make_float4(0.f, 0.f, 0.f, 0.f);
                const float b[4] = {b4.x, b4.y, b4.z, b4.w}, c[4] = {c4.x, c4.y, c4.z, c4.w};
                const uint4 x4 = EPI == LE_RESID ? xr[i][tt][h] : make_uint4(0, 0, 0, 0);
                const float x[4] = {__uint_as_float(x4.x), __uint_as_float(x4.y), __uint_as_float(x4.z), __uint_as_float(x4.w)};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v = y[i][tt][4 * h + e];
                    if constexpr (LN) v = rstd * (v - mean * c[e]);
                    v += b[e];
                    if constexpr (EPI == LE_RESID) v += x[e];
                    y[i][tt][4 * h + e] = v;
                }
            }
        if constexpr (EPI == LE_RESID) {
            // statistics of the wave's 16 TB columns (a.sg_out) or of each 16: eight values here, eight in the lane 32 further on
            auto stats = [&](int t0, int nt, int at) {
                float mu = 0.f, sq = 0.f;
#pragma unroll
                for (int tt = 0; tt < TB; ++tt)
                    if (tt >= t0 && tt < t0 + nt)
                        mu += ((y[i][tt][0] + y[i][tt][1]) + (y[i][tt][2] + y[i][tt][3])) + ((y[i][tt][4] + y[i][tt][5]) + (y[i][tt][6] + y[i][tt][7]));
                mu = half_sum(mu) / (16 * nt);
#pragma unroll
                for (int tt = 0; tt < TB; ++tt)
                    if (tt >= t0 && tt < t0 + nt)
#pragma unroll
                        for (int e = 0; e < 8; ++e) sq += (y[i][tt][e] - mu) * (y[i][tt][e] - mu);
                sq = half_sum(sq);
                if (r[i] < R && hi == 0) a.stats_out[(size_t)r[i] * (a.N >> a.sg_out) + at] = make_float2(mu, sq);
            };
            if (a.sg_out > 4) stats(0, TB, (tile0 * 16) >> a.sg_out);
            else
#pragma unroll
                for (int tt = 0; tt < TB; ++tt) stats(tt, 1, tile0 + tt);
        }
#pragma unroll
        for (int tt = 0; tt < TB; ++tt)
            if (tile0 + tt < NT) store16<EPI>(a, r[i], (tile0 + tt) * 16, hi, y[i][tt], kv[i]);
    }
}

// ---------------------------------------------------------------------------
// Tree-masked attention (Sec. 2.1): one (sequence, head) and QT tiles of 16 query rows per workgroup.  Keys: cache
// positions [0, L) and the rows of this forward at L + m where the query's mask bit m is set (CAUSAL: rows 0 .. n of a
// prompt pass, which may have more rows than the mask table).  The waves take 32-key blocks round-robin with a
// private online softmax (S^T = K Q^T, O^T += V^T P^T on MFMA) and merge through LDS.  The cache keeps K and V^T in blocks
// of 32 keys, each already in the layout of the MFMA operands (kc_off / vc_off in common.h).
// QT = 2 where there are workgroups enough for every compute unit: a key block is then fetched once for 32 queries.
// (64 sequences of 32 nodes, ~330 keys: 24 us a layer instead of 34; with 64 workgroups instead of 128 for one sequence
// it takes 6.1 instead of 4.5.)
// NW waves take the key blocks of a workgroup in turn.  What bounds it with few workgroups: misses (a compute unit has no more than some
// 64 KB on their way; 512 KB of keys and values took 9 us), so the workgroups of a head start at different blocks (128 queries, 2000 keys
// 12.4 -> 10.3 us a layer, 64 queries, 360 keys 5.7 -> 5.3), and eight waves instead of four where there are blocks for them and the
// workgroups do not fill the chip (attn_shape; sixteen waves were slower than eight, 10.7 instead of 10.3).
// Measured and not kept: the key blocks split over up to four workgroups with the last
// to arrive merging (2000 keys, 64 queries: 8.6 instead of 9.7, 1000 keys: 8.2 instead of 6.9); two blocks per step
// (2000 keys: 9.3, 320 keys: 5.2 instead of 4.5).
// ---------------------------------------------------------------------------
// The block at which workgroup y of a head's `tiles` starts: floor(blocks y / tiles), exact while blocks tiles^2 < 2^32 (at most 64 tiles: 2^20 blocks of 32 keys; beyond, at
// most one more, which is still a block of the sequence).
__host__ __device__ inline uint32_t turn_magic(uint32_t tiles) { return tiles > 1 ? (uint32_t)(((1ull << 32) + tiles - 1) / tiles) : 0; }
__device__ __forceinline__ int turn_of(int blocks, uint32_t y, uint32_t magic) { return (int)mulhi((uint32_t)blocks * y, magic); }
struct AttnArgs {   // what the first loads need is in k_attn's leading arguments
    bf16_t* att;
    const int32_t* n_rows;
    const uint32_t* mask;
    int M;
    const int32_t* row0;     // causal pass: each sequence's first row (its rows are n_rows many)
    const float* x;          // causal pass, where only the sequences' last rows go on: the residual stream, and
    float* x_last;           // where its last rows go, one behind the other like the attention's results (null: all rows go on)
    int heads;               // workgroups of the first dimension from here on have nothing to attend to
    TouchList<3> ahead;
};
template <bool CAUSAL, int QT, int NW, int NB>   // NB: buffers of a wave, all but one of them in flight
__global__ __launch_bounds__(64 * NW, NB > 2 ? 1 : 4) void k_attn(const bf16_t* q, const bf16_t* Kc, const bf16_t* Vc, const int32_t* L_of, int n_heads, int nH, uint32_t nH_magic, int maxpos, int blocks, uint32_t y_magic, AttnArgs a) {
    constexpr int SO = 17;   // floats per row of the merge buffer: the merge reads a dimension's 16 queries' worth 64 rows apart
    __shared__ float sm_o[QT][NW * 64 * SO], sm_m[QT][NW * 16], sm_l[QT][NW * 16];
    const int bh = blockIdx.x;
    if (__builtin_expect(bh >= n_heads, 0)) {
        if constexpr (QT == 1)   // (two query tiles are taken where no compute unit is idle)
            if (bh >= a.heads) touch<NW>(a.ahead, a.heads, 1, nullptr);
        return;
    }
    const int b = nH_magic ? (int)mulhi((uint32_t)bh, nH_magic) : bh, h = bh - b * nH, L = ldg(L_of + b);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, gq = lane >> 4, c = lane & 15;
    const size_t hb = (size_t)bh * kv_cap(maxpos) * 64;
    const bf16_t *Kh = Kc + hb, *Vh = Vc + hb;
    uint4 buf[NB][8];
    auto load_at = [&](int at, uint4 (&kvb)[8]) {
        const uint32_t off = (uint32_t)at * 2048u + lane * 8u;
#pragma unroll
        for (int i = 0; i < 4; ++i) { kvb[i] = ldg4(Kh + (off + i * 512)); kvb[4 + i] = ldg4(Vh + (off + i * 512)); }
    };
    // The workgroups of a head start at different blocks: side by side they would all wait for the same lines from HBM, and a compute unit
    // has no more than some 64 KB of misses on their way; so each brings in a part that the others find in the L2.
    // A wave's first block is asked for before anything has been read from memory, from where it lies if the sequence has `blocks` blocks: the host's upper bound,
    // which is exact where every step's tokens are fetched.  It is no more than a guess where to read: which wave takes which block follows from the sequence's own
    // length, so the order of a result's sums depends neither on whether tokens were fetched nor on the other sequences (as long as attn_shape takes the same waves).  Without it the chain of loads is arguments, length, keys, 2900
    // clocks until the first keys are on their way, behind everything that the idle workgroups touch (with this and masks without branches, us per step: 64 nodes
    // 328 -> 325, 128 nodes and 2000 keys 443 -> 434, 16 x 64 nodes 930 -> 925, 64 x 32 nodes 1501 -> 1489).  Measured and not kept: 16 waves for up to 16
    // blocks (64 nodes 329), keys and values touched by the launch before (no change).
    int asked = -1;
    if constexpr (!CAUSAL) {
        asked = wave + turn_of(blocks, blockIdx.y, y_magic);
        if (asked >= blocks) asked = max(asked - blocks, 0);
        load_at(min(asked, (kv_cap(maxpos) >> 5) - 1), buf[0]);
        SCHED_FENCE();
    }
    int qt0 = blockIdx.y * QT;
    if constexpr (CAUSAL) {
        // Later queries see more keys.  Workgroups i and i + 256 share a compute unit: heavy ones first, in rounds of 256 that run to and fro.
        const int per = max(1, 256 / a.heads), round = blockIdx.y / per, at = blockIdx.y - round * per, left = min(per, (int)gridDim.y - round * per);
        qt0 = ((int)gridDim.y - 1 - (round * per + (round & 1 ? left - 1 - at : at))) * QT;
    }
    const int n_rows = ldg(a.n_rows + b);
    const int M = CAUSAL ? n_rows : a.M, row0 = CAUSAL ? ldg(a.row0 + b) : b * a.M;   // the sequence's rows
    const bool last_only = CAUSAL && a.x_last;
    if constexpr (CAUSAL) {
        if (last_only) {
            qt0 = (M - 1) >> 4;
            if (tid < 16) *(float4*)(a.x_last + (size_t)b * nH * 64 + h * 64 + 4 * tid) = *(const float4*)(a.x + (size_t)(row0 + M - 1) * nH * 64 + h * 64 + 4 * tid);
        }
        if (qt0 * 16 >= M) return;
    }
    int node[QT];
    bf16x8_t Q0[QT], Q1[QT];
    uint4 mw[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        node[t] = min((qt0 + t) * 16 + c, M - 1);
        Q0[t] = __builtin_bit_cast(bf16x8_t, ldg4(q + toff(row0 + node[t], h * 64 + 8 * gq, nH * 2)));
        Q1[t] = __builtin_bit_cast(bf16x8_t, ldg4(q + toff(row0 + node[t], h * 64 + 32 + 8 * gq, nH * 2)));
        mw[t] = make_uint4(0, 0, 0, 0);
        if constexpr (!CAUSAL) mw[t] = ldg4(a.mask + (size_t)node[t] * MASK_WORDS);
    }
    constexpr int DT = NW > 4 ? 2 : 4;   // the merge's outputs of a thread, per tile: dimensions d_out .. of query q_out
    const int q_out = tid / (64 / DT), d_out = tid % (64 / DT) * DT;
    auto put = [&](int nd, const float (&o)[DT]) {
        if (nd >= M || (last_only && nd != M - 1)) return;
        bf16_t* to = a.att + toff(last_only ? b : row0 + nd, h * 64 + d_out, nH * 2);
        if constexpr (DT == 4) *(uint2*)to = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
        else *(uint32_t*)to = pack_bf16(o[0], o[1]);
    };
    if (!CAUSAL && n_rows == 0) {   // a finished sequence
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            const float zero[DT] = {};
            put((qt0 + t) * 16 + q_out, zero);
        }
        return;
    }
    // (a causal pass: no query of the workgroup sees keys behind its last row)
    const int T = min(CAUSAL ? L + min((qt0 + QT) * 16, M) : L + M, maxpos);
    const int nblk = (T + 31) >> 5;
    const int turn = turn_of(nblk, blockIdx.y, y_magic);
    auto at_turn = [&](int i) { return i + turn < nblk ? i + turn : i + turn - nblk; };
    // Loads are unconditional, so that the waits count exactly the loads behind: past the last block every lane reads the same
    // 16 bytes, which is one line.
    auto load_block = [&](int blk, uint4 (&kvb)[8]) {
        const uint32_t off = blk < nblk ? (uint32_t)at_turn(blk) * 2048u + lane * 8u : 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) { kvb[i] = ldg4(Kh + (off + i * 512)); kvb[4 + i] = ldg4(Vh + (off + i * 512)); }
    };
    constexpr float SCALE = 0.125f * 1.44269504088896340736f;   // head dim 64; powers of two
    float m_run[QT], l_run[QT];
    f32x4_t O[QT][4];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        m_run[t] = -1e30f;
        l_run[t] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) O[t][i] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    }
    if (wave < nblk) {
        if (asked != at_turn(wave)) load_block(wave, buf[0]);
#pragma unroll
        for (int j = 1; j < NB - 1; ++j) load_block(wave + NW * j, buf[j]);
    }
    // Which of the eight keys m .. m + 7 of this forward (negative: committed ones) the lane's query sees, without a branch: bits of its
    // mask row, or in a causal pass keys up to its own.
    auto visible = [&](int t, int m) -> unsigned {
        if constexpr (CAUSAL) return (1u << max(0, min(8, node[t] + 1 - m))) - 1u;
        const int at = max(m, 0), before = min(8, at - m);
        const bool odd = at & 32, upper = at & 64;   // (selected in pairs: a chain of four cases becomes branches)
        const uint32_t l0 = odd ? mw[t].y : mw[t].x, l1 = odd ? mw[t].w : mw[t].z, h0 = odd ? mw[t].z : mw[t].y, h1 = odd ? 0u : mw[t].w;
        const uint32_t lo = upper ? l1 : l0, hi = upper ? h1 : h0;
        const uint32_t bits = at < 128 ? (uint32_t)((((uint64_t)hi << 32) | lo) >> (at & 31)) & 0xffu : 0u;
        return ((bits << before) | ((1u << before) - 1u)) & 0xffu;
    };
    auto process = [&](const int blk, const uint4 (&cur)[8]) {
        const int p0 = at_turn(blk) << 5, v0 = p0 + 8 * gq;
        uint32_t pk[QT][4];
        float m_new[QT], psum[QT];
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            f32x4_t sa = (f32x4_t){0.f, 0.f, 0.f, 0.f}, sb = sa;
            sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, cur[0]), Q0[t], sa, 0, 0, 0);
            sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, cur[1]), Q1[t], sa, 0, 0, 0);
            sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, cur[2]), Q0[t], sb, 0, 0, 0);
            sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, cur[3]), Q1[t], sb, 0, 0, 0);
            // this lane: query c, keys v0 + 0..3 (sa) and v0 + 4..7 (sb).  Instantiated twice: blocks inside the committed
            // cache need no mask tests.  The running maximum is of the unscaled scores; exp((s - m) / 8) = 2^(s c - m c).
            auto softmax_block = [&](const unsigned okm) {
                float mx = -1e30f, sc[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    sc[j] = (okm >> j) & 1u ? (j < 4 ? sa[j] : sb[j - 4]) : -INFINITY;   // (2^-inf is 0)
                    mx = fmaxf(mx, sc[j]);
                }
                m_new[t] = fmaxf(m_run[t], rows_max(mx));
                const float mc = m_new[t] * SCALE;
                psum[t] = 0.f;
#pragma unroll
                for (int j = 0; j < 8; j += 2) {
                    const float p0f = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[j], SCALE, -mc));
                    const float p1f = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[j + 1], SCALE, -mc));
                    psum[t] += p0f + p1f;
                    pk[t][j >> 1] = pack_bf16(p0f, p1f);
                }
            };
            if (p0 + 32 > L + (CAUSAL ? min((qt0 + t) * 16, M - 1) + 1 : 0)) {   // the block reaches into this forward's rows, behind the tile's first query (same for the whole wave)
                softmax_block(visible(t, v0 - L));
            } else {
                softmax_block(0xffu);
            }
        }
        bool moved = false;
#pragma unroll
        for (int t = 0; t < QT; ++t) moved |= m_new[t] != m_run[t];
        if (!__all(!moved)) {   // (after the first blocks the maxima rarely move)
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                const float corr = __builtin_amdgcn_exp2f((m_run[t] - m_new[t]) * SCALE);
                l_run[t] *= corr;
                m_run[t] = m_new[t];
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) O[t][dt] *= corr;
            }
        }
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            l_run[t] += psum[t];
            const bf16x8_t pfrag = __builtin_bit_cast(bf16x8_t, make_uint4(pk[t][0], pk[t][1], pk[t][2], pk[t][3]));
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
                O[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, cur[4 + dt]), pfrag, O[t][dt], 0, 0, 0);
        }
    };
    for (int blk = wave; blk < nblk; blk += NW * NB) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int bi = blk + NW * i;
            if (bi < nblk) {
                load_block(bi + NW * (NB - 1), buf[(i + NB - 1) % NB]);
                process(bi, buf[i]);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        l_run[t] = rows_sum(l_run[t]);
        if (gq == 0) { sm_m[t][wave * 16 + c] = m_run[t]; sm_l[t][wave * 16 + c] = l_run[t]; }
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) sm_o[t][(wave * 64 + dt * 16 + 4 * gq + i) * SO + c] = O[t][dt][i];
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        float mstar = sm_m[t][q_out];
#pragma unroll
        for (int w = 1; w < NW; ++w) mstar = fmaxf(mstar, sm_m[t][w * 16 + q_out]);
        float lsum = 0.f, o[DT] = {};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = __builtin_amdgcn_exp2f((sm_m[t][w * 16 + q_out] - mstar) * SCALE);
            lsum += f * sm_l[t][w * 16 + q_out];
#pragma unroll
            for (int j = 0; j < DT; ++j) o[j] += f * sm_o[t][(w * 64 + d_out + j) * SO + q_out];
        }
        const float inv = 1.f / lsum;
#pragma unroll
        for (int j = 0; j < DT; ++j) o[j] *= inv;
        put((qt0 + t) * 16 + q_out, o);
    }
}

// ---------------------------------------------------------------------------
// Tree expansion + embedding (Sec. 2.1), one workgroup per row: the fp32 residual stream, its bf16 copy in operand
// tiles and the statistics of each 16 columns.  In prefill mode the rows are consecutive prompt tokens: text ids are
// passed as -(id + 1), speech ids as they are.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_embed_rows(Dims D, DevState s, int prefill_mode, int table) {
    const int r = blockIdx.x, tid = threadIdx.x, b = prefill_mode ? ldg(s.row_seq + r) : r / D.M, n = r - (prefill_mode ? ldg(s.row0 + b) : b * D.M);
    const int rows = prefill_mode ? ldg(s.n_rows + b) : ldg(s.finished + b) ? 0 : D.M;
    if (!prefill_mode && n == 0 && tid == 0) s.n_rows[b] = rows;
    const bool valid = n < rows;
    int tok = 0, pos = 0;
    const bf16_t* E = (const bf16_t*)s.E_speech;
    if (valid) {
        if (prefill_mode) {
            const int t = ldg(s.chunk_tok + r);
            pos = ldg(s.L + b) + n;
            if (t < 0) { tok = -t - 1; E = (const bf16_t*)s.E_text; }
            else tok = t;
        } else {
            const int dep = ldg(s.t_depth[table] + n);
            pos = ldg(s.L + b) + dep;
            tok = n == 0 ? ldg(s.root + b) : ldg(s.draft_topk + ((size_t)b * D.Hh + (dep - 1)) * VADUSA_MAX_TOPK + ldg(s.t_rank[table] + n));
            // a row of logits without a largest entry (all NaN) leaves the arg-max and the draft lists without an
            // answer: whatever they hold then, the row read below is one of the table's
            if ((unsigned)tok >= (unsigned)D.V1) tok = 0;
        }
        if (pos >= D.maxpos) pos = D.maxpos - 1;   // the host checks capacity before launching
    }
    if (tid == 0) s.tok[r] = tok;
    const bf16_t* e = E + (size_t)tok * D.d;
    const bf16_t* p = (const bf16_t*)s.P + (size_t)pos * D.d;
    for (int c0 = tid * 4; c0 < D.d; c0 += 1024) {
        float v[4];
        const uint2 ev = ldg2(e + c0), pv = ldg2(p + c0);
        v[0] = bf2f((bf16_t)ev.x) + bf2f((bf16_t)pv.x);
        v[1] = bf2f((bf16_t)(ev.x >> 16)) + bf2f((bf16_t)(pv.x >> 16));
        v[2] = bf2f((bf16_t)ev.y) + bf2f((bf16_t)pv.y);
        v[3] = bf2f((bf16_t)(ev.y >> 16)) + bf2f((bf16_t)(pv.y >> 16));
        if (!valid) v[0] = v[1] = v[2] = v[3] = 0.f;
        const float mean = quad_sum(v[0] + v[1] + v[2] + v[3]) * (1.f / 16.f);
        const float m2 = quad_sum((v[0] - mean) * (v[0] - mean) + (v[1] - mean) * (v[1] - mean) + (v[2] - mean) * (v[2] - mean) + (v[3] - mean) * (v[3] - mean));
        *(float4*)(s.x + (size_t)r * D.d + c0) = make_float4(v[0], v[1], v[2], v[3]);
        *(uint2*)(s.xb + toff(r, c0, D.d >> 5)) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
        if ((tid & 3) == 0) ((float2*)s.stats)[(size_t)r * (D.d >> 4) + (c0 >> 4)] = make_float2(mean, m2);
    }
}

// ---------------------------------------------------------------------------
// After the vocabulary map: Algorithm 1 on every edge (one wave per edge, eight for long rows), Sec. 2.3's path choice with the continuation
// (one workgroup per sequence), and, after the draft heads' maps, their top-k lists beside the KV compaction.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_edges(Dims D, DevState s, int tau) {
    const int e = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
    if (e >= D.B * D.M) return;
    const int b = e / D.M, n = e - b * D.M;
    const int fin = ldg(s.finished + b), ok = (n == 0 || dev_edge_count<1>(D, s, b, n, threadIdx.x & 63) < tau) && !fin;   // (one chain of loads, not two)
    if ((threadIdx.x & 63) == 0) s.edge_ok[e] = ok;
}

// The same with eight waves per edge, for rows of more than 4096 logits: one wave goes to memory 15 times one after the other for
// 16 001 logits, eight waves twice (64 edges, us per launch: 18.1 -> 5.4).  Up to 4096 one wave needs at most four trips.
__global__ __launch_bounds__(512) void k_edges_wide(Dims D, DevState s, int tau) {
    __shared__ int s_cnt[8];
    const int e = blockIdx.x, b = e / D.M, n = e - b * D.M;
    const int fin = ldg(s.finished + b);
    const int cnt = n == 0 ? 0 : dev_edge_count<8>(D, s, b, n, threadIdx.x);
    if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        int sum = 0;
        for (int w = 0; w < 8; ++w) sum += s_cnt[w];
        s.edge_ok[e] = (n == 0 || sum < tau) && !fin;
    }
}

__global__ __launch_bounds__(256) void k_select(Dims D, DevState s, int seq0, int ignore_eos) {
    __shared__ PathLds p;
    dev_select(D, s, seq0 + blockIdx.x, ignore_eos, p);
}

// What bounds it: a chain of dependent loads in one workgroup per sequence.  Everything that does not depend on the path is asked for at
// the start, the path stays in LDS and the residual row is requested ahead of the row of logits; the results go to the host
// from here (us per launch, 64 nodes, 1025 logits: 11.7 -> 7.0 in a kernel trace, and no launch for the results).
template <class T>
__global__ __launch_bounds__(256) void k_continue(Dims D, DevState s, int seq0, int prefill_mode, int ignore_eos, int select, int32_t* host, int nseq, TouchList<2> ahead, size_t zw1, size_t zw2) {
    __shared__ PathLds p;
    if ((int)blockIdx.x >= nseq) {   // the draft heads' maps
        const size_t z_w[2] = {zw1, zw2};
        touch<4>(ahead, nseq, D.Hh, z_w);
        return;
    }
    const int b = seq0 + blockIdx.x;
    if (select) dev_select(D, s, b, ignore_eos, p);
    else if (!prefill_mode) dev_load_path(D, s, b, p);
    dev_finalize<T>(D, s, b, prefill_mode, ignore_eos, p, host);
}

// Workgroups below `lists`: one draft head's list of one sequence; the others: four heads (a wave each) of one
// sequence's cache over `layers` layers.  Sequences seq0 .. seq0 + nseq - 1 only: the lists of a sequence whose verification
// is still pending stay what that verification used.
template <class T>
__global__ __launch_bounds__(256) void k_lists_commit(Dims D, DevState s, int lists, int seq0, int nseq, int layers) {
    if ((int)blockIdx.x < lists) { dev_topk(D, s, blockIdx.x / nseq, seq0 + blockIdx.x % nseq); return; }
    const int u = (int)blockIdx.x - lists, hq = cdiv(D.nH, 4);
    const int head = (u % hq) * 4 + (int)(threadIdx.x >> 6), b = (u / hq) % nseq, layer0 = u / (hq * nseq) * layers;
    if (head < D.nH) dev_commit_kv_layers<T>(D, s, layer0, min(layers, D.Ly - layer0), seq0 + b, head, threadIdx.x & 63);
}

#ifdef VADUSA_CLOCK_BUILD
__global__ void k_clock(DevState s, int ph) { s.tprof[ph * 8] = wall_clock64(); }
#endif

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Tile shape of a map in k_lin.  The rule counts what a compute unit has to pull in through L2: a workgroup reads its rows and
// its columns of K values, and the 256 compute units get cdiv(workgroups, 256) of them each.
struct LinShape { int rt, ct; };
static int lin_rounds(int RT, int NT, const LinShape& s) { return cdiv(cdiv(RT, s.rt) * cdiv(NT, s.ct), 256); }
static LinShape lin_shape(int R, int NT) {
    static const LinShape shapes[] = {{1, 1}, {1, 2}, {2, 1}, {2, 2}, {2, 4}, {3, 4}, {4, 2}, {4, 4}};
    const int RT = cdiv(R, 16);
    auto cost = [&](const LinShape& s) { return lin_rounds(RT, NT, s) * (s.rt + s.ct); };
    LinShape best = shapes[0];
    for (const LinShape& s : shapes)
        if (cost(s) < cost(best)) best = s;
    return best;
}

// Workgroups of further columns of a grid that idle compute units can take.
static unsigned idle_columns(const dim3& grid) {
    const unsigned rows = grid.y * grid.z;
    return grid.x * rows < 256 ? (256 - grid.x * rows) / rows / 8 * 8 : 0;
}
// Pieces `from` .. of groups of so many bytes, as many as `pieces` allows.
static Touch touch_of(const void* W, uint32_t bytes, int groups, int from, long pieces) {
    const int take = groups > 0 ? (int)std::min<long>(cdiv(bytes, 8192) - from, pieces / groups) : 0;
    if (take <= 0) return Touch{};
    return Touch{(const char*)W + (size_t)from * 8192, bytes, bytes - from * 8192 - 128, (uint32_t)take, (uint32_t)(((1ull << 32) + take - 1) / take), groups};
}
// The maps of a forward in the order in which they are read, and how far they have been touched.  What a launch may touch is bounded by what it can hide: it ends
// when the last line has arrived.  Measured per idle workgroup (us per step of 1 | 64 nodes, 128 nodes and 2000 keys, 5 x 27 nodes):
// attention 80 KiB 263 | 320 | 453 | 432, 112 KiB 263 | 324 | 450 | 445, 160 KiB 264 | 323 | 445 | 439; so by the keys it has to go through.  A map's launch
// 32 KiB and 2 MiB in all; 6 MiB, 1 node 276; 1 MiB 265 | 327 | 454 | 438.  (All at d = 1024; what these bounds give at other widths stands at Touch.)
struct Ahead {
    struct Map { const void* W; uint32_t bytes; int groups; };   // bytes of a group; groups 0: not touched
    std::vector<Map> maps;
    size_t next = 0;
    int from = 0;   // pieces of each group of map `next` that have been
    void reading(size_t i) {
        if (next <= i) { next = i + 1; from = 0; }
    }
    template <int N>
    void take(TouchList<N>& t, int workgroups, int kib, int most_kib) {
        long pieces = std::min((long)workgroups * kib, (long)most_kib) / 8;
        for (int i = 0; i < N && next < maps.size();) {
            const Map& m = maps[next];
            if (m.groups > 0) {
                const Touch one = touch_of(m.W, m.bytes, m.groups, from, pieces);
                if (!one.groups) break;
                t.map[i++] = one;
                pieces -= (long)one.take * one.groups;
                from += one.take;
                if ((uint32_t)from * 8192u < m.bytes) break;
            }
            ++next;
            from = 0;
        }
    }
};

template <int RT, int CT, int CH, int EPI, int NW = 4>
static void lin_launch(LinArgs a, hipStream_t st, int nz = 1, Ahead* ahead = nullptr) {
    const int per_block = (size_t)a.R * a.nks * 64 <= (3u << 20) ? 65536 / cdiv(a.R, RT * 16) : 0;   // (while an L2 of 4 MiB holds what its workgroups read)
    dim3 grid(pad8(cdiv(a.NT, CT)), cdiv(a.R, RT * 16), nz);
    const unsigned idle = ahead ? idle_columns(grid) : 0;
    TouchList<2> t{};
    if (idle) ahead->take(t, idle * grid.y, 32, 2048);
    if (t.map[0].groups) grid.x += idle;
    launch(a.nks % (NW * CH) ? k_lin<RT, CT, CH, EPI, NW, false> : k_lin<RT, CT, CH, EPI, NW, true>, grid, dim3(64 * NW), 0, st, a.X, a.W, a.nks, a.NT, a.R, per_block, a.z_w, a.z_x, a, t);
}
// The tiles of `rows` rows x 16 `ct` columns; an XCD's eighth of them: about as many columns as rows.
static TileGrid tile_grid(const LinArgs& a, int rows, int ct) {
    TileGrid g{cdiv(a.R, rows), cdiv(a.NT, ct), 1};
    while (g.strip < g.gc && (long)g.strip * g.strip * ct * 16 * 8 < (long)g.gr * g.gc * rows) ++g.strip;
    g.n = g.gr * g.gc;
    g.gs = g.gr * g.strip;
    const bool exact = (long)g.n * g.gs < 1l << 32;   // (both divisors are at most gs and both dividends below n: dividend x error < 2^32)
    g.gs_magic = exact ? (uint32_t)(((1ull << 32) + g.gs - 1) / g.gs) : 0;
    g.strip_magic = exact ? (uint32_t)(((1ull << 32) + g.strip - 1) / g.strip) : 0;
    return g;
}
template <int EPI>
static void big_launch(LinArgs& a, hipStream_t st) {
    const TileGrid g = tile_grid(a, BIG_RT * 16, 4 * BIG_CT);
    a.sg_out = 5;
    launch(k_big<EPI>, EPI == LE_RESID ? dim3(8 * cdiv(g.gr * g.gc, 8)) : dim3(pad8(g.gc), g.gr), dim3(256), 0, st, a.X, a.W, a.stats, a.nks, a.NT, a.R, g.n, g.gs, g.gs_magic, g.strip, a, g);
}
template <int RG, int CG, int EPI>
static void tile_launch(LinArgs& a, hipStream_t st) {
    const TileGrid g = tile_grid(a, 64 * RG, 4 * CG);
    a.sg_out = TileShape<RG, CG>::KSP > 1 ? 5 : a.N % 128 ? 4 : 6;   // (a wave's columns as one entry where that leaves a row an even number)
    launch((k_tile<RG, CG, EPI>), dim3(8 * cdiv(g.n, 8)), dim3(512), 0, st, a.X, a.W, a.stats, a.nks, a.NT, a.R, g.n, g.gs, g.gs_magic, g.strip, a, g);
}
// Which kernel: the one that is estimated to take least.  us per launch, fitted to 1445 maps of whole steps, each run with all four kernels (widths
// of 64 to 1024 with hidden layers of two and four times that, 64 to 16 384 rows, vocabulary maps of 1025 and 16 001 columns): the choice takes
// 1.008 times the best of the four in the mean, 1.06 at the 95th percentile, 1.33 at most.  What the terms stand for: rounds of the fullest of the 256 compute units, where
// a map numbered by columns gives an XCD whole column groups (18 of them: three for two of the XCDs, two for the others); k_lin's workgroups are
// small and many, padding included, so that their number counts too; rows of logits are stored in pieces of four bytes.  An estimate fitted at K = 1024
// and 4096 alone was up to 4.3 times the best (us, choice and best: width 256, 1536 rows QKV k_lin 11.0, k_big 7.0; 4096 rows out-projection 11.1, 8.5,
// FFN2 19.0, 11.7; width 1024, 16 384 rows to 1025 logits k_big 151, k_tile 91).
// What it decides at d = 1024 (us: k_lin, k_big, k_tile 256 x 128, k_tile 128 x 64; the choice in brackets):
//   320 rows QKV [10.6] 13.1 22.7 12.5    FFN1 14.0 12.0 19.5 [11.7]    FFN2 [12.0] 32.1 49.5 24.7
//   1024     QKV 23.9 [17.7] 25.0 23.2    FFN1 27.6 [17.5] 22.5 23.4    FFN2 [19.2] 33.1 53.0 27.9    out-projection [9.7] 12.7 22.5 12.2
//   2048     QKV 43.5 [24.8] 27.3 33.7    FFN1 51.3 28.0 [25.5] 39.6    FFN2 34.4 35.6 54.2 [30.3]    out-projection 16.2 14.6 23.1 [13.6]
//   3200     QKV 68.6 [37.2] 46.7 51.3    FFN1 80.1 42.8 [42.3] 64.4    FFN2 60.6 [44.1] 54.0 49.1    out-projection 27.5 [18.9] 23.9 20.7
enum { MAP_LIN = 0, MAP_BIG, MAP_TILE_256, MAP_TILE_128 };
static int map_kernel(int R, int NT, int nks, int epi) {
    auto by_columns = [](int gr, int gc) { return cdiv(cdiv(gc, 8) * gr, 32); };
    auto by_blocks = [](int gr, int gc) { return cdiv(gr * gc, 256); };
    const LinShape s = lin_shape(R, NT);
    const int gr = cdiv(cdiv(R, 16), s.rt), gc = cdiv(NT, s.ct), nl = by_columns(gr, gc);
    const int nb = epi == LE_RESID ? by_blocks(cdiv(R, 64), cdiv(NT, 8)) : by_columns(cdiv(R, 64), cdiv(NT, 8));
    const float logits = epi == LE_LOGITS ? 1.f : 0.f;
    const float us[4] = {2.8f + 0.0014f * pad8(gc) * gr + nl * (0.188f * s.rt * s.ct + 0.0117f * nks * (s.rt + s.ct)),
                         2.5f + nb * (2.4f + 1.7f * logits) + nks * std::max(0.213f, 0.15f * nb),
                         1.9f + by_blocks(cdiv(R, 256), cdiv(NT, 8)) * (8.5f + 8.5f * logits + 0.43f * nks),
                         1.6f + by_blocks(cdiv(R, 128), cdiv(NT, 4)) * (5.f + 3.f * logits + 0.157f * nks)};
    return (int)(std::min_element(us, us + 4) - us);
}
// big_min (tests): k_big from that many of its tiles on; -1, -2: k_tile for every map.
template <int EPI>
static void lin(LinArgs& a, int big_min, Ahead* ahead, hipStream_t st) {
    a.sg_out = 4;
    const int kernel = big_min < 0 ? (big_min == -1 ? MAP_TILE_256 : MAP_TILE_128)
                       : big_min > 0 ? ((long)cdiv(a.R, 16 * BIG_RT) * cdiv(a.NT, 4 * BIG_CT) >= big_min ? MAP_BIG : MAP_LIN)
                                     : map_kernel(a.R, a.NT, a.nks, EPI);
    if (kernel == MAP_BIG) { big_launch<EPI>(a, st); return; }
    if (kernel == MAP_TILE_256) { tile_launch<4, 2, EPI>(a, st); return; }
    if (kernel == MAP_TILE_128) { tile_launch<2, 1, EPI>(a, st); return; }
    const LinShape s = lin_shape(a.R, a.NT);
    if constexpr (EPI == LE_LOGITS) {   // (with a multiple of four column tiles 1 x 2 and 2 x 4 never take more workgroups than these)
        if (s.rt == 2 && s.ct == 1) { lin_launch<2, 1, 8, EPI>(a, st, 1, ahead); return; }
        if (s.rt == 4 && s.ct == 2) { lin_launch<4, 2, 4, EPI>(a, st, 1, ahead); return; }
    }
    if constexpr (EPI == LE_RESID) {
        // Long reductions: eight waves, so that a compute unit's 128 to 256 KB are all in flight instead of half of them (K = 4096, us:
        // 64 rows 6.7 -> 6.5, 135 rows 10.0 -> 9.3, 320 rows 13.2 -> 12.8, 512 rows 13.6 -> 13.1; sixteen spill).
        if (a.nks >= 64) {
            switch (s.rt * 8 + s.ct) {
            case 1 * 8 + 1: lin_launch<1, 1, 8, EPI, 8>(a, st, 1, ahead); return;
            case 1 * 8 + 2: lin_launch<1, 2, 4, EPI, 8>(a, st, 1, ahead); return;
            case 2 * 8 + 2: lin_launch<2, 2, 4, EPI, 8>(a, st, 1, ahead); return;
            case 2 * 8 + 4: lin_launch<2, 4, 2, EPI, 8>(a, st, 1, ahead); return;
            default: break;
            }
        }
    }
    switch (s.rt * 8 + s.ct) {
    case 1 * 8 + 1: lin_launch<1, 1, 8, EPI>(a, st, 1, ahead); break;
    case 1 * 8 + 2: lin_launch<1, 2, 8, EPI>(a, st, 1, ahead); break;
    case 2 * 8 + 2: lin_launch<2, 2, EPI == LE_RESID ? 4 : 8, EPI>(a, st, 1, ahead); break;
    case 2 * 8 + 4: lin_launch<2, 4, 4, EPI>(a, st, 1, ahead); break;
    case 3 * 8 + 4: lin_launch<3, 4, 4, EPI>(a, st, 1, ahead); break;
    default: lin_launch<4, 4, 2, EPI>(a, st, 1, ahead); break;
    }
}

// Timing points (tprof[phase][0] = device clock ahead of the phase's launch): only in the library built with
// -DVADUSA_CLOCK_BUILD, where each is a launch of its own.
static void clock_point(const DevState& s, int ph, hipStream_t st) {
#ifdef VADUSA_CLOCK_BUILD
    if (ph < 128) launch(k_clock, dim3(1), dim3(1), 0, st, s, ph);
#else
    (void)s; (void)ph; (void)st;
#endif
}

struct AttnCall { const bf16_t *q, *Kc, *Vc; const int32_t* L; int B, M, nH, maxpos; AttnArgs a; };
template <int QT, int NW, int NB>
static void attn_launch(const AttnCall& t, bool causal, int keys, Ahead& ahead, hipStream_t st) {
    AttnArgs a = t.a;
    dim3 grid(pad8(t.B * t.nH), a.x_last ? 1 : cdiv(cdiv(t.M, 16), QT));
    a.heads = grid.x;
    const unsigned idle = QT == 1 ? idle_columns(grid) : 0;
    if (idle) ahead.take(a.ahead, idle * grid.y, 64 + std::min(keys / 22, 96), 24 << 10);   // (24 MiB: three of the 4 MiB of each of the eight L2s)
    if (a.ahead.map[0].groups) grid.x += idle;
    launch(causal ? k_attn<true, QT, NW, NB> : k_attn<false, QT, NW, NB>, grid, dim3(64 * NW), 0, st, t.q, t.Kc, t.Vc, t.L, t.B * t.nH, t.nH, (uint32_t)(t.nH > 1 ? ((1ull << 32) + t.nH - 1) / t.nH : 0),
           t.maxpos, cdiv(std::min(keys, t.maxpos), 32), turn_magic(grid.y), a);
}
// Query tiles and waves of a workgroup for `heads` heads (of all sequences) of qt query tiles and up to `keys` keys (an upper bound of the longest
// sequence's): two query tiles from two workgroups per compute unit on, else eight waves while every one has a key block to take and
// the workgroups do not fill the chip.  Measured in steps and prompt passes (us: one tile and four waves, one and eight, two and four;
// the choice in brackets):
//   64 queries, 360 | 2000 keys, 64 workgroups of one tile    5.4 [5.1] 7.8 | 11.7 [9.7] 15.6
//   64 queries of 8 sequences, 1100 keys, 512                 14.9 [14.0] 13.9
//   64 queries of 16 sequences, 350 | 2000 keys, 1024         12.7 12.0 [10.8] | 66 82 [40]
//   896 | 1024 causal queries, twice the keys, 896 | 1024     [16.8] 16.0 14.7 | 20.3 19.6 [16.8]
// Two tiles with eight waves lose to four wherever two tiles are taken (512 workgroups, 1100 | 2000 keys 28.4 | 47.6 against 23.6 | 39.8; 1024
// causal queries 18.0 against 16.8), three buffers for eight waves to two (128 queries, 1100 | 2000 | 3000 keys 7.6 | 10.1 | 12.8 against 7.2 | 9.3 | 12.6).
struct AttnShape { int tiles, waves; };
static AttnShape attn_shape(int heads, int qt, int keys, int big_min) {
    if (qt > 1 && heads * cdiv(qt, 2) >= (big_min > 0 ? big_min : 512)) return {2, 4};
    return {1, cdiv(keys, 32) >= 10 && heads * qt <= 512 ? 8 : 4};
}
static void attn(const AttnCall& t, bool causal, int keys, int big_min, Ahead& ahead, hipStream_t st) {
    const AttnShape s = attn_shape(t.B * t.nH, t.a.x_last ? 1 : cdiv(t.M, 16), keys, big_min);
    if (s.tiles == 2) attn_launch<2, 4, 3>(t, causal, keys, ahead, st);
    else if (s.waves == 8) attn_launch<1, 8, 2>(t, causal, keys, ahead, st);
    else attn_launch<1, 4, 3>(t, causal, keys, ahead, st);
}

void launch_layers(const Dims& D, const DevState& s, const std::vector<LayerW>& layers, int table, int prefill_mode, bool head, int big_min, hipStream_t st) {
    const int R = D.R, d = D.d;
    const size_t kv_layer = (size_t)D.Bmax * D.nH * kv_cap(D.maxpos) * 64;
    clock_point(s, 0, st);
    launch(k_embed_rows, dim3(R), dim3(256), 0, st, D, s, prefill_mode, table);
    LinArgs base{};
    base.R = R; base.L = s.L; base.n_rows = s.n_rows; base.row_seq = s.row_seq; base.row0 = s.row0; base.M = D.M; base.nH = D.nH; base.maxpos = D.maxpos; base.d = d;
    base.m_magic = D.M > 1 ? (uint32_t)(((1ull << 32) + D.M - 1) / D.M) : 0;
    base.stats = (const float2*)s.stats; base.sg = 4;   // (k_embed_rows)
    Ahead ahead;
    {
        auto map = [&](const void* W, int r, int N, int K, int epi) {
            const int NT = cdiv(N, 16), ct = lin_shape(r, NT).ct;
            const uint32_t bytes = (uint32_t)ct * (K >> 5) * 1024;
            ahead.maps.push_back({W, bytes, big_min || map_kernel(r, NT, K >> 5, epi) != MAP_LIN ? 0 : NT / ct});
        };
        const int rows = D.last_only ? D.B : R;   // behind the last layer's attention
        ahead.maps.reserve(4 * D.Ly + 1);
        for (const LayerW& w : layers) {
            const bool end = &w == &layers.back();
            const int r = end ? rows : R;
            map(w.Wqkv, R, 3 * d, d, LE_QKV);
            if (end && prefill_mode && !head) break;   // (as below)
            map(w.Wo, r, d, d, LE_RESID); map(w.W1, r, D.F, d, LE_GELU); map(w.W2, r, d, D.F, LE_RESID);
        }
        if (head) map(s.W_out, rows, D.V1, d, LE_LOGITS);
    }
    for (int l = 0; l < D.Ly; ++l) {
        const LayerW& w = layers[l];
        bf16_t *Kc = (bf16_t*)s.Kc + l * kv_layer, *Vc = (bf16_t*)s.Vc + l * kv_layer;
        LinArgs a = base;
        a.X = s.xb; a.W = (const uint4*)w.Wqkv; a.bias = w.t_qkv; a.colsum = w.cs_qkv; a.nks = d >> 5; a.N = 3 * d; a.NT = a.N >> 4;
        a.out = (bf16_t*)s.q; a.Kc = Kc; a.Vc = Vc;
        clock_point(s, 1 + 5 * l, st);
        ahead.reading(4 * l);
        lin<LE_QKV>(a, big_min, &ahead, st);
        const bool end = l + 1 == D.Ly;
        if (end && prefill_mode && !head) break;   // what follows the last layer's keys and values is for the vocabulary map
        AttnCall t{(const bf16_t*)s.q, Kc, Vc, s.L, D.B, D.M, D.nH, D.maxpos, {(bf16_t*)s.att, s.n_rows, s.t_mask[table], D.M, s.row0, s.x, nullptr, 0, {}}};
        float* x = s.x;
        if (end && D.last_only) x = t.a.x_last = (float*)s.hid;   // (free until FFN1)
        clock_point(s, 2 + 5 * l, st);
        attn(t, table == 1, D.keys, big_min, ahead, st);
        LinArgs o = base;
        o.X = (const bf16_t*)s.att; o.W = (const uint4*)w.Wo; o.bias = w.bo; o.nks = d >> 5; o.N = d; o.NT = d >> 4;
        o.out = s.xb; o.outf = s.x; o.stats_out = (float2*)s.stats;
        if (end && D.last_only) base.R = o.R = D.B;
        o.resid = x;
        clock_point(s, 3 + 5 * l, st);
        ahead.reading(4 * l + 1);
        lin<LE_RESID>(o, big_min, &ahead, st);
        base.sg = o.sg_out;
        LinArgs f = base;
        f.X = s.xb; f.W = (const uint4*)w.W1; f.bias = w.t_w1; f.colsum = w.cs_w1; f.nks = d >> 5; f.N = D.F; f.NT = D.F >> 4;
        f.out = (bf16_t*)s.hid;
        clock_point(s, 4 + 5 * l, st);
        ahead.reading(4 * l + 2);
        lin<LE_GELU>(f, big_min, &ahead, st);
        LinArgs g = base;
        g.X = (const bf16_t*)s.hid; g.W = (const uint4*)w.W2; g.bias = w.b2; g.nks = D.F >> 5; g.N = d; g.NT = d >> 4;
        g.out = s.xb; g.outf = s.x; g.resid = s.x; g.stats_out = (float2*)s.stats;
        clock_point(s, 5 + 5 * l, st);
        ahead.reading(4 * l + 3);
        lin<LE_RESID>(g, big_min, &ahead, st);
        base.sg = g.sg_out;
    }
    if (head) {
        LinArgs a = base;
        a.X = s.xb; a.W = (const uint4*)s.W_out; a.bias = s.t_out; a.colsum = s.cs_out; a.nks = d >> 5; a.N = D.V1; a.NT = cdiv(D.V1, 16);
        a.outf = s.logits;
        clock_point(s, 1 + 5 * D.Ly + TP_HEAD, st);
        ahead.reading(4 * D.Ly);
        lin<LE_LOGITS>(a, big_min, &ahead, st);
    }
}

void launch_verify_tail(const Dims& D, const DevState& s, int tau, int ignore_eos, bool select, hipStream_t st) {
    clock_point(s, 1 + 5 * D.Ly + TP_EDGES, st);
    if (D.M > 1) {
        if (D.V1 > 4096) launch(k_edges_wide, dim3(D.B * D.M), dim3(512), 0, st, D, s, tau);
        else launch(k_edges, dim3(cdiv(D.B * D.M, 4)), dim3(256), 0, st, D, s, tau);
    }
    if (select) launch(k_select, dim3(D.B), dim3(256), 0, st, D, s, 0, ignore_eos);
}

// Rows of more than 4096 logits: the draft lists come from the stand-alone top-k kernel (1024 threads hold a row of 16 384; the 256
// of dev_topk hold 4096).
void launch_continue(const Dims& D, const DevState& s, const std::vector<DraftW>& draft, int seq0, int nseq, int prefill_mode, int ignore_eos, bool select, int32_t* host, int dtype, hipStream_t st) {
    const int H = 1 + 5 * D.Ly;
    clock_point(s, H + TP_FINAL, st);
    auto ahead = [&](const void* a, const void* b) { return D.Hh > 1 ? (size_t)((const char*)b - (const char*)a) : 0; };
    const DraftW &d0 = draft[0], &d1 = draft[D.Hh > 1 ? 1 : 0];
    const size_t zw1 = ahead(d0.W1, d1.W1), zw2 = ahead(d0.W2, d1.W2);
    TouchList<2> t{};   // the draft heads' maps (us per step: 1 node 267.2 -> 265.0, 64 nodes 325.4 -> 324.0)
    unsigned idle = dtype ? idle_columns(dim3(nseq)) : 0;
    const long pieces = (long)idle * 10 / D.Hh;
    t.map[0] = touch_of(d0.W1, (D.d >> 5) * 1024, D.d >> 4, 0, pieces);
    t.map[1] = touch_of(d0.W2, (D.d >> 5) * 1024, cdiv(D.V1, 16), 0, pieces - (long)t.map[0].take * t.map[0].groups);
    if (!t.map[0].groups) idle = 0;
    launch(dtype ? k_continue<bf16_t> : k_continue<float>, dim3(nseq + idle), dim3(256), 0, st, D, s, seq0, prefill_mode, ignore_eos, select ? 1 : 0, host, nseq, t, zw1, zw2);
    if (dtype) {
        LinArgs a{};
        a.X = (const bf16_t*)s.hbest; a.W = (const uint4*)d0.W1; a.bias = d0.b1; a.nks = D.d >> 5; a.N = D.d; a.NT = D.d >> 4; a.R = D.B;
        a.out = (bf16_t*)s.rdraft; a.z_w = zw1; a.z_b = ahead(d0.b1, d1.b1); a.z_out = s.draft_stride;
        clock_point(s, H + TP_COMMIT, st);
        if (D.B <= 16) lin_launch<1, 1, 8, LE_SILU>(a, st, D.Hh);
        else lin_launch<4, 1, 4, LE_SILU>(a, st, D.Hh);
        LinArgs z{};
        z.X = (const bf16_t*)s.rdraft; z.W = (const uint4*)d0.W2; z.nks = D.d >> 5; z.N = D.V1; z.NT = cdiv(D.V1, 16); z.R = D.B;
        z.outf = s.zdraft; z.z_w = zw2; z.z_x = s.draft_stride; z.z_out = (size_t)D.Bmax * D.V1;
        clock_point(s, H + TP_DRAFT2, st);
        if (D.B <= 16) lin_launch<1, 1, 8, LE_F32>(z, st, D.Hh);
        else lin_launch<4, 1, 4, LE_F32>(z, st, D.Hh);
    } else {
        launch_draft32(D, s, draft, seq0, nseq, st);
    }
    clock_point(s, H + TP_TOPK, st);
    const int lists = D.V1 > 4096 ? 0 : D.Hh * nseq, per_layer = cdiv(D.nH, 4) * nseq;
    const int layers = std::min(D.Ly, std::max(1, cdiv(D.Ly * per_layer, 256)));   // (layers per workgroup: one round of the 256 compute units)
    const int commits = prefill_mode ? 0 : cdiv(D.Ly, layers) * per_layer;
    if (lists + commits > 0) launch(dtype ? k_lists_commit<bf16_t> : k_lists_commit<float>, dim3(lists + commits), dim3(256), 0, st, D, s, lists, seq0, nseq, layers);
    if (lists == 0) launch_topk(D, s, seq0, nseq, st);
}
