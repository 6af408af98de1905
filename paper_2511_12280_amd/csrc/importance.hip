// d3tom_importance: decider-guided importance map (Section 3.2, "The Decider-Guided Mechanism";
// Algorithm 1, the line that forms S).
//
// S_j = (1/H) sum_h sum_{i in D} softmax_j(scale * q_{i,h} . k_{j,h}), softmax over ALL keys of the
// sample, written for the visual columns only.  The N x N matrix is never formed: only the |D|
// decider rows are ever evaluated.  Large decider sets take two sweeps over K (below); small ones keep
// the D x N x H logits of the first sweep and finish from those (imp_scores_from_logits; the generic path keeps probabilities):
//
//   sweep 1 (stats)   per (head, decider): running max and sum of exp2 over all keys, computed per
//                     chunk of keys by one workgroup each and combined later in a fixed order
//   sweep 2 (scores)  per (head, visual key): sum over deciders of exp2(logit - logsumexp), one row
//                     per head; a small third kernel adds the H rows in head order (no atomics)
//
// bf16 path: logits on MFMA 16x16x32.  Either a workgroup has its keys in registers, read straight from HBM/L2 in the MFMA operand
// layout, and the decider rows pass through LDS; or (large launches with many deciders) the decider rows are in registers and the keys
// pass through LDS.  K is streamed twice, the second time from the memory-side cache if it fits.
//
// The generic path (any float type / head size) is a kernel pair in plain float arithmetic.
#include <mutex>
#include <type_traits>
#include "internal.hpp"
#include "direct_load.hpp"

namespace d3tom {

// Keys per workgroup: 4 waves x SUB sub-tiles x 16.  Every workgroup fetches the decider rows of its head, so few large chunks (one
// workgroup per CU at 3.7k tokens x 32 heads) beat many small ones; when 512-key chunks would leave CUs idle (short sequences)
// the first sweep takes 256-key chunks instead (8.5 instead of 11.5 us at 1152 tokens).  The second sweep has no statistics to
// amortise: 256 (x 64 deciders x 32 heads: 11.3 -> 9.8 us).  With several rounds of such workgroups and more deciders than keep
// their logits, loads and arithmetic of a workgroup that fetches all its keys at once add up: there the keys stream
// through LDS (imp_stream_bf16).
constexpr int IMP_KC_STATS = 512, IMP_KC_SCORES = 256;
constexpr long IMP_MANY = 1024;        // 512-key chunks from which on a launch counts as several rounds
constexpr int IMP_STREAM_KEYS = 4096, IMP_STREAM_HEADS = 1024;     // a chunk's rows are addressed with 32-bit byte offsets
// Streaming launches: from how many deciders on, workgroups they should have, keys of a workgroup at least (the decider rows and the
// first stages are paid once in each).  Both sweeps, against keys at once, 2924 drawn batches of 2 to 32 samples of 500 to 4000 tokens, 8 to 32
// heads of 64 and 128, by the largest decider count: 129 .. 143 0.99 x, 144 .. 159 1.01, 160 .. 175 1.04, to 223 1.06, to 239 1.08, 240 .. 256
// 1.11 (single batches 0.85 to 1.36); with few of them the sweeps are bound by the keys, of which the other form has more in flight (16 samples of
// 1200 .. 2300 tokens, at most 38 deciders 97 us at once and 104 streaming, 77 105 and 113, 127 111 and 116, 254 167 and 149).  On the same batches
// 1024 or 2048 workgroups instead of 1536, or 640 keys instead of 448, change the mean by at most 0.6 % (single batches by 21 % either way),
// 896 keys lose up to 3 %.
constexpr int IMP_STREAM_D = 144, IMP_STREAM_WGS = 1536, IMP_STREAM_MIN = 448;

constexpr int IMP_KEEP_MAXD_WS = 32;   // largest decider set whose logits are kept (workspace is sized for it)
struct ImpWs {
    size_t part_off, sp_off, c_off, logit_off, total;
    int KC, KCS, NCH, NCHV, DPAD, VPAD, NKB;
    bool many;
};
__host__ inline ImpWs imp_ws_layout(int B, int max_N, int max_V, int H, int max_D, bool many) {
    ImpWs w;
    const long chunks = (long)ceil_div(max_N, IMP_KC_STATS) * H * B;
    // keys per chunk of the first sweep and of the second
    auto stream_chunk = [&](int keys) {
        const int want = ceil_div(IMP_STREAM_WGS, H * B < IMP_STREAM_WGS ? H * B : IMP_STREAM_WGS), most = keys < 2 * IMP_STREAM_MIN ? 1 : keys / IMP_STREAM_MIN;
        const int cuts = want < most ? want : most;
        const int c = ceil_div(ceil_div(keys, cuts), 64) * 64;
        return c < IMP_STREAM_KEYS ? c : IMP_STREAM_KEYS;
    };
    w.many = many;
    w.KC = many ? stream_chunk(max_N) : chunks < 256 ? IMP_KC_STATS / 2 : IMP_KC_STATS;
    w.KCS = many ? stream_chunk(max_V) : IMP_KC_SCORES;
    w.NCH = ceil_div(max_N, w.KC);
    w.NCHV = ceil_div(max_V, w.KCS);
    w.DPAD = ceil_div(max_D, 16) * 16;
    w.VPAD = w.NCHV * w.KCS;
    size_t o = 0;
    w.part_off = o; o += align_up((size_t)B * H * w.NCH * w.DPAD * sizeof(float2), 256);
    w.sp_off = o;   o += align_up((size_t)B * H * w.VPAD * sizeof(float), 256);
    w.c_off = o;    o += align_up((size_t)B * H * max_D * sizeof(float), 256);   // generic path
    w.NKB = w.NCH * (w.KC / 16);
    w.logit_off = o;                                                              // kept logits (small decider sets)
    if (max_D <= IMP_KEEP_MAXD_WS) o += align_up((size_t)B * w.NKB * H * max_D * 16 * sizeof(float), 256);
    w.total = o;
    return w;
}
// The two forms pad statistics and per-head rows differently: where only one of them fits the library's static array, it is that one.
// Both entry points follow this rule, so that their scores are the same bits.
__host__ inline ImpWs imp_ws_layout(int B, int max_N, int max_V, int H, int max_D) {
    const ImpWs w = imp_ws_layout(B, max_N, max_V, H, max_D, false);
    if ((long)ceil_div(max_N, IMP_KC_STATS) * H * B < IMP_MANY || max_D <= IMP_KEEP_MAXD_WS || H > IMP_STREAM_HEADS) return w;
    const ImpWs m = imp_ws_layout(B, max_N, max_V, H, max_D, true);
    const size_t lim = D3TOM_IMPORTANCE_STATIC_BYTES;
    if (max_D <= IMP_STREAM_D) return (w.total > lim && m.total <= lim) ? m : w;
    return (m.total > lim && w.total <= lim) ? w : m;
}
size_t importance_ws_bytes(int B, int max_N, int max_V, int H, int dh, int max_D) {
    (void)dh;
    // a workspace sized for a bound on the decider count must also serve every smaller count: small sets
    // keep their logits, which can take more room than the statistics of a large set
    const size_t a = imp_ws_layout(B, max_N, max_V, H, max_D).total;
    const size_t b = imp_ws_layout(B, max_N, max_V, H, max_D < IMP_KEEP_MAXD_WS ? max_D : IMP_KEEP_MAXD_WS).total;
    return a > b ? a : b;
}

// MFMA operand fragments of SUB x 16 key rows of one head, straight from memory: lane (r = lane % 16, g = lane / 16) takes elements
// [kk*32 + g*8, +8) of its row for k-step kk, so the four lanes of a row fetch 64 contiguous bytes per
// load instruction.  `first` = the workgroup's first row, of which `rows` exist; others (and rows past the end) read as zeros.
template <int DH, int SUB>
__device__ __forceinline__ void load_keys(const uint16_t* first, int rows, int H, int row0, int r, int g, bf16x8 (&f)[SUB][DH / 32]) {
#if defined(__HIP_DEVICE_COMPILE__)
    const int row_bytes = H * DH * 2;
    const __amdgpu_buffer_rsrc_t rsrc = make_uniform_rsrc(first, (uint32_t)(rows - 1) * row_bytes + DH * 2);
    const int voff = (row0 + r) * row_bytes + g * 16;
#pragma unroll
    for (int s = 0; s < SUB; ++s)
#pragma unroll
        for (int kk = 0; kk < DH / 32; ++kk)
            f[s][kk] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff + kk * 64, s * 16 * row_bytes, 0));
#endif
}

// The decider rows of one head, [16 * nblk rows][DH] with 16-byte chunks swizzled by the row, go to LDS once per workgroup, by
// direct loads that run beside those of the keys; rows past the sample's deciders repeat the last one.  (Fetched by every wave
// for itself, 64 rows at a time, they cost a trip to memory per 64 rows in each of them.)  At most IMP_QROWS of them at a time, so
// that LDS leaves room for as many workgroups as the registers do.  Positions first, keys behind them, rows last: `positions` and
// `rows` are called around the key loads.
constexpr int IMP_QROWS = 128, IMP_QBLK = IMP_QROWS / 16;
template <int DH>
struct ImpQueries {
    static constexpr int ROWB = DH * 2, NCHK = DH / 8, RPI = 64 / NCHK, MAXL = IMP_QROWS / RPI / 4;
    int pos[MAXL];                          // as they were loaded
    __device__ __forceinline__ static int swizzle(int x) { return DH == 128 ? (x & 15) : ((x >> 1) & 7); }
    // rows i0 .. i0 + 16 * nblk - 1
    __device__ __forceinline__ void positions(const int32_t* dec, int i0, int D) {
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
        for (int u = 0; u < MAXL; ++u) pos[u] = dec[min(i0 + (wave + 4 * u) * RPI + lane / NCHK, D - 1)];
    }
    __device__ __forceinline__ void rows(const uint16_t* q, int tok0, int N, int H, int h, int nblk, char* lds) {
#if defined(__HIP_DEVICE_COMPILE__)
        // All positions were requested, wanted or not, and are waited for here: loads under the condition below were each waited for in it, one trip
        // to memory behind the other and the keys behind them all (first sweep over 3773 tokens, 64 deciders 11.6 -> 11.0 us, 1152 tokens, 32 deciders
        // 6.5 -> 6.0, second sweep 9.2 -> 8.6 with the statistics in front).
#pragma unroll
        for (int u = 0; u < MAXL; ++u) asm volatile("" : "+v"(pos[u]));
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
#pragma unroll
        for (int u = 0; u < MAXL; ++u) {
            const int l = wave + 4 * u;
            if (l * RPI < nblk * 16) {
                const int x = l * RPI + lane / NCHK;
                const uint16_t* p = q + ((size_t)(tok0 + min(max(pos[u], 0), N - 1)) * H + h) * DH + (((lane % NCHK) ^ swizzle(x)) << 3);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                                 (lds_ptr_t)(lds + l * 1024), 16, 0, 0);
            }
        }
#endif
    }
    // operand fragments of decider rows blk * 16 + r
    __device__ __forceinline__ static void fragments(const char* lds, int blk, int r, int g, bf16x8 (&f)[DH / 32]) {
        const char* p = lds + (blk * 16 + r) * ROWB;
#pragma unroll
        for (int kk = 0; kk < DH / 32; ++kk) f[kk] = *reinterpret_cast<const bf16x8*>(p + (((kk * 4 + g) ^ swizzle(r)) << 4));
    }
};
// block(blk, fragments) for every 16-decider block; AHEAD: the next one's fragments are read before it (where registers allow)
template <int DH, bool AHEAD, typename F>
__device__ __forceinline__ void imp_for_blocks(const char* lds, int nblk, int r, int g, F&& block) {
    bf16x8 f0[DH / 32], f1[DH / 32];
    if constexpr (!AHEAD) {
#pragma unroll 1
        for (int blk = 0; blk < nblk; ++blk) {
            ImpQueries<DH>::fragments(lds, blk, r, g, f0);
            block(blk, f0);
        }
    } else {
        ImpQueries<DH>::fragments(lds, 0, r, g, f0);
#pragma unroll 1
        for (int blk = 0; blk < nblk; blk += 2) {
            ImpQueries<DH>::fragments(lds, min(blk + 1, nblk - 1), r, g, f1);
            block(blk, f0);
            if (blk + 1 >= nblk) break;
            ImpQueries<DH>::fragments(lds, min(blk + 2, nblk - 1), r, g, f0);
            block(blk + 1, f1);
        }
    }
}

// log2-sum-exp2 of a decider row from the statistics of its nch chunks of keys (of which `first` has up to eight), summed around the
// common maximum of eight chunks at a time, in ascending order.  LEAVE: a branch at every chunk instead of a selection (for 16 waves that have
// nothing else to do; with keys under way it costs 0.4 us).
template <bool LEAVE>
__device__ __forceinline__ float imp_lse(float2 (&first)[8], const float2* p, int nch, int NCH, int DPAD) {
    float m = -INFINITY, z = 0.f;
    for (int c0 = 0;;) {
        float mn = m;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (LEAVE && c0 + u >= nch) break;               // uniform
            mn = fmaxf(mn, c0 + u < nch ? first[u].x : -INFINITY);
        }
        const float ref = (mn == -INFINITY) ? 0.f : mn;      // nothing but empty chunks so far
        z *= __builtin_amdgcn_exp2f(m - ref);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (LEAVE && c0 + u >= nch) break;
            z += c0 + u < nch ? first[u].y * __builtin_amdgcn_exp2f(first[u].x - ref) : 0.f;
        }
        m = mn;
        c0 += 8;
        if (c0 >= nch) break;
#pragma unroll
        for (int u = 0; u < 8; ++u) first[u] = p[(size_t)min(c0 + u, NCH - 1) * DPAD];
    }
    return m + __builtin_amdgcn_logf(z);
}

// (running max, running sum of exp2) of decider rows over one chunk of IMP_SUB_STATS x 64 keys of one head
template <int DH, bool KEEP, int IMP_SUB_STATS>
__global__ __launch_bounds__(256, 2) void imp_stats_bf16(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, int H, float scale2,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ dec_idx, const int32_t* __restrict__ dec_off,
    int max_D, int DPAD, int NCH, float2* __restrict__ part, int NKB, float* __restrict__ logits) {
    constexpr int KS = DH / 32;
    // heads vary fastest over the grid: workgroups that run together read neighbouring 2*DH-byte pieces of the same key rows
    const int h = blockIdx.x, chunk = blockIdx.y, b = blockIdx.z;
    constexpr int KC = IMP_SUB_STATS * 64;
    int tok0 = seq_off[b], tok1 = seq_off[b + 1], d0 = dec_off[b], d1 = dec_off[b + 1];
    request_together(tok0, tok1, d0, d1);
    const int N = min(tok1 - tok0, NCH * KC);                         // the workspace holds NCH chunks per head
    const int D = min(d1 - d0, max_D);
    const int32_t* dec = dec_idx + d0;
    const int key_base = chunk * KC;
    if (key_base >= N || D <= 0) return;

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int nblk = (D + 15) >> 4;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* qs = smem;                                                    // the decider rows
    float2* wstat = reinterpret_cast<float2*>(smem + min(DPAD, IMP_QROWS) * DH * 2);   // [4 waves][4 key groups][min(DPAD, IMP_QROWS)]
    const int wrows = min(DPAD, IMP_QROWS);

    ImpQueries<DH> queries;
    queries.positions(dec, 0, D);
    bf16x8 kf[IMP_SUB_STATS][KS];
    const int wave_key = key_base + wave * IMP_SUB_STATS * 16;
    load_keys<DH, IMP_SUB_STATS>(k + ((size_t)(tok0 + key_base) * H + h) * DH, min(N - key_base, KC), H, wave * IMP_SUB_STATS * 16, r, g, kf);
    queries.rows(q, tok0, N, H, h, min(nblk, IMP_QBLK), qs);
    const bool ragged = wave_key + IMP_SUB_STATS * 16 > N;              // uniform: some of the wave's keys lie past the end
    for (int b0 = 0; b0 < nblk; b0 += IMP_QBLK) {
    const int nb = min(nblk - b0, IMP_QBLK);
    if (b0 > 0) queries.rows(q, tok0, N, H, h, nb, qs);
    __syncthreads();
    if (b0 + IMP_QBLK < nblk) queries.positions(dec, (b0 + IMP_QBLK) * 16, D);
    imp_for_blocks<DH, true>(qs, nb, r, g, [&](int blk, const bf16x8 (&qf)[KS]) {
        // acc[s][e]: logit of decider (b0 + blk) * 16 + r and key 4 g + e of sub-tile s
        f32x4 acc[IMP_SUB_STATS];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
#pragma unroll
            for (int s = 0; s < IMP_SUB_STATS; ++s) {
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[s][kk], qf[kk], kk ? acc[s] : zero, 0, 0, 0);
            }
        if (ragged) {
#pragma unroll
            for (int s = 0; s < IMP_SUB_STATS; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (wave_key + s * 16 + 4 * g + e >= N) acc[s][e] = -INFINITY;
        }
        if constexpr (KEEP) {
            // [key block][head][decider][key in block]: a lane stores four keys of its decider, a wave 1 KB in one piece
            const int row = (b0 + blk) * 16 + r;
#pragma unroll
            for (int s = 0; s < IMP_SUB_STATS; ++s) {
                acc[s] *= scale2;
                const int kb = (key_base >> 4) + wave * IMP_SUB_STATS + s;
                if (row < D) *reinterpret_cast<f32x4*>(logits + (((size_t)(b * NKB + kb) * H + h) * max_D + row) * 16 + 4 * g) = acc[s];
            }
        }
        // maximum of this lane's keys first, then one exp2 per logit; lanes and waves meet at the end
        float m = acc[0][0];
#pragma unroll
        for (int s = 0; s < IMP_SUB_STATS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) m = fmaxf(m, acc[s][e]);
        const float scl = KEEP ? 1.f : scale2, ms = m * scl;
        const float ref = (m == -INFINITY) ? 0.f : ms;                  // no key at all: the sum stays 0
        float z = 0.f;
#pragma unroll
        for (int s = 0; s < IMP_SUB_STATS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) z += __builtin_amdgcn_exp2f(KEEP ? acc[s][e] - ref : __builtin_fmaf(acc[s][e], scale2, -ref));
        wstat[(wave * 4 + g) * wrows + blk * 16 + r] = make_float2(ms, z);
    });
    __syncthreads();
    for (int t = threadIdx.x; t < nb * 16; t += 256) {
        float2 a[16];
#pragma unroll
        for (int w = 0; w < 16; ++w) a[w] = wstat[w * wrows + t];
        float m = a[0].x, z = 0.f;
#pragma unroll
        for (int w = 1; w < 16; ++w) m = fmaxf(m, a[w].x);
        // Every logit of the chunk is -inf or NaN: it counts as empty, (-inf, 0), so that a row of NaN alone has no sum, -inf for its logarithm and
        // NaN for its probabilities.
        const bool empty = !(m > -INFINITY);
        const float ref = empty ? 0.f : m;
#pragma unroll
        for (int w = 0; w < 16; ++w) z += a[w].y * __builtin_amdgcn_exp2f(a[w].x - ref);
        part[((size_t)(b * H + h) * NCH + chunk) * DPAD + b0 * 16 + t] = empty ? make_float2(-INFINITY, 0.f) : make_float2(m, z);
    }
    }
}

// per-head score rows: sp[h][j] = sum over deciders of exp2(logit - log2sumexp2)
template <int DH>
__global__ __launch_bounds__(256, 4) void imp_scores_bf16(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, int H, float scale2,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ dec_idx, const int32_t* __restrict__ dec_off,
    const int32_t* __restrict__ vis_start, const int32_t* __restrict__ vis_count,
    int max_D, int max_V, int DPAD, int NCH, int KC, int VPAD, const float2* __restrict__ part, float* __restrict__ sp) {
    constexpr int KS = DH / 32, IMP_SUB_SCORES = 4, KCS = IMP_SUB_SCORES * 64;
    // heads vary fastest over the grid: workgroups that run together read neighbouring 2*DH-byte pieces of the same key rows
    const int h = blockIdx.x, chunk = blockIdx.y, b = blockIdx.z;
    int tok0 = seq_off[b], tok1 = seq_off[b + 1], d0 = dec_off[b], d1 = dec_off[b + 1], vs0 = vis_start[b], vc = vis_count[b];
    // The statistics (a decider to a thread) are requested with the offsets, the keys with the deciders' positions, and the
    // statistics are put together while those are under way.
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r = lane & 15, g = lane >> 4;
    const float2* p = part + ((size_t)(b * H + h) * NCH) * DPAD + min(tid, DPAD - 1);
    float2 a[8];                                                        // chunks of keys requested at once
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] = p[(size_t)min(u, NCH - 1) * DPAD];
#pragma unroll
    for (int u = 0; u < 8; ++u) asm volatile("" : "+v"(a[u]));          // or the compiler requests them behind the keys
    request_together(tok0, tok1, d0, d1, vs0, vc);
    const int N = min(tok1 - tok0, NCH * KC);
    const int D = min(d1 - d0, max_D);
    const int32_t* dec = dec_idx + d0;
    const int vs = min(max(vs0, 0), N);
    const int V = min(min(vc, max_V), N - vs);
    const int key_base = chunk * KCS;
    if (key_base >= V || D <= 0) return;

    const int nblk = (D + 15) >> 4;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* qs = smem;                                                    // the decider rows
    float* c_lds = reinterpret_cast<float*>(smem + min(DPAD, IMP_QROWS) * DH * 2);     // [DPAD] log2-sum-exp2

    ImpQueries<DH> queries;
    queries.positions(dec, 0, D);
    bf16x8 kf[IMP_SUB_SCORES][KS];
    float acc_s[IMP_SUB_SCORES];
    load_keys<DH, IMP_SUB_SCORES>(k + ((size_t)(tok0 + vs + key_base) * H + h) * DH, min(V - key_base, KCS), H,
                                  wave * IMP_SUB_SCORES * 16, r, g, kf);
    static_assert(D3TOM_MAX_DECIDERS <= 256, "a thread for every decider");
    if (wave * 64 < nblk * 16) {
        // log2-sum-exp2 of every decider row of this head, key chunks combined in ascending order
        const int nch = (N + KC - 1) / KC;
        const float c = imp_lse<false>(a, p, nch, NCH, DPAD);
        if (tid < nblk * 16) c_lds[tid] = tid < D ? c : INFINITY;       // padded rows contribute exp2(-inf) = 0
    }
#pragma unroll
    for (int s = 0; s < IMP_SUB_SCORES; ++s) acc_s[s] = 0.f;
    queries.rows(q, tok0, N, H, h, min(nblk, IMP_QBLK), qs);
    for (int b0 = 0; b0 < nblk; b0 += IMP_QBLK) {
    const int nb = min(nblk - b0, IMP_QBLK);
    if (b0 > 0) {
        __syncthreads();
        queries.rows(q, tok0, N, H, h, nb, qs);
    }
    __syncthreads();
    if (b0 + IMP_QBLK < nblk) queries.positions(dec, (b0 + IMP_QBLK) * 16, D);
    imp_for_blocks<DH, false>(qs, nb, r, g, [&](int blk, const bf16x8 (&qf)[KS]) {
        const f32x4 cc = *reinterpret_cast<const f32x4*>(c_lds + (b0 + blk) * 16 + 4 * g);
        f32x4 acc[IMP_SUB_SCORES];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
#pragma unroll
            for (int s = 0; s < IMP_SUB_SCORES; ++s) {
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[kk], kf[s][kk], kk ? acc[s] : zero, 0, 0, 0);
            }
#pragma unroll
        for (int s = 0; s < IMP_SUB_SCORES; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc_s[s] += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[s][e], scale2, -cc[e]));
    });
    }
    float* sp_row = sp + (size_t)(b * H + h) * VPAD;
#pragma unroll
    for (int s = 0; s < IMP_SUB_SCORES; ++s) {
        float v = acc_s[s];
        v += __shfl_xor(v, 16, WAVE);
        v += __shfl_xor(v, 32, WAVE);
        if (g == 0) sp_row[key_base + (wave * IMP_SUB_SCORES + s) * 16 + r] = v;
    }
}

// Both sweeps of large launches: the keys of a chunk go through a ring of 64-key stages in LDS, the decider rows stay in registers, a
// quarter of the 16-decider blocks per wave.  Key loads run beside the arithmetic, each key row is fetched once per workgroup, each
// decider row once, and the statistics of a decider live in one lane column from the first key to the last.
//   SCORES = false: D = K Q^T, lane (r, g) = decider r, keys 4 g + e of every 16: running maximum and sum over the chunk
//   SCORES = true:  D = Q K^T, lane (r, g) = key r, deciders 4 g + e: sum over the deciders; the four waves' sums of a stage meet in LDS
// 16 samples of 2688 tokens, 169 deciders on average: 115 -> 98 and 99 -> 77 us, 3.6 and 3.9 TB/s.  The loads alone take 58 us, the
// arithmetic alone 75 (480 clocks per block and stage for two waves of a SIMD, 452 of them vector issue); together the card's clock
// falls to 1.63 GHz, and the order of heavy and light samples no longer matters.
constexpr int IMP_NS = 4;                   // stages in the ring
constexpr float IMP_NONE = -3.0e38f;        // the maximum of no logits
constexpr int IMP_WBLK = D3TOM_MAX_DECIDERS / 64;      // 16-decider blocks of a wave at most
template <int DH, bool SCORES>
__global__ __launch_bounds__(256, 2) void imp_stream_bf16(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, int H, float scale2,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ dec_idx, const int32_t* __restrict__ dec_off,
    const int32_t* __restrict__ vis_start, const int32_t* __restrict__ vis_count,
    int max_D, int max_V, int DPAD, int NCH, int KC, int KCS, int VPAD, float2* __restrict__ part, float* __restrict__ sp) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int KS = DH / 32, ROWB = DH * 2, NCHK = DH / 8, RPI = 64 / NCHK, LD = 64 / RPI / 4, STAGE = 64 * ROWB;
    __shared__ __attribute__((aligned(16))) char ring[IMP_NS * STAGE];
    __shared__ float c_lds[SCORES ? D3TOM_MAX_DECIDERS : 1];            // log2-sum-exp2 of the deciders
    __shared__ float sums[SCORES ? 2 : 1][4][64];                       // [stage parity][wave][key]
    // heads vary fastest over the grid: workgroups that run together read neighbouring 2*DH-byte pieces of the same key rows
    const int h = blockIdx.x, chunk = blockIdx.y, b = blockIdx.z;
    int tok0 = seq_off[b], tok1 = seq_off[b + 1], d0 = dec_off[b], d1 = dec_off[b + 1], vs0 = vis_start[b], vc = vis_count[b];
    request_together(tok0, tok1, d0, d1, vs0, vc);
    const int N = min(tok1 - tok0, NCH * KC);                         // the workspace holds NCH chunks per head
    const int D = min(d1 - d0, max_D);
    const int32_t* dec = dec_idx + d0;
    const int vs = min(max(vs0, 0), N);
    const int V = min(min(vc, max_V), N - vs);
    const int key_base = chunk * (SCORES ? KCS : KC);
    const int keys = SCORES ? min(V - key_base, KCS) : min(N - key_base, KC);      // of this chunk
    if (keys <= 0 || D <= 0) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const int nblk = (D + 15) >> 4;
    // this wave's blocks: w0, w0 + 4, ...; which wave has one more than others goes by the head
    const int w0 = (wave + h) & 3, nb = (nblk - w0 + 3) >> 2;

    const int row_bytes = H * ROWB;
    const __amdgpu_buffer_rsrc_t rk = make_uniform_rsrc(k + ((size_t)(tok0 + (SCORES ? vs : 0) + key_base) * H + h) * DH,
                                                        (uint32_t)(keys - 1) * (uint32_t)row_bytes + ROWB);    // rows past the chunk read as 0
    auto swizzle = [](int x) { return DH == 128 ? (x & 15) : ((x >> 1) & 7); };
    const uint32_t ring0 = (uint32_t)(size_t)(lds_ptr_t)ring;
    int k_off[LD];
#pragma unroll
    for (int i = 0; i < LD; ++i) {
        const int x = (wave * LD + i) * RPI + lane / NCHK;
        k_off[i] = x * row_bytes + (((lane % NCHK) ^ swizzle(x)) << 4);
    }
    auto issue = [&](int j) {
#pragma unroll
        for (int i = 0; i < LD; ++i)
            direct_load_16(rk, k_off[i] + j * 64 * row_bytes, ring0 + (j % IMP_NS) * STAGE + (wave * LD + i) * 1024);
    };
    int pos[IMP_WBLK];
#pragma unroll
    for (int i = 0; i < IMP_WBLK; ++i) pos[i] = min(max(dec[min((w0 + 4 * i) * 16 + r, D - 1)], 0), N - 1);
    issue(0);
    issue(1);
    issue(2);
    static_assert(IMP_NS == 4, "three stages ahead");
    bf16x8 qf[IMP_WBLK][KS];
#pragma unroll
    for (int i = 0; i < IMP_WBLK; ++i)
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
            qf[i][kk] = *reinterpret_cast<const bf16x8*>(q + ((size_t)(tok0 + pos[i]) * H + h) * DH + kk * 32 + g * 8);
    f32x4 cc[IMP_WBLK];                     // SCORES: log2-sum-exp2 of deciders 4 g + e of each block
    if constexpr (SCORES) {
        const int nch = (N + KC - 1) / KC;
        for (int t = threadIdx.x; t < nblk * 16; t += 256) {
            const float2* p = part + ((size_t)(b * H + h) * NCH) * DPAD + t;
            float m = -INFINITY, z = 0.f;
            for (int c0 = 0; c0 < nch; c0 += 4) {          // 4 independent loads in flight, combined in order
                float2 a[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) a[u] = p[(size_t)min(c0 + u, nch - 1) * DPAD];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (c0 + u < nch) lse2_combine_fast(m, z, a[u].x, a[u].y);
            }
            c_lds[t] = t < D ? m + __builtin_amdgcn_logf(z) : INFINITY;     // padded rows contribute exp2(-inf) = 0
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < IMP_WBLK; ++i) cc[i] = *reinterpret_cast<const f32x4*>(c_lds + min(w0 + 4 * i, nblk - 1) * 16 + 4 * g);
    }
    // running maximum of the raw logits (a value below every logit until there is one) and sum, of this lane's keys
    float m[IMP_WBLK], z[IMP_WBLK];
#pragma unroll
    for (int i = 0; i < IMP_WBLK; ++i) { m[i] = IMP_NONE; z[i] = 0.f; }
    int f_addr[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) f_addr[kk] = r * ROWB + (((kk * 4 + g) ^ swizzle(r)) << 4);
    float* sp_row = sp + (size_t)(b * H + h) * VPAD + key_base;

    const int nst = (keys + 63) >> 6;
    // one loop for each number of blocks, without branches between them
    auto sweep = [&](auto nb_c) {
    constexpr int NB = decltype(nb_c)::value;
#pragma unroll 1
    for (int j = 0; j < nst; ++j) {
        // stage j is there (later ones stay in flight), and everybody is done with stage j - 1
        wait_loads<2 * LD>();
        __builtin_amdgcn_s_waitcnt(0xC07F);
        phase_barrier();
        issue(j + 3);                       // past the last stage: rows of the buffer's end, zeros
        if (SCORES && j > 0 && wave == (j & 3)) {
            const float* s = &sums[(j - 1) & 1][0][lane];
            sp_row[(j - 1) * 64 + lane] = (s[0] + s[64]) + (s[128] + s[192]);
        }
        const char* st = ring + (j % IMP_NS) * STAGE;
        bf16x8 kf[4][KS];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) kf[s][kk] = *reinterpret_cast<const bf16x8*>(st + s * 16 * ROWB + f_addr[kk]);
        const bool ragged = !SCORES && (j + 1) * 64 > keys;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            f32x4 acc[4];
#pragma unroll
            for (int kk = 0; kk < KS; ++kk)
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                    acc[s] = SCORES ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[i][kk], kf[s][kk], kk ? acc[s] : zero, 0, 0, 0)
                                    : __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[s][kk], qf[i][kk], kk ? acc[s] : zero, 0, 0, 0);
                }
            if constexpr (SCORES) {
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[s] += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[s][e], scale2, -cc[i][e]));
            } else {
                if (ragged) {
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (j * 64 + s * 16 + 4 * g + e >= keys) acc[s][e] = -INFINITY;
                }
                float t = m[i];
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) t = fmaxf(t, acc[s][e]);
                float zi = z[i] * __builtin_amdgcn_exp2f((m[i] - t) * scale2);
                m[i] = t;
                const float ms = t > IMP_NONE ? t * scale2 : 0.f;      // no key yet: the sum stays 0
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) zi += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[s][e], scale2, -ms));
                z[i] = zi;
            }
        }
        if constexpr (SCORES) {
            // over the four lane groups: after the exchanges lane l has the sum of key l of the stage
            typedef unsigned u2 __attribute__((ext_vector_type(2)));
            auto swap_add = [](float a, float c, bool wide) {
                const u2 x = wide ? __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(c), false, false)
                                  : __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(c), false, false);
                return __uint_as_float(x[0]) + __uint_as_float(x[1]);
            };
            sums[j & 1][wave][lane] = swap_add(swap_add(v[0], v[2], true), swap_add(v[1], v[3], true), false);
        }
    }
    };
    static_assert(IMP_WBLK == 4, "five cases");
    switch (nb) {
        case 0: sweep(std::integral_constant<int, 0>()); break;
        case 1: sweep(std::integral_constant<int, 1>()); break;
        case 2: sweep(std::integral_constant<int, 2>()); break;
        case 3: sweep(std::integral_constant<int, 3>()); break;
        default: sweep(std::integral_constant<int, 4>());
    }
    wait_loads<0>();                        // nothing may be in flight into LDS when the workgroup ends
    if constexpr (SCORES) {
        __syncthreads();
        if (wave == (nst & 3)) {
            const float* s = &sums[(nst - 1) & 1][0][lane];
            sp_row[(nst - 1) * 64 + lane] = (s[0] + s[64]) + (s[128] + s[192]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < IMP_WBLK; ++i) {
            if (i >= nb) break;
            float mq = m[i], zq;
            mq = fmaxf(mq, __shfl_xor(mq, 16, WAVE));
            mq = fmaxf(mq, __shfl_xor(mq, 32, WAVE));
            zq = z[i] * __builtin_amdgcn_exp2f((m[i] - mq) * scale2);
            zq += __shfl_xor(zq, 16, WAVE);
            zq += __shfl_xor(zq, 32, WAVE);
            if (g == 0) part[((size_t)(b * H + h) * NCH + chunk) * DPAD + (w0 + 4 * i) * 16 + r] = make_float2(mq * scale2, zq);
        }
    }
#endif
}

// Small decider sets (at most IMP_KEEP_MAXD): the first sweep also writes its scaled logits, D x N x H
// floats (a quarter of K's bytes at 16 deciders), in blocks of [16 keys' block][head][decider][16 keys], and
// the scores come from those instead of a second sweep over K: one workgroup per 16-key block reads its
// contiguous H x D x 64 bytes, subtracts each (head, decider) row's log-sum-exp and adds the exponentials
// over deciders and heads, so the mean over heads is finished in the same pass (no per-head rows, no
// third launch, K fetched once).
// Bound by the chain request -> statistics -> exponentials -> reduction, so it has 16 waves: every thread holds one or two
// (head, decider) rows of the statistics and at most 16 logits at 32 heads x 32 deciders, all requested at once.  (Statistics behind the
// logits and offsets, each chunk rescaling the sum before it: 1024 rows of 1152 keys 5.6 us, then 5.0, and 4.6 without conditions for rows
// that every sample has; 208 of 817 3.7, 3.3, 3.2.  Blocks of 8 keys on
// twice as many compute units 5.2.)
// Unrolled for 1, 4 or 16 (head, decider) rows a thread: rows that a block does not have cost their instructions all the same, in four
// waves per SIMD (16 for all against these: 64 rows of 208 keys 4.2 -> 2.7 us (float32), of 3773 4.8 -> 3.4, 208 rows of 817 4.6 -> 3.7).
constexpr int IMP_KEEP_MAXD = IMP_KEEP_MAXD_WS;
constexpr int IMP_FL_THREADS = 1024, IMP_FL_GROUPS = IMP_FL_THREADS / 16;
template <int IMP_FL_ROWS>
__global__ __launch_bounds__(IMP_FL_THREADS) void imp_scores_from_logits(
    int H, const int32_t* __restrict__ seq_off, const int32_t* __restrict__ dec_off,
    const int32_t* __restrict__ vis_start, const int32_t* __restrict__ vis_count, const int32_t* __restrict__ score_off,
    int max_D, int max_V, int DPAD, int NCH, int KC, int NKB, const float2* __restrict__ part, const float* __restrict__ logits,
    float* __restrict__ scores) {
#if defined(__HIP_DEVICE_COMPILE__)
    const int kb = blockIdx.x, b = blockIdx.y;
    int tok0 = seq_off[b], tok1 = seq_off[b + 1], d0 = dec_off[b], d1 = dec_off[b + 1], vs0 = vis_start[b], vc = vis_count[b], s0 = score_off[b];
    request_together(tok0, tok1, d0, d1, vs0, vc, s0);
    const int N = min(tok1 - tok0, NCH * KC);
    const int D = min(d1 - d0, max_D);
    const int vs = min(max(vs0, 0), N);
    const int V = min(min(vc, max_V), N - vs);
    const int key0 = kb * 16;
    constexpr int PASS = IMP_FL_ROWS * IMP_FL_GROUPS;   // rows of a pass
    // log2-sum-exp2, +inf for rows past the sample's deciders and the block's rows; the rows of a thread side by side
    extern __shared__ __attribute__((aligned(16))) float c_lds[];
    __shared__ float red[IMP_FL_THREADS / 64][16];
    __shared__ int odd[IMP_FL_THREADS / 64];            // a wave met a row of the sample whose sum of exponentials is not finite
    // thread (key = t % 16, group = t / 16) takes rows group, group + 64, ... of the block's H x max_D logit rows: 64
    // consecutive rows are 4 KB in one piece.  They, the statistics and the sample's offsets are requested together (they come from another
    // XCD's writes, i.e. from memory): no request depends on an offset, what a sample does not have is left out when it is there.
    const int key = threadIdx.x & 15, grp = threadIdx.x >> 4;
    const int rows = H * max_D;
    const __amdgpu_buffer_rsrc_t lb = make_uniform_rsrc(logits + ((size_t)(b * NKB + kb) * rows) * 16, (uint32_t)rows * 64u);   // rows past the block's read as 0
    float l[IMP_FL_ROWS];
    auto request = [&](int r0) {
#pragma unroll
        for (int u = 0; u < IMP_FL_ROWS; ++u)
            l[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(lb, threadIdx.x * 4u, (uint32_t)(r0 + u * IMP_FL_GROUPS) * 64u, 0));
    };
    request(0);
    // the statistics of row t: head t / max_D (exact: (t + 1/2) / max_D is 1/64 or more away from the integers, t below 12288), decider the rest
    const float per_head = __builtin_amdgcn_rcpf((float)max_D);
    float2 a[8];                                            // chunks of keys requested at once
    int i = 0;
    const float2* p = nullptr;
    auto statistics = [&](int t) {
        const int h = (int)(((float)t + 0.5f) * per_head);
        i = t - h * max_D;
        p = part + ((size_t)(b * H + h) * NCH) * DPAD + i;
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = p[min(u, NCH - 1) * DPAD];
    };
    const int wave0 = __builtin_amdgcn_readfirstlane((int)threadIdx.x & ~63);
    if (wave0 < rows) statistics(min((int)threadIdx.x, rows - 1));
    if (D <= 0 || key0 >= vs + V || key0 + 16 <= vs || key0 >= N) return;
    const int nch = min((N + KC - 1) / KC, NCH);
    const int padded = (rows + PASS - 1) / PASS * PASS;
    bool bad = false;
    for (int t0 = wave0; t0 < padded;) {
        const int t = t0 + ((int)threadIdx.x & 63);
        float c = INFINITY;
        if (t0 < rows) {
            const float lse = imp_lse<true>(a, p, nch, NCH, DPAD);
            c = t < rows && i < D ? lse : INFINITY;
            bad |= t < rows && i < D && !(lse < INFINITY);
        }
        c_lds[t / PASS * PASS + (t % IMP_FL_GROUPS) * IMP_FL_ROWS + t % PASS / IMP_FL_GROUPS] = c;
        t0 += IMP_FL_THREADS;
        if (t0 < rows) statistics(min(t0 + ((int)threadIdx.x & 63), rows - 1));
    }
    odd[threadIdx.x >> 6] = __builtin_amdgcn_ballot_w64(bad) != 0;
    __syncthreads();
    float acc = 0.f;
    // (16 waves on four SIMDs: an instruction for every row of every thread is 20 clocks x 16.  Most samples have all of the launch's rows.)
    const bool whole = D == max_D && rows == padded && __builtin_amdgcn_ballot_w64(odd[threadIdx.x & 15] != 0) == 0;
    auto add_rows = [&](int r0) {
        const float* c = c_lds + r0 + grp * IMP_FL_ROWS;
        if (whole) {
#pragma unroll
            for (int u = 0; u < IMP_FL_ROWS; ++u) acc += __builtin_amdgcn_exp2f(l[u] - c[u]);
        } else {
            // a row past the sample's deciders was never written: whatever it holds must not reach the sum (nor does a row whose logits went
            // beyond float32)
#pragma unroll
            for (int u = 0; u < IMP_FL_ROWS; ++u) acc += (c[u] < INFINITY) ? __builtin_amdgcn_exp2f(l[u] - c[u]) : 0.f;
        }
    };
    add_rows(0);
    for (int r0 = PASS; IMP_FL_ROWS == 16 && r0 < rows; r0 += PASS) {     // more than 1024 rows
        request(r0);
        add_rows(r0);
    }
    acc = quad_combine(acc, [](float x, float y) { return x + y; });
    if ((threadIdx.x & 63) < 16) red[threadIdx.x >> 6][key] = acc;
    __syncthreads();
    const int j = key0 + (int)threadIdx.x - vs;          // visual index of key threadIdx.x of this block
    if (threadIdx.x < 16 && j >= 0 && j < V) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < IMP_FL_THREADS / 64; ++w) sum += red[w][threadIdx.x];      // waves in ascending order
        scores[s0 + j] = sum / (float)H;
    }
#endif
}

// S_j = mean over heads of the per-head rows, heads added in ascending order
__global__ __launch_bounds__(256) void imp_finish_kernel(
    const float* __restrict__ sp, int H, int VPAD, const int32_t* __restrict__ seq_off,
    const int32_t* __restrict__ vis_start, const int32_t* __restrict__ vis_count, const int32_t* __restrict__ score_off,
    int max_V, float* __restrict__ scores) {
#if defined(__HIP_DEVICE_COMPILE__)
    const int b = blockIdx.y, j = blockIdx.x * 256 + threadIdx.x;
    int tok0 = seq_off[b], tok1 = seq_off[b + 1], vs0 = vis_start[b], vc = vis_count[b], s0 = score_off[b];
    float a[32];                                           // 32 independent loads in flight, added in head order
    auto request = [&](int h0) {                           // heads behind the last read as 0
        const __amdgpu_buffer_rsrc_t rows = make_uniform_rsrc(sp + (size_t)(b * H + h0) * VPAD, (uint32_t)(min(H - h0, 32) * VPAD) * 4u);
#pragma unroll
        for (int u = 0; u < 32; ++u) a[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows, (uint32_t)(u * VPAD + j) * 4u, 0, 0));
    };
    request(0);                                            // with the offsets, not behind them: without the next line the compiler puts them there
#pragma unroll
    for (int u = 0; u < 32; u += 8)
        asm volatile("" : "+v"(a[u]), "+v"(a[u + 1]), "+v"(a[u + 2]), "+v"(a[u + 3]), "+v"(a[u + 4]), "+v"(a[u + 5]), "+v"(a[u + 6]), "+v"(a[u + 7]));
    request_together(tok0, tok1, vs0, vc, s0);
    const int N = tok1 - tok0;
    const int vs = min(max(vs0, 0), N);
    const int V = min(min(vc, max_V), N - vs);
    if (j >= V) return;
    float s = 0.f;
    for (int h0 = 0;;) {
#pragma unroll
        for (int u = 0; u < 32; ++u) s += a[u];
        h0 += 32;
        if (h0 >= H) break;
        request(h0);
    }
    scores[s0 + j] = s / (float)H;
#endif
}

// ---------------------------------------------------------------------------------------------
// generic path: one workgroup per (decider, head) for the stats; it has all logits of its row of the softmax and leaves the probabilities
// of a small decider set, whose scores are then sums over (head, decider) rows; one per 8 visual keys for the scores of larger sets.
// Plain float arithmetic, any head size up to 256.  Bound by latency: a wave takes 64 keys at a time, 16 lanes to a key (208 keys x 4 heads x
// 16 deciders of 64 floats 5.0 us with a key to a lane, 3.8 so), and there are waves for up to 1024 keys at once (256 keys at once:
// 420 keys x 72 rows 5.1 us, now 4.8; 576 x 36 8.2, now 6.9).
// ---------------------------------------------------------------------------------------------
template <typename T, int THREADS>
__global__ __launch_bounds__(THREADS) void imp_stats_generic(
    const T* __restrict__ q, const T* __restrict__ k, int H, int dh, float scale2,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ dec_idx, const int32_t* __restrict__ dec_off,
    int max_D, int NK, float* __restrict__ probs, float* __restrict__ cws) {
    const int i = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    int tok0 = seq_off[b], tok1 = seq_off[b + 1], d0 = dec_off[b], d1 = dec_off[b + 1];
    request_together(tok0, tok1, d0, d1);
    const int N = tok1 - tok0, kept = min(N, NK);
    const int D = min(d1 - d0, max_D);
    float* row = probs + ((size_t)(b * H + h) * max_D + i) * NK;       // if there are any
    if (i >= D) {                                          // no such decider in this sample: it adds nothing
        if (probs)
            for (int j = threadIdx.x; j < kept; j += THREADS) row[j] = 0.f;
        return;
    }
    __shared__ float2 red[THREADS / 64];
    const int pos = min(max(dec_idx[d0 + i], 0), N - 1);
    const T* qr = q + ((size_t)(tok0 + pos) * H + h) * dh;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    float m = -INFINITY, z = 0.f, first = 0.f;             // first: the logit of this thread's first key (the others wait in `row`)
    for (int j0 = wave * 64; j0 < N; j0 += THREADS) {
        const int j = j0 + wave_dots_row(lane);
        float dot[1];
        wave_row_dots<T, 1>({qr}, k + ((size_t)(tok0 + j0) * H + h) * dh, (size_t)H * dh, N - j0, dh, lane, dot);
        const float s = dot[0] * scale2;
        if (j < N) {
            if (j0 < THREADS) first = s;
            else if (probs && j < kept) row[j] = s;
            lse2_combine(m, z, s, 1.0f);
        }
    }
    const float mw = wave_max(m);
    z = wave_sum(m == -INFINITY ? 0.f : z * exp2f(m - mw));
    if (lane == 0) red[wave] = make_float2(mw, z);
    __syncthreads();
    float2 a = red[0];
    for (int w = 1; w < THREADS / 64; ++w) lse2_combine(a.x, a.y, red[w].x, red[w].y);
    const float c = a.x + log2f(a.y);
    if (!probs) {
        if (threadIdx.x == 0) cws[(size_t)(b * H + h) * max_D + i] = c;
        return;
    }
    for (int j0 = wave * 64; j0 < kept; j0 += THREADS) {
        const int j = j0 + wave_dots_row(lane);
        if (j < kept) row[j] = c < INFINITY ? exp2f((j0 < THREADS ? first : row[j]) - c) : 0.f;      // (a row whose logits went beyond float32 adds nothing)
    }
}

// Scores from the probabilities: a workgroup has 64 visual keys, a wave a quarter of the rows (375 keys x 72 rows 3.2 us; with every score's
// dot products formed again 7.5 us for 144 x 64).
__global__ __launch_bounds__(256) void imp_sum_generic(ScoreSums s, const int32_t* __restrict__ seq_off, const int32_t* __restrict__ vis_count,
                                                       const int32_t* __restrict__ score_off, int max_V, float* __restrict__ scores) {
    const int b = blockIdx.y, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    int tok0 = seq_off[b], tok1 = seq_off[b + 1], vs0 = s.vis_start[b], vc = vis_count[b], s0 = score_off[b];
    request_together(tok0, tok1, vs0, vc, s0);
    const int N = tok1 - tok0, vs = min(max(vs0, 0), N), V = min(min(vc, max_V), N - vs);
    const int j = blockIdx.x * 64 + lane;
    if ((int)blockIdx.x * 64 >= V) return;
    __shared__ float part[SUM_PARTS][64];
    part[wave][lane] = score_sum_part<32>(s, b, vs + min(j, V - 1), wave);
    __syncthreads();
    if (wave == 0 && j < V) scores[s0 + j] = score_of_parts(part[0][lane], part[1][lane], part[2][lane], part[3][lane], s.H);
}

// One workgroup per 8 visual keys: thread = (key, one of 32 groups), the groups take the (head, decider) pairs in turn,
// 16-byte loads.  (One thread per key looping over every head, decider and channel was one serial chain of H * D * dh
// scalar loads on a single compute unit: 363 us at 144 keys x 4 heads x 16 deciders x 64; this takes 7.7 us.)
constexpr int IMG_KEYS = 8, IMG_GROUPS = 256 / IMG_KEYS;
template <typename T>
__global__ __launch_bounds__(256) void imp_scores_generic(
    const T* __restrict__ q, const T* __restrict__ k, int H, int dh, float scale2,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ dec_idx, const int32_t* __restrict__ dec_off,
    const int32_t* __restrict__ vis_start, const int32_t* __restrict__ vis_count, const int32_t* __restrict__ score_off,
    int max_D, int max_V, const float* __restrict__ cws, float* __restrict__ scores) {
    const int b = blockIdx.y;
    const int key = threadIdx.x % IMG_KEYS, grp = threadIdx.x / IMG_KEYS;
    const int j = blockIdx.x * IMG_KEYS + key;
    const int tok0 = seq_off[b];
    const int N = seq_off[b + 1] - tok0;
    const int D = min(dec_off[b + 1] - dec_off[b], max_D);
    const int vs = min(max(vis_start[b], 0), N);
    const int V = min(min(vis_count[b], max_V), N - vs);
    if (blockIdx.x * IMG_KEYS >= V || D <= 0) return;
    __shared__ float red[4][IMG_KEYS];
    const T* kr = k + (size_t)(tok0 + vs + min(j, V - 1)) * H * dh;
    float acc = 0.f;
    for (int p = grp; p < H * D; p += IMG_GROUPS) {
        const int h = p / D, i = p - h * D;
        const int pos = min(max(dec_idx[dec_off[b] + i], 0), N - 1);
        const float s = row_dot<T>(q + ((size_t)(tok0 + pos) * H + h) * dh, kr + h * dh, dh);
        // The logit to the same bits as in the sum of exponentials, rounded where it is rounded there: its rounding, which grows with it, then drops
        // out of the probability of a key that has most of the row.  (300 tokens x 4 heads x 48 deciders of 64 floats: 1.2e-7 off
        // against float64; with the products added in another order 2.6e-7.)
        {
#pragma clang fp contract(off)
            const float s2 = s * scale2;
            acc += exp2f(s2 - cws[(size_t)(b * H + h) * max_D + i]);
        }
    }
#pragma unroll
    for (int o = IMG_KEYS; o < 64; o <<= 1) acc += __shfl_xor(acc, o, WAVE);
    if ((threadIdx.x & 63) < IMG_KEYS) red[threadIdx.x >> 6][key] = acc;
    __syncthreads();
    if (threadIdx.x < IMG_KEYS && j < V)
        scores[score_off[b] + j] = ((red[0][key] + red[1][key]) + (red[2][key] + red[3][key])) / (float)H;
}

}  // namespace d3tom

using namespace d3tom;

// Host-side argument checks shared by the entry points (everything except the workspace).
int d3tom::importance_check(const void* q, const void* k, int dt, int B, const int32_t* seq_off, int H, int dh, float scale,
                            const int32_t* dec_idx, const int32_t* dec_off, int min_D, int max_D,
                            const int32_t* vis_start, const int32_t* vis_count, const int32_t* score_off,
                            int max_N, int max_V, const float* scores) {
    if (!q || !k || !seq_off || !dec_idx || !dec_off || !vis_start || !vis_count || !score_off || !scores)
        return D3TOM_ERR_INVALID_ARG;
    if (B < 1 || H < 1 || dh < 1 || max_N < 1 || max_V < 1 || max_V > max_N || min_D < 0 || max_D < min_D)
        return D3TOM_ERR_INVALID_ARG;
    if (dt != D3TOM_F32 && dt != D3TOM_BF16) return D3TOM_ERR_INVALID_ARG;
    if (!(scale > 0.f) || !(scale < 3.0e38f)) return D3TOM_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k)) return D3TOM_ERR_INVALID_ARG;
    if (min_D == 0) return D3TOM_ERR_NO_DECIDERS;
    if (max_D > D3TOM_MAX_DECIDERS) return D3TOM_ERR_UNSUPPORTED;
    if (dh > 256 || (dt == D3TOM_BF16 ? (dh % 8) : (dh % 4))) return D3TOM_ERR_UNSUPPORTED;
    return D3TOM_OK;
}

// The scores come from kept logits if the workspace has them and the log-sum-exps of all (head, decider) pairs fit in 48 KB of LDS.
static bool imp_keeps_logits(int H, int max_D) { return max_D <= IMP_KEEP_MAXD && (long)H * max_D <= 12288; }

// The launches; arguments and workspace have been checked.
int d3tom::importance_run(const void* q, const void* k, int dt,
                          int B, const int32_t* seq_off, int H, int dh, float scale,
                          const int32_t* dec_idx, const int32_t* dec_off, int max_D,
                          const int32_t* vis_start, const int32_t* vis_count, const int32_t* score_off,
                          int max_N, int max_V, float* scores, void* ws, void* stream, ScoreSums* left) {
    if (left) *left = ScoreSums();
    const ImpWs w = imp_ws_layout(B, max_N, max_V, H, max_D);
    hipStream_t st = (hipStream_t)stream;
    char* wsb = (char*)ws;
    const float scale2 = scale * LOG2E;
    const int rows = H * max_D;
    if (dt == D3TOM_BF16 && (dh == 128 || dh == 64)) {
        float2* part = (float2*)(wsb + w.part_off);
        float* sp = (float*)(wsb + w.sp_off);
        const dim3 g1(H, w.NCH, B), g2(H, w.NCHV, B), g3(ceil_div(max_V, 256), B);
        const uint16_t* qq = (const uint16_t*)q;
        const uint16_t* kk = (const uint16_t*)k;
        // small decider sets: the first sweep keeps its logits and the scores come from them (K fetched once)
        const bool keep = imp_keeps_logits(H, max_D);
        float* logits = (float*)(wsb + w.logit_off);
        // the decider rows and each wave's statistics (or the log-sum-exps)
        const int qrows = w.DPAD < IMP_QROWS ? w.DPAD : IMP_QROWS;
        const size_t lds1 = (size_t)qrows * (dh * 2 + 16 * sizeof(float2)), lds2 = (size_t)qrows * dh * 2 + w.DPAD * sizeof(float);
#define D3TOM_IMP_STREAM(ID, GRID, DHV, SCORESV)                                                              \
    D3TOM_LAUNCH(ID, st, (imp_stream_bf16<DHV, SCORESV><<<GRID, 256, 0, st>>>(                                   \
        qq, kk, H, scale2, seq_off, dec_idx, dec_off, vis_start, vis_count, max_D, max_V, w.DPAD, w.NCH, w.KC, w.KCS, w.VPAD, part, sp)))
#define D3TOM_IMP_STATS(DHV, KEEPV, SUBV)                                                                     \
    D3TOM_LAUNCH(IMP_STATS, st, (imp_stats_bf16<DHV, KEEPV, SUBV><<<g1, 256, lds1, st>>>(                        \
        qq, kk, H, scale2, seq_off, dec_idx, dec_off, max_D, w.DPAD, w.NCH, part, w.NKB, logits)))
        const bool big = w.KC == IMP_KC_STATS;
        if (w.many) {
            if (dh == 128) { D3TOM_IMP_STREAM(IMP_STATS, g1, 128, false); D3TOM_IMP_STREAM(IMP_SCORES, g2, 128, true); }
            else           { D3TOM_IMP_STREAM(IMP_STATS, g1, 64, false);  D3TOM_IMP_STREAM(IMP_SCORES, g2, 64, true); }
        } else if (dh == 128) {
            if (keep) { if (big) D3TOM_IMP_STATS(128, true, 8); else D3TOM_IMP_STATS(128, true, 4); }
            else      { if (big) D3TOM_IMP_STATS(128, false, 8); else D3TOM_IMP_STATS(128, false, 4); }
        } else {
            if (keep) { if (big) D3TOM_IMP_STATS(64, true, 8); else D3TOM_IMP_STATS(64, true, 4); }
            else      { if (big) D3TOM_IMP_STATS(64, false, 8); else D3TOM_IMP_STATS(64, false, 4); }
        }
#undef D3TOM_IMP_STATS
#undef D3TOM_IMP_STREAM
        if (keep) {
#define D3TOM_IMP_FROM_LOGITS(ROWS)                                                                                                       \
    D3TOM_LAUNCH(IMP_SCORES, st, (imp_scores_from_logits<ROWS><<<dim3(ceil_div(max_N, 16), B), IMP_FL_THREADS, (size_t)ceil_div(rows, ROWS * IMP_FL_GROUPS) * ROWS * IMP_FL_GROUPS * sizeof(float), st>>>(   \
        H, seq_off, dec_off, vis_start, vis_count, score_off, max_D, max_V, w.DPAD, w.NCH, w.KC, w.NKB, part, logits, scores)))
            if (rows <= IMP_FL_GROUPS) D3TOM_IMP_FROM_LOGITS(1);
            else if (rows <= 4 * IMP_FL_GROUPS) D3TOM_IMP_FROM_LOGITS(4);
            else D3TOM_IMP_FROM_LOGITS(16);
#undef D3TOM_IMP_FROM_LOGITS
            return D3TOM_OK;
        }
#define D3TOM_IMP_SCORES(DHV)                                                                                 \
    D3TOM_LAUNCH(IMP_SCORES, st, (imp_scores_bf16<DHV><<<g2, 256, lds2, st>>>(                                   \
        qq, kk, H, scale2, seq_off, dec_idx, dec_off, vis_start, vis_count, max_D, max_V, w.DPAD, w.NCH, w.KC, w.VPAD, part, sp)))
        if (!w.many) { if (dh == 128) D3TOM_IMP_SCORES(128); else D3TOM_IMP_SCORES(64); }
#undef D3TOM_IMP_SCORES
        D3TOM_LAUNCH(IMP_FINISH, st, imp_finish_kernel<<<g3, 256, 0, st>>>(
            sp, H, w.VPAD, seq_off, vis_start, vis_count, score_off, max_V, scores));
        return D3TOM_OK;
    }
    float* cws = (float*)(wsb + w.c_off);
    const bool keep = max_D <= IMP_KEEP_MAXD;
    float* probs = keep ? (float*)(wsb + w.logit_off) : nullptr;
    const ScoreSums sums = {probs, rows, w.NKB * 16, H, vis_start};
    const dim3 g1(max_D, H, B), g2(ceil_div(max_V, IMG_KEYS), B);
#define D3TOM_IMP_GENERIC_OF(T, THREADS)                                                                     \
    D3TOM_LAUNCH(IMP_STATS, st, (imp_stats_generic<T, THREADS><<<g1, THREADS, 0, st>>>(                          \
        (const T*)q, (const T*)k, H, dh, scale2, seq_off, dec_idx, dec_off, max_D, sums.NK, probs, cws)))
#define D3TOM_IMP_GENERIC(T)                                                                                  \
    do { if (max_N <= 256) D3TOM_IMP_GENERIC_OF(T, 256); else if (max_N <= 512) D3TOM_IMP_GENERIC_OF(T, 512); else D3TOM_IMP_GENERIC_OF(T, 1024); } while (0)
    if (dt == D3TOM_F32) D3TOM_IMP_GENERIC(float); else D3TOM_IMP_GENERIC(uint16_t);
#undef D3TOM_IMP_GENERIC
#undef D3TOM_IMP_GENERIC_OF
    if (keep) {
        if (left && topk_takes_sums(rows, max_V)) *left = sums;
        else D3TOM_LAUNCH(IMP_SCORES, st, imp_sum_generic<<<dim3(ceil_div(max_V, 64), B), 256, 0, st>>>(sums, seq_off, vis_count, score_off, max_V, scores));
    } else if (dt == D3TOM_F32) {
        D3TOM_LAUNCH(IMP_SCORES, st, imp_scores_generic<float><<<g2, 256, 0, st>>>(
            (const float*)q, (const float*)k, H, dh, scale2, seq_off, dec_idx, dec_off, vis_start, vis_count, score_off,
            max_D, max_V, cws, scores));
    } else {
        D3TOM_LAUNCH(IMP_SCORES, st, imp_scores_generic<uint16_t><<<g2, 256, 0, st>>>(
            (const uint16_t*)q, (const uint16_t*)k, H, dh, scale2, seq_off, dec_idx, dec_off, vis_start, vis_count,
            score_off, max_D, max_V, cws, scores));
    }
    return D3TOM_OK;
}

extern "C" int d3tom_importance(const void* q, const void* k, int dt,
                                int B, const int32_t* seq_off, int H, int dh, float scale,
                                const int32_t* dec_idx, const int32_t* dec_off, int min_D, int max_D,
                                const int32_t* vis_start, const int32_t* vis_count, const int32_t* score_off,
                                int max_N, int max_V,
                                float* scores, void* ws, size_t ws_bytes, void* stream) {
    const int rc = importance_check(q, k, dt, B, seq_off, H, dh, scale, dec_idx, dec_off, min_D, max_D, vis_start,
                                    vis_count, score_off, max_N, max_V, scores);
    if (rc != D3TOM_OK) return rc;
    const ImpWs w = imp_ws_layout(B, max_N, max_V, H, max_D);
    if (!ws || ws_bytes < w.total || (((uintptr_t)ws) & 255u)) return ws ? D3TOM_ERR_WORKSPACE_TOO_SMALL : D3TOM_ERR_INVALID_ARG;
    return importance_run(q, k, dt, B, seq_off, H, dh, scale, dec_idx, dec_off, max_D, vis_start, vis_count, score_off,
                          max_N, max_V, scores, ws, stream);
}

// ---- the same call for callers that cannot allocate ---------------------------------------------
// The workspace is a file-scope device array instead of a caller buffer.  Every GPU the library runs on
// holds its own copy of the array at its own address; host code never uses the array's name as an
// address (it is a host-side stand-in) but the device address of the current GPU's copy, asked for
// once per device and kept.
static __device__ __align__(256) unsigned char scratch[D3TOM_IMPORTANCE_STATIC_BYTES];

namespace {
constexpr int MAX_GPUS = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_GPUS] = {};
}

extern "C" int d3tom_importance_static(const void* q, const void* k, int dt,
                                       int B, const int32_t* seq_off, int H, int dh, float scale,
                                       const int32_t* dec_idx, const int32_t* dec_off, int min_D, int max_D,
                                       const int32_t* vis_start, const int32_t* vis_count, const int32_t* score_off,
                                       int max_N, int max_V, float* scores, void* stream) {
    const int rc = importance_check(q, k, dt, B, seq_off, H, dh, scale, dec_idx, dec_off, min_D, max_D, vis_start,
                                    vis_count, score_off, max_N, max_V, scores);
    if (rc != D3TOM_OK) return rc;
    if (imp_ws_layout(B, max_N, max_V, H, max_D).total > (size_t)D3TOM_IMPORTANCE_STATIC_BYTES) return D3TOM_ERR_UNSUPPORTED;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_GPUS) return D3TOM_ERR_DEVICE;
    void* ptr = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_scratch_mu);
        if (!g_scratch_ptr[dev]) {
            void* p = nullptr;
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return D3TOM_ERR_DEVICE;
            g_scratch_ptr[dev] = p;
        }
        ptr = g_scratch_ptr[dev];
    }
    return importance_run(q, k, dt, B, seq_off, H, dh, scale, dec_idx, dec_off, max_D, vis_start, vis_count, score_off,
                          max_N, max_V, scores, ptr, stream);
}
