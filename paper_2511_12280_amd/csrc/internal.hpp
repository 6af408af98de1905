// Entry-point bodies shared between the C ABI functions of different source files (not part of the C ABI).
#pragma once
#include "common.hpp"
#include "direct_load.hpp"

namespace d3tom {

struct MergePrep;

// d3tom_importance after its argument and workspace checks
int importance_check(const void* q, const void* k, int dt, int B, const int32_t* seq_off, int H, int dh, float scale,
                     const int32_t* dec_idx, const int32_t* dec_off, int min_D, int max_D,
                     const int32_t* vis_start, const int32_t* vis_count, const int32_t* score_off,
                     int max_N, int max_V, const float* scores);
// Probabilities of the generic path's small decider sets in the importance workspace, [B][rows][NK]: a visual token's score is the
// sum of its column over the (head, decider) rows, divided by the heads.  In SUM_PARTS parts of consecutive rows, wherever it is formed.
struct ScoreSums {
    const float* probs = nullptr;            // none: there is nothing to sum
    int rows = 0, NK = 0, H = 0;
    const int32_t* vis_start = nullptr;
};
constexpr int SUM_PARTS = 4;
template <int R>                             // rows requested at once
__device__ __forceinline__ float score_sum_part(const ScoreSums& s, int b, int token, int part) {
    const int per = (s.rows + SUM_PARTS - 1) / SUM_PARTS, r1 = min(s.rows, (part + 1) * per);
    const float* p = s.probs + (size_t)b * s.rows * s.NK + min(token, s.NK - 1);
    float acc = 0.f;
    for (int r = part * per; r < r1; r += R) {
        float a[R];
#pragma unroll
        for (int u = 0; u < R; ++u) a[u] = p[(size_t)min(r + u, r1 - 1) * s.NK];
#pragma unroll
        for (int u = 0; u < R; ++u) acc += r + u < r1 ? a[u] : 0.f;
    }
    return acc;
}
__device__ __forceinline__ float score_of_parts(float p0, float p1, float p2, float p3, int H) { return ((p0 + p1) + (p2 + p3)) / (float)H; }
// Whether the selection of the one-call merge layer forms such scores itself, up to 32 rows of a key to a thread: a launch less, which counts
// on the host too (float32 layers of 48 .. 205 visual tokens, 4 heads, 5 .. 26 deciders 24.0 .. 25.5 us with a launch for the scores, 21.6 .. 24.7 so;
// with 375 visual tokens, in two turns, 26.1 and 27.5).
constexpr int SUM_MAX_V = 256, SUM_MAX_ROWS = 128;
inline bool topk_takes_sums(int rows, int max_V) { return rows <= SUM_MAX_ROWS && max_V <= SUM_MAX_V; }

// left, if given: sums that the selection is to form (their probabilities, or none: the scores are written)
int importance_run(const void* q, const void* k, int dt, int B, const int32_t* seq_off, int H, int dh, float scale,
                   const int32_t* dec_idx, const int32_t* dec_off, int max_D,
                   const int32_t* vis_start, const int32_t* vis_count, const int32_t* score_off,
                   int max_N, int max_V, float* scores, void* ws, void* stream, ScoreSums* left = nullptr);
size_t importance_ws_bytes(int B, int max_N, int max_V, int H, int dh, int max_D);

// Sum of squares of one row of d elements (bf16 or float32, 16-byte aligned, d a multiple of the elements per 16
// bytes), computed by one wave: lane-strided 16-byte chunks, eight loads in flight per lane, elements added in
// storage order inside a lane, lanes combined by wave_sum.  Every lane returns the total.  One definition, so that
// every launch that leaves norms for a cosine kernel leaves the same bits.  (A split contraction takes its norms from its own slices
// instead, in the one-call merge layer too: which of two near-equal cosines wins must not depend on how the merge is called.)
template <typename T>
__device__ __forceinline__ float row_sum_squares(const T* __restrict__ row, int d, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int EPC = 16 / sizeof(T);       // elements per 16-byte chunk
    float ss = 0.f;
    const int nch = d / EPC;
    const __amdgpu_buffer_rsrc_t rows = make_uniform_rsrc(row, (uint32_t)d * sizeof(T));      // past the row: reads as 0
    for (int c0 = 0; c0 < nch; c0 += 64 * 8) {
        uint4 w8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            w8[u] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rows, (uint32_t)(c0 + u * 64 + lane) * 16u, 0, 0));
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint4 w = w8[u];
            if constexpr (sizeof(T) == 2) {
                const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) { const float a = bf16_lo(ww[e]), c2 = bf16_hi(ww[e]); ss += a * a; ss += c2 * c2; }
            } else {
                const float a0 = __uint_as_float(w.x), a1 = __uint_as_float(w.y), a2 = __uint_as_float(w.z), a3 = __uint_as_float(w.w);
                ss += a0 * a0; ss += a1 * a1; ss += a2 * a2; ss += a3 * a3;
            }
        }
    }
    return wave_sum(ss);
#else
    return 0.f;
#endif
}
__device__ __forceinline__ float reciprocal_norm(float sum_squares) { return 1.0f / fmaxf(sqrtf(sum_squares), 1e-15f); }

// Table entry of a visual token: (order-preserving integer image of its best value so far) << 32 | (2^32-1 - slot).
// Unsigned comparison of entries = (value, then lower slot); 0 = nothing yet (below every real entry); a kept
// token holds the largest high word with its own slot and is never a target of an update.
typedef unsigned long long table_t;
__device__ __forceinline__ uint32_t value_key(float f) {       // ascending uint order == ascending float order
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ table_t table_entry(float value, int slot) {
    return ((table_t)value_key(value) << 32) | (table_t)(0xFFFFFFFFu - (uint32_t)slot);
}
__device__ __forceinline__ table_t table_entry_kept(int slot) {
    return ((table_t)0xFFFFFFFFu << 32) | (table_t)(0xFFFFFFFFu - (uint32_t)slot);
}

// What the merge needs before its cosine kernel, when the selection launch prepares it (the one-call merge layer):
// the selection keeps one compute unit per sample busy, so the launch carries further workgroups that stream the
// visual rows of the similarity features (one wave per row) and leave 1 / norm of EVERY visual row in rnorm, indexed
// by token; the rows are then in the memory-side cache when the cosine kernel gathers them, and the separate norms
// launch is not needed.  The selecting workgroup writes the ascending pruned list and the initial token table
// (0 for a pruned token, its own slot at the largest value for a kept one) while it emits the kept list.
struct MergePrep {
    const void* feat = nullptr;              // similarity features [sum N, d], 16-byte aligned rows
    int d = 0, dt = 0;
    const int32_t* vis_start = nullptr;
    const int32_t* vis_count = nullptr;
    float* rnorm = nullptr;                  // [B, max_V]
    int32_t* pruned = nullptr;               // [B, max_V]
    table_t* table = nullptr;                // [B, VP]
    int VP = 0;
};
// the arrays above inside a merge workspace
void merge_prep_targets(void* merge_ws, int B, int max_V, MergePrep* prep);

// Whether the preparing launch is used for a batch: only where the streaming workgroups can form their rows
// (per-sample offsets, 16-byte reads) and where it pays: rows that overflow the memory-side cache (256 MB, shared
// with everything else the step touches) would be gone again before the cosine kernel wants them, and reading every
// row then costs more than the norms of the kept rows alone.
constexpr size_t MERGE_PREP_MAX_BYTES = (size_t)160 << 20;
inline bool merge_prep_usable(const MergePrep* q, int B, int max_V, const int32_t* seq_off) {
    if (!q || !q->feat || !seq_off || !q->vis_start || !q->vis_count || !q->rnorm || !q->pruned || !q->table) return false;
    if (q->VP < max_V || (q->dt != D3TOM_BF16 && q->dt != D3TOM_F32) || q->d < 1) return false;
    const size_t row_bytes = (size_t)q->d * (q->dt == D3TOM_BF16 ? 2 : 4);
    if (row_bytes % 16 != 0 || (((uintptr_t)q->feat) & 15u) != 0) return false;
    return (size_t)B * max_V * row_bytes <= MERGE_PREP_MAX_BYTES;
}

// The streaming job of the preparing launch: 1 / norm of the visual rows of sample b, one wave per row, waves
// wave_id, wave_id + nwaves, ... (rows clamped to the sample)
__device__ __forceinline__ void stream_row_norms(const MergePrep& prep, int max_V, int b, const int32_t* __restrict__ seq_off,
                                                 int wave_id, int nwaves, int lane) {
    int tok0 = seq_off[b], tok1 = seq_off[b + 1], vs0 = prep.vis_start[b], vc = prep.vis_count[b];
    request_together(tok0, tok1, vs0, vc);
    const int n = tok1 - tok0;
    const int vs = min(max(vs0, 0), n);
    const int cnt = min(min(max(vc, 0), n - vs), max_V);
    float* rn = prep.rnorm + (size_t)b * max_V;
    for (int r = wave_id; r < cnt; r += nwaves) {
        const size_t row = (size_t)(tok0 + vs + r) * prep.d;
        const float ss = (prep.dt == D3TOM_BF16) ? row_sum_squares(static_cast<const uint16_t*>(prep.feat) + row, prep.d, lane)
                                                 : row_sum_squares(static_cast<const float*>(prep.feat) + row, prep.d, lane);
        if (lane == 0) rn[r] = reciprocal_norm(ss);
    }
}

// d3tom_select_topk; with a usable prep the launch prepares the merge and *prepared says so; with keep_ratio != nullptr the kept counts are computed on the device from the ratios and
// written, with their prefix sums and the output row offsets, to keep_k / kept_off / out_off
// sums: scores that are left to form; they are written to `scores` on the way
int topk_run(float* scores, int B, const int32_t* score_off, const int32_t* keep_k, const int32_t* kept_off, int max_V,
             int32_t* kept_idx, int32_t* slot_of, const double* keep_ratio, const int32_t* seq_off, int32_t* keep_k_out,
             int32_t* kept_off_out, int32_t* out_off_out, void* stream, const MergePrep* prep = nullptr,
             bool* prepared = nullptr, const ScoreSums& sums = ScoreSums());

// d3tom_attend without its 64-query tiles (bf16): the blocks of a stack on samples that no merge has shortened, where a merge may follow.  Which of
// two near-equal cosines takes a token goes by the last bits of these sums.  Above 512 tokens the groups of those tiles add the keys in another
// order than the wider ones do, and whether they are taken goes by the number of samples; tiles of 128, 192 and 256 queries add alike.  (Of 26 drawn
// merged stacks of 200 to 2000 visual tokens, 4 had tokens that went to another row of 1e-5 to 5e-5 less or more cosine with them.)  What still moves
// the sums of a sample of up to 512 tokens is whether the batch is for the short-sample kernel: its longest sample, and its 128-query tiles.
int attend_whole_run(const void* q, const void* k, const void* v, int B, const int32_t* cu_seqlens, int max_seqlen, int H, int dh, float scale,
                     void* o, void* stream);

// d3tom_merge / d3tom_merge_kv; prepared: the selection launch has filled the workspace as MergePrep describes;
// out_rows_hint: output rows per sample to expect when max_out is only a loose bound (a sample may have more)
int merge_run(const void* x0, void* y0, const void* x1, void* y1, const void* sim, int d, int d_sim, int dt,
              int B, const int32_t* seq_off, const int32_t* vis_start, const int32_t* vis_count,
              const int32_t* vis_off, const int32_t* kept_idx, const int32_t* kept_off,
              int max_N, int max_V, int max_keep, int max_pruned, int max_out, int mode,
              const int32_t* out_off, int32_t* assign, int32_t* counts, int32_t* src_pos,
              void* ws, size_t ws_bytes, void* stream, bool prepared = false, int out_rows_hint = 0);
size_t merge_ws_bytes(int B, int max_V);
// whether such a merge reads norms of the rows (one that cuts the contraction into slices sums the squares itself)
bool merge_takes_norms(int B, int max_V, int max_keep, int max_pruned, int d_sim, int dt);

}  // namespace d3tom
