// d3tom_select_topk: keep / merge partition (Section 3.2: V_kept = tokens whose score rank is at most
// the kept count; Algorithm 1, the TopK line).
//
// One 1024-thread workgroup per sample, the whole score vector in registers (at most 16 per thread) as order-preserving
// 32-bit keys.  The keys are binned linearly between their minimum and maximum (2048 bins), the bin that holds the k-th
// largest key is found by a suffix sum, and its few members (about V / 150 for scores that spread like a sum of many
// exponentials) are gathered and ranked exactly; only a bin of more than 1024 members is binned again, over its own range.
// Then one ordered compaction (ballots, one table of wave counts) emits the kept positions ascending.  Equal keys at the
// threshold are taken lowest index first, which makes the selection identical to ranking by
// (score descending, index ascending).  Integer LDS atomics only: deterministic.
// Bound by its chain of barriers on one compute unit: this takes 9 of them.  (A digit-by-digit radix selection with one
// histogram per wave and keys in LDS took about 25: 8.0 us instead of 5.7 at 729 keys, 13.1 instead of 9.9 at 16 x 2304.)  Between them
// exchanges and sums stay in the vector ALU, and the members are ranked sixteen lanes to each (729 keys 5.4 -> 4.4 us, 16 x 2304 8.6 -> 7.8).
// A kernel of a few us also pays for the code that it fetches: unrolled for 1, 4 or 16 keys a thread it is 7, 11 or 27 KB (32 KB for
// all sizes against these: 144 keys 4.8 -> 4.2 us, 729 4.6 -> 3.9, 1024 beside streamed rows 6.0 -> 5.0, 3645 8.4 -> 7.5).  And with 16 waves
// on four SIMDs every instruction that all of them execute costs 20 clocks: what the waves have to tell each other is combined by the lanes of
// a row, waves without members skip the ranking, bins are found with one comparison (144 keys 3.7 -> 3.4, 1024 4.1 -> 3.6, 3645 6.4 -> 5.3; with 4 or 8
// waves that have four or two keys a thread 1024 keys 5.4 and 4.4).
//
// The selection is a chain of short dependent passes on one compute unit per sample.  Called from the one-call
// merge layer, the launch carries further workgroups (blockIdx.y > 0) that do not select anything: one wave per
// visual row, they read the rows of the similarity features front to back and store 1 / norm of each.  That
// leaves the rows in the memory-side cache for the gathers of the cosine kernel (a sequential read of cold rows
// is several times cheaper than the 128-byte gathers that kernel would otherwise send to HBM) and replaces the
// merge's norms launch; the selecting workgroup writes the pruned list and the initial token table beside the
// kept list.
#include "internal.hpp"

namespace d3tom {

constexpr int TOPK_THREADS = 1024;
// Streaming workgroups per launch, shared out among the samples.  Merge layers of 1 to 8 samples of 144 .. 3645 rows of 512 bytes .. 8 KB, rows cold
// and cached: of one or two samples 64 lose up to 9 %, 96 up to 4 %, 160 to 256 lose or gain up to 3 %; below 400 rows a sample, 64 to 256 are the
// same.  Of 8 samples of 729 rows or more, 64 lose 3 to 15 %, 192 gain 1 to 6 %.  (Whole steps of 3645 cold rows of 8 KB, 2 and 64 deciders: 64
// of them 68.9 and 140.0 us, 96 67.3 and 137.9, 112 66.0 and 137.7, 128 65.5 and 135.7, 144 the same, 192 66.2 and 136.5.)
constexpr int TOPK_STREAM_WGS = 128;

// Kept count at a keep ratio (Section 3.2: rank at most (1 - alpha)|V|; a fractional product is rounded up):
// ceil(ratio * V - 1e-9) clamped to [1, V], in double with separately rounded product and difference, i.e.
// the same arithmetic as the host helper d3tom_keep_count.
__device__ __forceinline__ int keep_count_device(int V, double ratio) {
    double c = ceil(__dsub_rn(__dmul_rn(ratio, (double)V), 1e-9));
    if (!(c >= 1.0)) c = 1.0;
    if (c > (double)V) c = (double)V;
    return (int)c;
}

constexpr int TOPK_BINS = 2048;
[[maybe_unused]] constexpr int TOPK_CAND = 1024;                                // members of one bin that are ranked directly

// Exchanges between lanes inside the vector ALU (data-parallel moves and row swaps: some 8 clocks a step, a __shfl goes through LDS and
// takes some 100).
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ int row16_sum_i(int v) {
    v += dpp_move_i<0xB1>(v);
    v += dpp_move_i<0x4E>(v);
    v += dpp_move_i<0x141>(v);
    v += dpp_move_i<0x140>(v);
    return v;
}
__device__ __forceinline__ int wave_total(int v) { return __builtin_amdgcn_readlane(wave_incl_scan(v), 63); }
__device__ __forceinline__ uint32_t row16_min_u(uint32_t v) {
    v = min(v, (uint32_t)dpp_move_i<0xB1>((int)v));
    v = min(v, (uint32_t)dpp_move_i<0x4E>((int)v));
    v = min(v, (uint32_t)dpp_move_i<0x141>((int)v));
    v = min(v, (uint32_t)dpp_move_i<0x140>((int)v));
    return v;
}
__device__ __forceinline__ uint32_t wave_min_u(uint32_t v) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    v = row16_min_u(v);
    u2 r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = min(r[0], r[1]);
    r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return min(r[0], r[1]);
}
#endif

template <int TOPK_PER, bool SUMS>               // TOPK_PER: keys per thread at most.  SUMS: the scores are formed here
__global__ __launch_bounds__(TOPK_THREADS) void topk_select_kernel(
    float* __restrict__ scores, const int32_t* __restrict__ score_off, const int32_t* __restrict__ keep_k,
    const int32_t* __restrict__ kept_off, int max_V, int32_t* __restrict__ kept_idx, int32_t* __restrict__ slot_of,
    const double* __restrict__ keep_ratio, const int32_t* __restrict__ seq_off, int32_t* __restrict__ keep_k_out,
    int32_t* __restrict__ kept_off_out, int32_t* __restrict__ out_off_out, MergePrep prep, ScoreSums sums) {
#if defined(__HIP_DEVICE_COMPILE__)
    if (blockIdx.y > 0) {
        // streaming workgroups: norms of the sample's visual rows
        stream_row_norms(prep, max_V, blockIdx.x, seq_off, (int)(blockIdx.y - 1) * (TOPK_THREADS / 64) + (int)(threadIdx.x >> 6),
                         (int)(gridDim.y - 1) * (TOPK_THREADS / 64), threadIdx.x & 63);
        return;
    }
    __shared__ int hist[TOPK_BINS];
    __shared__ uint2 cand[TOPK_CAND];             // (key, index) of the members of the threshold's bin
    __shared__ int wsum[16];
    __shared__ uint32_t wrange[32];
    __shared__ int wcnt[TOPK_PER * 16];           // per 64 consecutive keys: how many are kept (equal to the threshold)
    __shared__ int sel[4];                        // bin of the k-th largest key, its rank inside the bin, members of the bin
    __shared__ uint32_t thr_s[2];                 // threshold key, highest index kept among the keys equal to it
    __shared__ int plan[2];                       // kept count of this sample, first slot of this sample in kept_idx
    const int b = blockIdx.x;
    int s0 = score_off[b], s1 = score_off[b + 1];
    const int V = min(s1 - s0, max_V);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;

    // thread t holds keys t, t + 1024, ...
    uint32_t key[TOPK_PER];
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
    static_assert(!SUMS || TOPK_PER == 1, "");
    __shared__ float part[SUMS ? SUM_PARTS : 1][SUMS ? SUM_MAX_V : 1];
    if constexpr (SUMS) {
        const int vs = max(sums.vis_start[b], 0);
        for (int j = tid & 255; j < V; j += 256) part[wave >> 2][j] = score_sum_part<16>(sums, b, vs + j, wave >> 2);
    } else {
        const __amdgpu_buffer_rsrc_t mine = make_uniform_rsrc(scores + s0, (uint32_t)max(V, 0) * 4u);       // beyond the sample: 0, not fetched
#pragma unroll
        for (int c = 0; c < TOPK_PER && c < 4; ++c) key[c] = __builtin_amdgcn_raw_buffer_load_b32(mine, (c * TOPK_THREADS + tid) * 4, 0, 0);
        if (V > 4 * TOPK_THREADS) {                   // requests beyond the sample take their turn in the load path too
#pragma unroll
            for (int c = 4; c < TOPK_PER; ++c) key[c] = __builtin_amdgcn_raw_buffer_load_b32(mine, (c * TOPK_THREADS + tid) * 4, 0, 0);
        }
    }
    if (keep_ratio && wave == 15) {
        // kept counts from the ratios, on the device: this sample's count, and the prefix sums over the samples
        // in front of it (every workgroup repeats that, a sample per lane; the last one also writes the totals)
        const int kb = V > 0 ? keep_count_device(V, keep_ratio[b]) : 0;
        const int nb = (seq_off[b + 1] - seq_off[b]) - (V - kb);
        int koff = 0, ooff = 0;
        for (int b0 = 0; b0 < b; b0 += 64) {
            const int bb = b0 + lane;
            int kcur = 0, ncur = 0;
            if (bb < b) {
                const int Vb = min(score_off[bb + 1] - score_off[bb], max_V);
                kcur = Vb > 0 ? keep_count_device(Vb, keep_ratio[bb]) : 0;
                ncur = (seq_off[bb + 1] - seq_off[bb]) - (Vb - kcur);
            }
            koff += wave_total(kcur);
            ooff += wave_total(ncur);
        }
        if (lane == 0) {
            plan[0] = kb; plan[1] = koff;
            keep_k_out[b] = kb; kept_off_out[b] = koff; out_off_out[b] = ooff;
            if (b == (int)gridDim.x - 1) { kept_off_out[b + 1] = koff + kb; out_off_out[b + 1] = ooff + nb; }
        }
    }
    for (int t = tid; t < TOPK_BINS; t += TOPK_THREADS) hist[t] = 0;
    if (tid == 0) sel[3] = 0;
    if constexpr (SUMS) {
        __syncthreads();
        if (tid < V) {
            const float v = score_of_parts(part[0][tid], part[1][tid], part[2][tid], part[3][tid], sums.H);
            scores[s0 + tid] = v;
            key[0] = __float_as_uint(v);
        }
    }
#pragma unroll
    for (int c = 0; c < TOPK_PER; ++c) {
        if (c * TOPK_THREADS >= V) break;
        if (c * TOPK_THREADS + tid < V) {
            key[c] = value_key(__uint_as_float(key[c]));
            kmin = min(kmin, key[c]); kmax = max(kmax, key[c]);
        }
    }
    kmin = wave_min_u(kmin);
    kmax = ~wave_min_u(~kmax);
    if (lane == 0) { wrange[wave] = kmin; wrange[16 + wave] = kmax; }
    __syncthreads();
    if (V <= 0) return;
    kmin = row16_min_u(wrange[lane & 15]);        // (16 waves' values by the lanes of a row: a loop over them is 32 instructions in every wave)
    kmax = ~row16_min_u(~wrange[16 + (lane & 15)]);
    int remaining = keep_ratio ? plan[0] : min(max(keep_k[b], 1), V);      // rank of the threshold among the keys in [lo, hi]
    const int k0 = keep_ratio ? plan[1] : kept_off[b], kept_count = remaining;

    uint32_t lo = kmin, hi = kmax;
    int members = V;
    uint32_t range;
    for (;;) {                                    // one turn, unless a bin holds more than TOPK_CAND members
        range = hi - lo;
        const int shift = (range < TOPK_BINS) ? 0 : 21 - __clz(range);        // range >> shift < 2048
#pragma unroll
        for (int c = 0; c < TOPK_PER; ++c) {
            if (c * TOPK_THREADS >= V) break;
            const uint32_t above = key[c] - lo;                               // beyond the range if it is below lo, too
            if (c * TOPK_THREADS + tid < V && above <= range) {
                // a whole wave in one bin would serialise on one LDS address: add it once instead
                const int bin = (int)(above >> shift);
                const uint64_t here = __builtin_amdgcn_ballot_w64(true);
                if (__builtin_amdgcn_ballot_w64(bin == __builtin_amdgcn_readfirstlane(bin)) == here) {
                    if (lane == __builtin_ctzll(here)) atomicAdd(&hist[bin], __popcll(here));
                } else atomicAdd(&hist[bin], 1);
            }
        }
        __syncthreads();
        // thread t owns bins 2047 - 2t and 2046 - 2t: keys above its bins = the bins of the threads before it
        const int h0 = hist[TOPK_BINS - 1 - 2 * tid], h1 = hist[TOPK_BINS - 2 - 2 * tid];
        const int inc = wave_incl_scan(h0 + h1);
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        const int before = inc - h0 - h1 + row16_sum_i((lane & 15) < wave ? wsum[lane & 15] : 0);
        if (before < remaining && remaining <= before + h0) {
            sel[0] = TOPK_BINS - 1 - 2 * tid; sel[1] = remaining - before; sel[2] = h0;
        } else if (before + h0 < remaining && remaining <= before + h0 + h1) {
            sel[0] = TOPK_BINS - 2 - 2 * tid; sel[1] = remaining - before - h0; sel[2] = h1;
        }
        __syncthreads();
        lo += (uint32_t)sel[0] << shift;
        hi = min(hi, lo + (uint32_t)((1u << shift) - 1u));
        range = hi - lo;
        remaining = sel[1];
        members = sel[2];
        if (TOPK_PER == 1 || members <= TOPK_CAND || shift == 0) break;       // (at most 1024 keys)
        for (int t = tid; t < TOPK_BINS; t += TOPK_THREADS) hist[t] = 0;
        __syncthreads();
    }
    if (TOPK_PER == 1 || members <= TOPK_CAND) {
        // gather the members (any order) and rank each: the one with remaining - 1 members in front of it is the threshold
#pragma unroll
        for (int c = 0; c < TOPK_PER; ++c) {
            if (c * TOPK_THREADS >= V) break;
            const int j = c * TOPK_THREADS + tid;
            if (j < V && key[c] - lo <= range) cand[atomicAdd(&sel[3], 1)] = make_uint2(key[c], (uint32_t)j);
        }
        __syncthreads();
        if (members <= TOPK_THREADS / 16) {
            // sixteen lanes to a member (one to a member: a chain of that many trips to LDS); a wave has four members, most waves none
            if (wave * 4 < members) {
                const int c = tid >> 4;
                const uint2 me = cand[min(c, members - 1)];
                int rank = 0;
                for (int t0 = 0; t0 < members; t0 += 16) {
                    const int t = t0 + (tid & 15);
                    const uint2 o = cand[min(t, members - 1)];
                    rank += (t < members) && ((o.x > me.x) || (o.x == me.x && o.y < me.y));
                }
                if (row16_sum_i(rank) == remaining - 1 && c < members) { thr_s[0] = me.x; thr_s[1] = me.y; }
            }
        } else if (tid < members) {
            const uint2 me = cand[tid];
            int rank = 0;
#pragma unroll 8
            for (int t = 0; t < members; ++t) {
                const uint2 o = cand[t];
                rank += (o.x > me.x) || (o.x == me.x && o.y < me.y);
            }
            if (rank == remaining - 1) { thr_s[0] = me.x; thr_s[1] = me.y; }
        }
    } else {
        // more than TOPK_CAND keys are equal to the threshold (lo == hi): find the remaining-th of them by position
#pragma unroll
        for (int c = 0; c < TOPK_PER; ++c) {
            if (c * TOPK_THREADS >= V) break;
            const bool eq = (c * TOPK_THREADS + tid < V) && key[c] == lo;
            const unsigned long long m = __builtin_amdgcn_ballot_w64(eq);
            if (lane == 0) wcnt[c * 16 + wave] = __popcll(m);
        }
        __syncthreads();
        int run = 0;
#pragma unroll
        for (int c = 0; c < TOPK_PER; ++c) {
            if (c * TOPK_THREADS >= V) break;
            int bef = run;
            for (int w = 0; w < 16; ++w) { bef += (w < wave) ? wcnt[c * 16 + w] : 0; run += wcnt[c * 16 + w]; }
            const bool eq = (c * TOPK_THREADS + tid < V) && key[c] == lo;
            const unsigned long long m = __builtin_amdgcn_ballot_w64(eq);
            if (eq && bef + __popcll(m & ((1ull << lane) - 1ull)) == remaining - 1) {
                thr_s[0] = lo; thr_s[1] = (uint32_t)(c * TOPK_THREADS + tid);
            }
        }
    }
    __syncthreads();
    const uint32_t thr = thr_s[0];
    const int thr_idx = (int)thr_s[1];
    auto kept = [&](int c) {
        const int j = c * TOPK_THREADS + tid;
        return j < V && (key[c] > thr || (key[c] == thr && j <= thr_idx));
    };
#pragma unroll
    for (int c = 0; c < TOPK_PER; ++c) {
        if (c * TOPK_THREADS >= V) break;
        const unsigned long long m = __builtin_amdgcn_ballot_w64(kept(c));
        if (lane == 0) wcnt[c * 16 + wave] = __popcll(m);
    }
    __syncthreads();
    // Where a thread has several keys the stores go through buffers, those that a key does not take part in and those of keys beyond the sample
    // to nowhere: fewer instructions a key, which are what several keys cost (3645 keys 6.2 -> 5.8 us; with one key a thread 4.0 -> 4.2).
    constexpr bool BUFFERS = TOPK_PER > 1;
    constexpr uint32_t NOWHERE = 0x80000000u;
    __amdgpu_buffer_rsrc_t slots, list, entries, others;
    if constexpr (BUFFERS) {
        slots = make_uniform_rsrc(slot_of + s0, (uint32_t)V * 4u);
        list = make_uniform_rsrc(kept_idx + k0, (uint32_t)kept_count * 4u);
        entries = make_uniform_rsrc(prep.table + (size_t)b * prep.VP, prep.table ? (uint32_t)V * 8u : 0u);
        others = make_uniform_rsrc(prep.pruned + (size_t)b * max_V, prep.table ? (uint32_t)V * 4u : 0u);
    }
    // kept keys in front of each run of 64: four chunks (64 runs, one per lane) at a time
    int base = 0;
#pragma unroll
    for (int c4 = 0; c4 < TOPK_PER; c4 += 4) {
        if (c4 * TOPK_THREADS >= V) break;
        const int mine = ((c4 * 16 + lane) * 64 < V) ? wcnt[c4 * 16 + lane] : 0;
        const int inc = wave_incl_scan(mine);
        const int exc = inc - mine;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c4 + u;
            if (c >= TOPK_PER || c * TOPK_THREADS >= V) break;
            const int j = c * TOPK_THREADS + tid;
            const bool keep = kept(c);
            const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
            const int slot = base + __builtin_amdgcn_readlane(exc, u * 16 + wave) + __popcll(m & ((1ull << lane) - 1ull));
            // slot = kept tokens in front of j: a pruned token sits at position j - slot of the ascending pruned list
            if constexpr (BUFFERS) {
                __builtin_amdgcn_raw_buffer_store_b32((uint32_t)(keep ? slot : -1), slots, j * 4, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b32((uint32_t)j, list, keep ? (uint32_t)slot * 4u : NOWHERE, 0, 0);
                if (prep.table) {
                    typedef unsigned u2 __attribute__((ext_vector_type(2)));
                    const u2 entry = {keep ? 0xFFFFFFFFu - (uint32_t)slot : 0u, keep ? 0xFFFFFFFFu : 0u};    // table_entry_kept(slot) or nothing yet
                    __builtin_amdgcn_raw_buffer_store_b64(entry, entries, j * 8, 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b32((uint32_t)j, others, keep || j >= V ? NOWHERE : (uint32_t)(j - slot) * 4u, 0, 0);
                }
            } else if (j < V) {
                slot_of[s0 + j] = keep ? slot : -1;
                if (prep.table) {
                    prep.table[(size_t)b * prep.VP + j] = keep ? table_entry_kept(slot) : (table_t)0;
                    if (!keep) prep.pruned[(size_t)b * max_V + (j - slot)] = j;
                }
                if (keep) kept_idx[k0 + slot] = j;
            }
        }
        base += __builtin_amdgcn_readlane(inc, 63);
    }
#endif
}

}  // namespace d3tom

using namespace d3tom;

int d3tom::topk_run(float* scores, int B, const int32_t* score_off, const int32_t* keep_k, const int32_t* kept_off,
                    int max_V, int32_t* kept_idx, int32_t* slot_of, const double* keep_ratio, const int32_t* seq_off,
                    int32_t* keep_k_out, int32_t* kept_off_out, int32_t* out_off_out, void* stream, const MergePrep* prep_in,
                    bool* prepared, const ScoreSums& sums) {
    if (prepared) *prepared = false;
    if (!scores || !score_off || !kept_idx || !slot_of) return D3TOM_ERR_INVALID_ARG;
    if (keep_ratio ? (!seq_off || !keep_k_out || !kept_off_out || !out_off_out) : (!keep_k || !kept_off)) return D3TOM_ERR_INVALID_ARG;
    if (B < 1 || max_V < 1) return D3TOM_ERR_INVALID_ARG;
    if (max_V > D3TOM_MAX_VISUAL) return D3TOM_ERR_UNSUPPORTED;
    hipStream_t st = (hipStream_t)stream;
    const bool streaming = merge_prep_usable(prep_in, B, max_V, seq_off);
    const MergePrep prep = streaming ? *prep_in : MergePrep();
    const int extra = streaming ? (B >= TOPK_STREAM_WGS ? 1 : TOPK_STREAM_WGS / B) : 0;
#define D3TOM_SELECT(PER, SUMS)                                                                                 \
    D3TOM_LAUNCH(TOPK_SELECT, st, (topk_select_kernel<PER, SUMS><<<dim3(B, 1 + extra), TOPK_THREADS, 0, st>>>(           \
        scores, score_off, keep_k, kept_off, max_V, kept_idx, slot_of, keep_ratio, seq_off, keep_k_out, kept_off_out, out_off_out, prep, sums)))
    if (sums.probs) D3TOM_SELECT(1, true);
    else if (max_V <= TOPK_THREADS) D3TOM_SELECT(1, false);
    else if (max_V <= 4 * TOPK_THREADS) D3TOM_SELECT(4, false);
    else D3TOM_SELECT(D3TOM_MAX_VISUAL / TOPK_THREADS, false);
#undef D3TOM_SELECT
    if (prepared) *prepared = streaming;
    return D3TOM_OK;
}

extern "C" int d3tom_select_topk(const float* scores, int B, const int32_t* score_off, const int32_t* keep_k,
                                 const int32_t* kept_off, int max_V,
                                 int32_t* kept_idx, int32_t* slot_of,
                                 void* ws, size_t ws_bytes, void* stream) {
    (void)ws; (void)ws_bytes;
    return topk_run(const_cast<float*>(scores), B, score_off, keep_k, kept_off, max_V, kept_idx, slot_of, nullptr, nullptr, nullptr, nullptr,
                    nullptr, stream);
}
