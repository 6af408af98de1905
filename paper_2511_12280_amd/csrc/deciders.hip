// d3tom_update_deciders: the decider set of the next step (Section 3.2, "The Decider-Guided Mechanism":
// the tokens revealed in the preceding iteration, i.e. positions that hold a token now and held [MASK]
// one iteration earlier; Algorithm 1, the last line of the denoising loop).
//
// One workgroup per sample, or per run of samples where there are more than DEC_GROUPS.  The list is packed exactly as d3tom_importance
// reads it (dec_idx + prefix-sum offsets) without a host round trip, so a workgroup needs the counts of all samples in front of
// its own: it takes them itself, a wave per sample, 16 positions a lane in flight.  Of its own samples it tests 4096 positions at a time, four
// a thread, and compacts the flags in ascending position order (ballots, then a prefix over the 64 pieces of 64 positions).
// Bound by trips to memory: the offsets, then a trip per 1024 positions of the longest sample in front, the own sample's beside
// them.  DEC_GROUPS bounds what the counting reads again: half of DEC_GROUPS times all ids.
// (One workgroup for all samples, 1024 positions at a time: 16 samples of 2688 ids 34.2 us, now 6.4; 64 of 1152 82 -> 12.6; 200 of 1000
// 217 -> 24.5; 4 of 3773 12.1 -> 5.6; one of 9000 7.2 -> 4.5; one of 208 .. 3773 4.1 .. 4.3 -> 3.7.)
#include "internal.hpp"

namespace d3tom {

constexpr int DEC_THREADS = 1024, DEC_WAVES = DEC_THREADS / 64;
constexpr int DEC_PER = 4;                       // positions of a thread per turn
constexpr int DEC_COUNT = 16;                    // positions of a lane per turn of the count
constexpr int DEC_GROUPS = 64;

__global__ __launch_bounds__(DEC_THREADS) void update_deciders_kernel(
    const int32_t* __restrict__ prev_ids, const int32_t* __restrict__ cur_ids, int mask_id, int B, int run,
    const int32_t* __restrict__ seq_off, int max_D, int32_t* __restrict__ dec_idx, int32_t* __restrict__ dec_off,
    int32_t* __restrict__ dec_count) {
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ int wtot[DEC_PER * DEC_WAVES];    // deciders in each 64 positions of a turn
    __shared__ int wsum[DEC_WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = (int)blockIdx.x * run, b1 = min(b0 + run, B);
    // which of U pieces of 64 positions each hold deciders: positions i0 + 64 * (first + stride * u) + lane of the sample
    auto test = [&](int tok0, int N, int i0, int first, int stride, auto pieces, uint64_t* m) {
        constexpr int U = decltype(pieces)::value;
        const int left = min(N - i0, DEC_PER * DEC_THREADS);                    // beyond the sample: outside the buffer, not fetched
        const __amdgpu_buffer_rsrc_t cur = make_uniform_rsrc(cur_ids + (size_t)tok0 + i0, (uint32_t)left * 4u);
        const __amdgpu_buffer_rsrc_t prev = make_uniform_rsrc(prev_ids + (size_t)tok0 + i0, (uint32_t)left * 4u);
        int c[U], p[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int at = (64 * (first + stride * u) + lane) * 4;
            c[u] = __builtin_amdgcn_raw_buffer_load_b32(cur, at, 0, 0);
            p[u] = __builtin_amdgcn_raw_buffer_load_b32(prev, at, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            m[u] = __builtin_amdgcn_ballot_w64(64 * (first + stride * u) + lane < left && c[u] != mask_id && p[u] == mask_id);
    };
    // entries written for the samples in front of this workgroup's
    int mine = 0;
    for (int b = wave; b < b0; b += DEC_WAVES) {
        const int tok0 = __builtin_amdgcn_readfirstlane(seq_off[b]), N = __builtin_amdgcn_readfirstlane(seq_off[b + 1]) - tok0;
        int found = 0;
        for (int i0 = 0; i0 < N; i0 += 64 * DEC_COUNT) {
            uint64_t m[DEC_COUNT];
            test(tok0, N, i0, 0, 1, std::integral_constant<int, DEC_COUNT>{}, m);
#pragma unroll
            for (int u = 0; u < DEC_COUNT; ++u) found += __popcll(m[u]);
        }
        mine += min(found, max_D);
    }
    if (lane == 0) wsum[wave] = mine;
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int w = 0; w < DEC_WAVES; ++w) base += wsum[w];
    if (b0 == 0 && tid == 0) dec_off[0] = 0;
    for (int b = b0; b < b1; ++b) {
        const int tok0 = seq_off[b], N = seq_off[b + 1] - tok0;
        int found = 0;                                     // deciders of this sample seen so far (all of them)
        for (int i0 = 0; i0 < N; i0 += DEC_PER * DEC_THREADS) {                 // uniform trip count
            uint64_t m[DEC_PER];
            test(tok0, N, i0, wave, DEC_WAVES, std::integral_constant<int, DEC_PER>{}, m);
            __syncthreads();                               // wtot of the turn before has been read
            if (lane == 0)
#pragma unroll
                for (int u = 0; u < DEC_PER; ++u) wtot[u * DEC_WAVES + wave] = __popcll(m[u]);
            __syncthreads();
            static_assert(DEC_PER * DEC_WAVES == 64, "a piece per lane");
            const int upto = wave_incl_scan(wtot[lane]);
#pragma unroll
            for (int u = 0; u < DEC_PER; ++u) {
                const int piece = u * DEC_WAVES + wave;
                const int ord = found + (piece ? __builtin_amdgcn_readlane(upto, piece - 1) : 0) + __popcll(m[u] & ((1ull << lane) - 1ull));
                if (((m[u] >> lane) & 1) && ord < max_D) dec_idx[base + ord] = i0 + 64 * piece + lane;     // beyond max_D: counted, not listed
            }
            found += __builtin_amdgcn_readlane(upto, 63);
        }
        const int kept = min(found, max_D);
        if (tid == 0) {
            dec_off[b + 1] = base + kept;
            if (dec_count) dec_count[b] = found;
        }
        base += kept;
    }
#endif
}

}  // namespace d3tom

using namespace d3tom;

extern "C" int d3tom_update_deciders(const int32_t* prev_ids, const int32_t* cur_ids, int mask_id,
                                     int B, const int32_t* seq_off, int max_D,
                                     int32_t* dec_idx, int32_t* dec_off, int32_t* dec_count, void* stream) {
    if (!prev_ids || !cur_ids || !seq_off || !dec_idx || !dec_off) return D3TOM_ERR_INVALID_ARG;
    if (B < 1 || max_D < 1) return D3TOM_ERR_INVALID_ARG;
    if (max_D > D3TOM_MAX_DECIDERS) return D3TOM_ERR_UNSUPPORTED;
    hipStream_t st = (hipStream_t)stream;
    const int run = (B + DEC_GROUPS - 1) / DEC_GROUPS;
    D3TOM_LAUNCH(UPDATE_DECIDERS, st, update_deciders_kernel<<<(B + run - 1) / run, DEC_THREADS, 0, st>>>(
        prev_ids, cur_ids, mask_id, B, run, seq_off, max_D, dec_idx, dec_off, dec_count));
    return D3TOM_OK;
}
