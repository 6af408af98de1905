// d3tom_update_deciders: the decider set of the next step (Section 3.2, "The Decider-Guided Mechanism":
// the tokens revealed in the preceding iteration, i.e. positions that hold a token now and held [MASK]
// one iteration earlier; Algorithm 1, the last line of the denoising loop).
//
// One workgroup per sample, or per run of samples where there are more than DEC_GROUPS.  The list is packed exactly as d3tom_importance
// reads it (dec_idx + prefix-sum offsets) without a host round trip, so a workgroup needs the counts of all samples in front of
// its own: it takes them itself, a wave per sample, 16 positions a lane in flight.  Of its own samples it tests 4096 positions at a time, four
// a thread, and compacts the flags in ascending position order (ballots, then a prefix over the 64 pieces of 64 positions).
// Bound by trips to memory: the offsets, then the own sample's first ids and the ids in front, for a wave every 16th sample, 1024 positions a trip; behind the barrier a
// trip per further 4096 positions.  Few positions are bound by the instructions of 16 waves on one unit: waves skip what lies past the end, and the list's part if they found
// nothing.  DEC_GROUPS bounds what the counting reads again: half of DEC_GROUPS times all ids.
// (One workgroup for all samples, 1024 positions at a time; own ids requested behind the count and its barrier, every wave all of a turn; now.  Calls in a graph: one sample of 64 ids 2.03,
// 2.50 and 2.2 us, of 1000 2.15, 2.7 and 2.4, of 4097 4.6, 3.6 and 3.3; two of 64 2.55, 3.3 and 2.4; 16 of 64 10.8, 4.3 and 3.1, of 500 .. 4000 32, 7.1 and 6.5; 64 of 1025 82, 12.7 and 9.2; 200 of
// 1000 157, 21.9 and 19.9.)
#include "internal.hpp"

namespace d3tom {

constexpr int DEC_THREADS = 1024, DEC_WAVES = DEC_THREADS / 64;
constexpr int DEC_PER = 4;                       // positions of a thread per turn
constexpr int DEC_COUNT = 16, DEC_FEW = 4;       // positions of a lane per turn of the count, and where no more are left
constexpr int DEC_GROUPS = 64;

__global__ __launch_bounds__(DEC_THREADS) void update_deciders_kernel(
    const int32_t* __restrict__ prev_ids, const int32_t* __restrict__ cur_ids, int mask_id, int B, int run,
    const int32_t* __restrict__ seq_off, int max_D, int32_t* __restrict__ dec_idx, int32_t* __restrict__ dec_off,
    int32_t* __restrict__ dec_count) {
#if defined(__HIP_DEVICE_COMPILE__)
    __shared__ int wtot[2][DEC_PER * DEC_WAVES]; // deciders in each 64 positions of a turn; turns alternate
    __shared__ int wsum[DEC_WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b0 = (int)blockIdx.x * run, b1 = min(b0 + run, B);
    // the `left` ids of a sample from position i0 on (beyond them: outside the buffer, not fetched), and which of 64 positions hold deciders
    auto buffer = [&](const int32_t* ids, int tok0, int i0, int left) { return make_uniform_rsrc(ids + (size_t)tok0 + i0, (uint32_t)max(left, 0) * 4u); };
    auto test = [&](int left, int at, int c, int p) { return __builtin_amdgcn_ballot_w64(at + lane < left && c != mask_id && p == mask_id); };
    // a turn of the own samples: this wave's pieces, of those past the end not even the instructions
    int c[DEC_PER], p[DEC_PER];
    auto request = [&](int tok0, int i0, int left) {
        const __amdgpu_buffer_rsrc_t cur = buffer(cur_ids, tok0, i0, left), prev = buffer(prev_ids, tok0, i0, left);
#pragma unroll
        for (int u = 0; u < DEC_PER; ++u) {
            const int at = DEC_THREADS * u + wave * 64;
            if (at >= left) break;
            c[u] = __builtin_amdgcn_raw_buffer_load_b32(cur, (at + lane) * 4, 0, 0);
            p[u] = __builtin_amdgcn_raw_buffer_load_b32(prev, (at + lane) * 4, 0, 0);
        }
    };
    // the first turn of the own sample is on its way while those in front are counted
    int tok0 = seq_off[b0], N = seq_off[b0 + 1] - tok0;
    request(tok0, 0, N);
    if (b0 > 0) {
        // entries written for the samples in front of this workgroup's
        int mine = 0;
        for (int b = wave; b < b0; b += DEC_WAVES) {
            const int t = __builtin_amdgcn_readfirstlane(seq_off[b]), n = __builtin_amdgcn_readfirstlane(seq_off[b + 1]) - t;
            int found = 0;
            auto count = [&](int i0, auto pieces) {
                constexpr int U = decltype(pieces)::value;
                const __amdgpu_buffer_rsrc_t cur = buffer(cur_ids, t, i0, n - i0), prev = buffer(prev_ids, t, i0, n - i0);
                int cc[U], pp[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    cc[u] = __builtin_amdgcn_raw_buffer_load_b32(cur, (64 * u + lane) * 4, 0, 0);
                    pp[u] = __builtin_amdgcn_raw_buffer_load_b32(prev, (64 * u + lane) * 4, 0, 0);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) found += __popcll(test(n - i0, 64 * u, cc[u], pp[u]));
            };
            for (int i0 = 0; i0 < n; i0 += 64 * DEC_COUNT) {
                if (n - i0 > 64 * DEC_FEW) count(i0, std::integral_constant<int, DEC_COUNT>());
                else count(i0, std::integral_constant<int, DEC_FEW>());
            }
            mine += min(found, max_D);
        }
        if (lane == 0) wsum[wave] = mine;
    } else if (tid == 0) {
        dec_off[0] = 0;
    }
    int base = 0, turns = 0;
    for (int b = b0; b < b1; ++b) {
        if (b > b0) {
            tok0 = seq_off[b]; N = seq_off[b + 1] - tok0;
            request(tok0, 0, N);
        }
        int found = 0;                                     // deciders of this sample seen so far (all of them)
        for (int i0 = 0;;) {                               // uniform trip count, one turn for a sample without positions
            const int left = N - i0;
            const bool more = left > DEC_PER * DEC_THREADS;
            uint64_t m[DEC_PER], any = 0;
            int* const w = wtot[turns & 1];
#pragma unroll
            for (int u = 0; u < DEC_PER; ++u) {
                const int at = DEC_THREADS * u + wave * 64;
                m[u] = at < left ? test(left, at, c[u], p[u]) : 0;
                any |= m[u];
                if (at < left && lane == 0) w[u * DEC_WAVES + wave] = __popcll(m[u]);
            }
            __syncthreads();                               // (the turn after this one writes the other half, the one after that is behind another barrier)
            if (turns++ == 0 && b0 > 0) {
#pragma unroll
                for (int v = 0; v < DEC_WAVES; ++v) base += wsum[v];
            }
            if (any || wave == 0 || more || b + 1 < b1) {  // (the others are done)
                static_assert(DEC_PER * DEC_WAVES == 64, "a piece per lane");
                const int upto = wave_incl_scan(lane * 64 < left ? w[lane] : 0);
#pragma unroll
                for (int u = 0; u < DEC_PER; ++u) {
                    if (m[u] == 0) continue;
                    const int piece = u * DEC_WAVES + wave;
                    const int ord = found + (piece ? __builtin_amdgcn_readlane(upto, piece - 1) : 0) +
                                    __builtin_amdgcn_mbcnt_hi((uint32_t)(m[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[u], 0));
                    if (((m[u] >> lane) & 1) && ord < max_D) dec_idx[base + ord] = i0 + 64 * piece + lane;     // beyond max_D: counted, not listed
                }
                found += __builtin_amdgcn_readlane(upto, 63);
            }
            if (!more) break;
            i0 += DEC_PER * DEC_THREADS;
            request(tok0, i0, N - i0);
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
