// d3tom_merge: similarity-based merging (Section 3.2, "Similarity-Based Merging"; Algorithm 1, the
// FORALL block and the "Remove positions" line).
//
// Stages, all on the caller's stream:
//   norms     1 / ||row|| of every KEPT row of the similarity features (1 wave / row; a split contraction sums the
//             squares itself and needs no such launch): the argmax over
//             kept slots of dot / (|m| |k|) does not depend on |m|, the pruned row's own norm; the same
//             waves write the ascending list of pruned visual tokens (the gaps of the ascending kept_idx)
//             and initialise the token -> (best value, slot) table
//   cosine    pruned x kept similarity GEMM on MFMA 16x16x32 bf16 with the argmax fused into the
//             epilogue: only (best value, best slot) per (pruned row, 128-slot column tile) ever
//             leaves the registers, as ONE 64-bit integer atomic max on the row's table entry (value in
//             the high word as an order-preserving integer, 2^32-1-slot in the low word: the maximum is
//             the best cosine, the lowest slot among equals, whatever order the tiles arrive in, so the
//             result is bit-reproducible); the M x k matrix is never written
//   scatter   one workgroup per OUTPUT row: a merged row scans the table for its members (ascending
//             token order), streams them with 16-byte loads and accumulates in float32 in that order,
//             other rows are copied; one store per element, no float atomics
//
// All similarities are taken on the rows as given (assignment first, aggregation afterwards).
#include <type_traits>
#include "internal.hpp"
#include "direct_load.hpp"

namespace d3tom {

constexpr int COS_BN = 128;        // kept slots per column tile (96 where that fills the chip better)
constexpr int COS_BK = 64;         // contraction elements per LDS stage

// split-K partial products: at most COS_SPLIT_BLOCKS (tile, k-slice) blocks of 64 x 128 floats
constexpr int COS_SPLIT_BLOCKS = 256;
constexpr int COS_MAX_SLICES = 16;
struct MergeWs {
    size_t pruned_off, rnorm_off, table_off, dots_off, sq_off, total;
    int VP;                    // table entries per sample
};
__host__ inline MergeWs merge_ws_layout(int B, int max_V) {
    MergeWs w;
    w.VP = (int)align_up((size_t)max_V, 4);
    size_t o = 0;
    w.pruned_off = o; o += align_up((size_t)B * max_V * 4, 256);
    w.rnorm_off = o;  o += align_up((size_t)B * max_V * 4, 256);
    w.table_off = o;  o += align_up((size_t)B * w.VP * 8, 256);     // token -> (best value, slot) table
    w.dots_off = o;   o += (size_t)COS_SPLIT_BLOCKS * 64 * 128 * sizeof(float);
    w.sq_off = o;     o += (size_t)COS_SPLIT_BLOCKS * 128 * sizeof(float);           // sums of squares per (k-slice, kept slot)
    w.total = o;
    return w;
}
size_t merge_ws_bytes(int B, int max_V) { return merge_ws_layout(B, max_V).total; }
void merge_prep_targets(void* merge_ws, int B, int max_V, MergePrep* prep) {
    const MergeWs w = merge_ws_layout(B, max_V);
    char* wsb = (char*)merge_ws;
    prep->pruned = (int32_t*)(wsb + w.pruned_off);
    prep->rnorm = (float*)(wsb + w.rnorm_off);
    prep->table = (table_t*)(wsb + w.table_off);
    prep->VP = w.VP;
}

struct SampleGeom { int tok0, N, vs, V, k, M, k0; };
__device__ __forceinline__ SampleGeom geom_of(int t0, int t1, int vs, int vc, int k0, int k1, int max_V, int max_keep) {
    SampleGeom s;
    s.tok0 = t0;
    s.N = t1 - t0;
    s.vs = min(max(vs, 0), s.N);
    s.V = min(min(vc, max_V), s.N - s.vs);
    s.k0 = k0;
    s.k = min(min(k1 - k0, max_keep), s.V);
    s.M = s.V - s.k;
    return s;
}
// more0, more1: further offsets to be read with the sample's
__device__ __forceinline__ SampleGeom sample_geom(int b, const int32_t* seq_off, const int32_t* vis_start, const int32_t* vis_count,
                                                  const int32_t* kept_off, int max_V, int max_keep, int& more0, int& more1) {
    int t0 = seq_off[b], t1 = seq_off[b + 1], vs = vis_start[b], vc = vis_count[b], k0 = kept_off[b], k1 = kept_off[b + 1];
    request_together(t0, t1, vs, vc, k0, k1, more0, more1);
    return geom_of(t0, t1, vs, vc, k0, k1, max_V, max_keep);
}
__device__ __forceinline__ SampleGeom sample_geom(int b, const int32_t* seq_off, const int32_t* vis_start,
                                                  const int32_t* vis_count, const int32_t* kept_off, int max_V, int max_keep) {
    int none0 = 0, none1 = 0;
    return sample_geom(b, seq_off, vis_start, vis_count, kept_off, max_V, max_keep, none0, none1);
}

// ---- norms + pruned list + table init --------------------------------------------------------------
// One wave per kept slot r computes 1 / ||row|| of that slot's token.  The same wave also writes the
// piece of the ascending pruned list that lies in front of its token: kept_idx is ascending, so the
// pruned tokens j between kept_idx[r-1] and kept_idx[r] have exactly r kept tokens before them and sit
// at positions j - r of the list (the wave of the last slot also writes the piece behind its token).
// No scan, no extra workgroup.  The table entries of the same tokens are set on the way: "nothing yet"
// for the pruned ones, its own slot for the kept one.
template <typename T>
__global__ __launch_bounds__(256) void merge_norms_kernel(
    const T* __restrict__ f, int d, const int32_t* __restrict__ seq_off, const int32_t* __restrict__ vis_start,
    const int32_t* __restrict__ vis_count, const int32_t* __restrict__ kept_idx, const int32_t* __restrict__ kept_off,
    int max_V, int max_keep, float* __restrict__ rnorm, int32_t* __restrict__ pruned, table_t* __restrict__ table, int VP) {
    const int b = blockIdx.y;
    const SampleGeom s = sample_geom(b, seq_off, vis_start, vis_count, kept_off, max_V, max_keep);
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6);      // kept slot
    const int lane = threadIdx.x & 63;
    if (r >= s.k) return;
    const int32_t* kp = kept_idx + s.k0;
    const int j = min(max(kp[r], 0), s.V - 1);
    {
        int32_t* pr = pruned + (size_t)b * max_V;
        table_t* tab = table + (size_t)b * VP;
        const int lo = (r == 0) ? -1 : min(max(kp[r - 1], 0), s.V - 1);
        // positions are >= 0 whenever kept_idx is ascending and free of repeats; the guard only keeps an
        // invalid list from writing in front of the array
        for (int t = lo + 1 + lane; t < j; t += 64) { tab[t] = 0; if (t >= r) pr[t - r] = t; }
        if (r == s.k - 1)
            for (int t = j + 1 + lane; t < s.V; t += 64) { tab[t] = 0; if (t >= s.k) pr[t - s.k] = t; }
        if (lane == 0) tab[j] = table_entry_kept(r);
    }
    const float ss = row_sum_squares(f + (size_t)(s.tok0 + s.vs + j) * d, d, lane);
    if (lane == 0) rnorm[(size_t)b * max_V + r] = reciprocal_norm(ss);
}

// ---- cosine GEMM + fused argmax, bf16 MFMA ---------------------------------------------------
// Workgroup tile: (TM*64) pruned rows x 128 kept slots; waves 0..3 compute (2 x 2, wave tile (TM*32) x 64),
// waves 4..7 only issue the loads.
//
// Operand tiles go HBM/L2 -> LDS with direct loads (buffer_load ... lds, 16 bytes per lane, no register
// staging) into a ring of COS_NS stages of 64 contraction elements; the loads of stage kt+3 are in
// flight while stage kt feeds the MFMAs, one s_barrier per stage.  A wave-load writes 1 KB of LDS
// contiguously (8 rows x 128 B), so rows cannot be padded; instead the 16-byte chunk that lands in
// position p of row r is chunk p ^ ((r >> 1) & 7) of that row (the lane picks its global address
// accordingly), which spreads the MFMA operand reads of 16 consecutive rows over all 64 banks.
//
// Workgroup ids are mapped to tiles per XCD: ids are dealt round-robin to the 8 XCDs by the hardware.  The
// tiles of a sample are numbered band by band (RB row tiles high, column-major inside a band) and that
// sequence is cut into 8 runs of equal length, one per XCD: every XCD gets the same number of tiles
// (a rectangle per XCD leaves some XCDs with more tiles than they have CUs while others idle), and a
// run covers a compact block of about RB x (run / RB) tiles, so its private L2 sees few operand rows.
// The loads are buffer loads: each lane's byte offset (row and swizzled chunk) is fixed for the whole
// sweep and the k-slice moves through the scalar offset, so a stage costs no address arithmetic.
//
// What bounds it is what one CU takes in: 55 .. 60 bytes per clock when another CU of the XCD has had the rows, 27 when none
// has; 32 KB a stage at 44 are 745 clocks, the MFMAs of a 128-row tile 512.  The computing waves therefore only have to keep
// out of the way: fragments one k-step ahead across the stage's barrier, the smaller MFMA shape (less power: 1.6 GHz
// against 1.5), the kept rows' norms read once in the epilogue (read for every row, 400 clocks each, it took 5 us of 35).
// Workgroups behind the last sample's tiles, if the launch has any, are helpers: they pull rows from HBM for the others.
// Measured at d = 4096: 1822 x 1823 rows 37.9 -> 31.8 us, 2733 x 912 32.4 -> 28.5, 16 samples of 2304 rows 195 -> 167.
constexpr int cos_ring_stages(int TM) { return TM >= 4 ? 3 : 4; }     // 256-row tiles: 3 stages of 48 KB fit the 160 KB of LDS

// Helpers (see the launch): the first lines of a helper's rows answer within this time, in ticks of 10 ns, where the rows lie in the
// memory-side cache, and later where they lie in HBM.  (0.45 and 0.55 us tell the two apart at all sizes measured; from 0.65 us
// on, rows in HBM are taken for cached ones more and more often.)
constexpr uint32_t COS_CACHED_TICKS = 55;

// row tiles of a band, for a sample with per_b tiles on each XCD in a launch sized for `per`
__device__ __forceinline__ int band_height(int RB, int per_b, int per, int nrt_b) {
    int rb = RB;
    if (per_b < per) { rb = 1; while ((rb + 1) * (rb + 1) <= per_b) ++rb; }
    return min(rb, nrt_b);
}

// SPLIT (contraction cut into ksplit > 1 slices): the workgroups of row tile 0 sum the squares of their kept rows (the diagonal of
// B B^T, two MFMAs per block of 16 rows and stage where the load path leaves the matrix core idle), and without a preparing launch
// the kernel derives the pruned tokens from the kept list itself and writes the pruned list and the kept tokens' table entries
// for the kernels behind it: no norms launch (4 of the 21 us that a merge of 356 tokens takes).  The norms are summed here whether
// or not the selection launch has left others: near-ties of two cosines go by their last bits, and the one call and the
// separate calls agree on them where their bounds on the kept and pruned counts give the same number of slices (tight bounds do).
template <int TM, int CBK, bool SPLIT>     // CBK: 16-column blocks of a wave
__global__ __launch_bounds__(512) void cos_argmax_bf16(
    const uint16_t* __restrict__ f, int d, const int32_t* __restrict__ seq_off, const int32_t* __restrict__ vis_start,
    const int32_t* __restrict__ vis_count, const int32_t* __restrict__ kept_idx, const int32_t* __restrict__ kept_off,
    int max_V, int max_keep, int32_t* __restrict__ pruned, const float* __restrict__ rnorm,
    table_t* __restrict__ table, int VP, int per, int RB, int ksplit, float* __restrict__ dots, int nrt_launch, int nct_launch, int prepared,
    int nB, float* __restrict__ sq) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BM = TM * 64, BN = CBK * 32;
    constexpr int COS_NS = cos_ring_stages(TM);
    constexpr int STAGE = (BM + BN) * 128;          // bytes per ring stage (64 bf16 = 128 B per row)
    constexpr int A_LD = BM / 32;                       // direct loads per wave and stage, A tile (8 rows each)
    constexpr int B_LD = BN / 32;
    extern __shared__ __attribute__((aligned(16))) char ring[];
    __shared__ float rnB[BN];

    // blockIdx.x & 7 is the XCD the hardware puts the workgroup on.  The launch is sized for the largest sample (per = one XCD's share
    // of its tiles); every sample numbers ITS OWN tiles and cuts that sequence into 8 equal runs, so that a sample with fewer tiles
    // still loads its XCDs alike (numbered on the launch's grid, the tiles of a short sample would all fall to the first XCDs).
    // Where the runs do not come out even the first XCDs have the longer ones, so sample b begins at another XCD than b - 1 does (64
    // samples of 100 .. 144 rows: 91 -> 68 us, 16 of 200 .. 300 42 -> 36).
    //
    // TM 4, for launches of several rounds: the tiles of all samples, one behind the other, are cut into 8 equal runs, one per XCD,
    // so that the XCDs end together whatever the sizes of the samples (which the host does not know), and a sample's rows
    // are read by two or three XCDs.  An XCD's run is rounds of 32 tiles, one a CU, and a rest, which would be a round as long as
    // the others: rests of up to 16 or 8 tiles are cut into half or quarter row tiles (of 0.67 and 0.5 of the time).  Merges at d = 4096 against
    // runs of a sample's tiles on two XCDs and no cuts: 16 samples of 1152 .. 2304 rows keeping 0.1 .. 0.5 of them 181 -> 163 us,
    // 12 135 -> 118, 24 274 -> 257, 16 of 2304 251 -> 247, 13 of 2304 keeping a quarter 210 -> 173.
    const int wx = blockIdx.x >> 3;
    int b = wx / per, id = wx % per, xcd = blockIdx.x & 7;
    if (TM < 4) xcd = (xcd + (b < nB ? b : (wx - per * nB) % nB)) & 7;     // (helpers: as the sample that they help)
    int cut = 0, part = 0;                                 // TM 4: this is part `part` of a row tile cut into 1 << cut
    if constexpr (TM == 4) {
        const int lane = threadIdx.x & 63;
        auto tiles_upto = [&](int b0) {                    // of samples b0 .. b0 + lane
            int n = 0;
            if (b0 + lane < nB) {
                const int i = b0 + lane;
                const SampleGeom g = geom_of(seq_off[i], seq_off[i + 1], vis_start[i], vis_count[i], kept_off[i], kept_off[i + 1], max_V, max_keep);
                n = min((g.M + BM - 1) / BM, nrt_launch) * min((g.k + BN - 1) / BN, nct_launch);
            }
            return wave_incl_scan(n);
        };
        const int first = tiles_upto(0);
        int all = __builtin_amdgcn_readlane(first, 63);
        for (int b0 = 64; b0 < nB; b0 += 64) all += __builtin_amdgcn_readlane(tiles_upto(b0), 63);
        const int lo = (int)((long)all * xcd / 8), n = (int)((long)all * (xcd + 1) / 8) - lo;      // this XCD's run
        const int odd = n & 31, whole = n - odd;
        int t = wx;
        if (t >= whole) {
            cut = odd <= 8 ? 2 : odd <= 16 ? 1 : 0;
            t = whole + ((wx - whole) >> cut);
            part = (wx - whole) & ((1 << cut) - 1);
        }
        if (t >= n) return;
        t += lo;
        int before = 0;
        b = nB;
        for (int b0 = 0; b0 < nB; b0 += 64) {              // t < all: some sample has it
            const int upto = b0 ? before + tiles_upto(b0) : first;
            const uint64_t behind = __builtin_amdgcn_ballot_w64(upto > t);
            if (behind) {
                const int j = __builtin_ctzll(behind);
                b = b0 + j;
                id = t - (j ? __builtin_amdgcn_readlane(upto, j - 1) : before);
                break;
            }
            before = __builtin_amdgcn_readlane(upto, 63);
        }
    }
    if (b >= nB) {
        if constexpr (!SPLIT && TM < 4) {
            // A helper: requests a dword of every 128-byte line of pruned rows that tiles of this XCD use, four lines of each
            // row at a time, so that the rows come from HBM into the XCD's L2 ahead of the tiles that walk through them.  Of the
            // XCDs that use a row tile, the one with its tile in column `pick` has it.
            const int hx = (int)(blockIdx.x >> 3) - per * nB, nx = (int)(gridDim.x >> 3) - per * nB;   // helper hx of the XCD's nx
            const int hb = hx % nB, h0 = hx / nB, hn = (nx - hb + nB - 1) / nB;                        // the h0-th of sample hb's hn
            const SampleGeom s = sample_geom(hb, seq_off, vis_start, vis_count, kept_off, max_V, max_keep);
            const int nrt_b = min((s.M + BM - 1) / BM, nrt_launch), nct_b = min((s.k + BN - 1) / BN, nct_launch);
            const int per_b = (nrt_b * nct_b + 7) / 8;
            const int tid = threadIdx.x, wave = tid >> 6;
            uint64_t* owned = reinterpret_cast<uint64_t*>(ring);                 // bit per row tile (one round: at most 256)
            const int rb = band_height(RB, per_b, per, nrt_b);
            bool mine = false;
            if (tid < nrt_b && nct_b > 0) {
                const int first = tid / rb * rb, high = min(rb, nrt_b - first);  // the band's first row tile and height
                const int pick = ((tid - first) * 2 + 1) * nct_b / (high * 2);
                mine = (first * nct_b + pick * high + tid - first) / per_b == xcd;
            }
            const uint64_t bits = __builtin_amdgcn_ballot_w64(mine);
            if ((tid & 63) == 0) owned[wave] = bits;
            __syncthreads();
            // the helpers of a sample share each of these row tiles; thread t takes a quarter of each line group of the t / 4-th row
            const int rows = (BM + hn - 1) / hn;
            int p = -1, cnt = 0;
            for (int w = 0; w < 4; ++w)
                for (uint64_t m = owned[w]; m && cnt < 128; m &= m - 1, cnt += rows) {
                    const int i = (tid >> 2) - cnt, rt = w * 64 + __builtin_ctzll(m);
                    if (i >= 0 && i < rows && h0 * rows + i < BM) p = rt * BM + h0 * rows + i;
                }
            __syncthreads();                                                    // the list is read; the loads below land on it
            const __amdgpu_buffer_rsrc_t rsrc = make_uniform_rsrc(f + (size_t)(s.tok0 + s.vs) * d, (uint32_t)((size_t)s.V * d * sizeof(uint16_t)));
            const uint32_t sink = __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(lds_ptr_t)ring + wave * 256);
            if (p >= 0 && p < s.M) {
                const int off = min(max(pruned[(size_t)hb * max_V + p], 0), s.V - 1) * d * 2 + (tid & 3) * 128;
                const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
                for (int c = 0; c < d * 2; c += 512) {                           // behind the sample's rows: outside the buffer, not read
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(size_t)sink, 4, off, c, 0, 0);
                    if (c == 0) {
                        wait_loads<0>();
                        if (__builtin_amdgcn_s_memrealtime() - t0 < COS_CACHED_TICKS) break;    // in a cache already: nothing to help with
                    }
                    __builtin_amdgcn_s_sleep(20);                                // 0.7 us: no faster than the tiles
                }
            }
            wait_loads<0>();
        }
        return;
    }
    const SampleGeom s = sample_geom(b, seq_off, vis_start, vis_count, kept_off, max_V, max_keep);
    const int nrt_b = min((s.M + BM - 1) / BM, nrt_launch), nct_b = min((s.k + BN - 1) / BN, nct_launch);
    const int tiles_b = nrt_b * nct_b;
    const bool derive = SPLIT && !prepared;                // uniform
    if (derive) {
        // a sample that keeps everything has no tiles: its table entries are written here
        if (s.M <= 0 && id == 0 && xcd == 0 && blockIdx.y == 0)
            for (int r = threadIdx.x; r < s.k; r += 512)
                table[(size_t)b * VP + min(max(kept_idx[s.k0 + r], 0), s.V - 1)] = table_entry_kept(r);
    }
    const int per_b = TM == 4 ? 32 : (tiles_b + 7) / 8;
    if (TM < 4 && id >= per_b) return;
    const int t_lin = TM == 4 ? id : xcd * per_b + id;
    if (t_lin >= tiles_b) return;
    int rt, ct;
    {
        // bands about as high as a run's block is wide (RB was chosen that way for the launch's grid; a smaller
        // sample gets its own)
        const int rb = band_height(RB, per_b, per, nrt_b);
        const int band = rb * nct_b, nfull = nrt_b / rb;
        if (t_lin < nfull * band) { const int rem = t_lin % band; rt = (t_lin / band) * rb + rem % rb; ct = rem / rb; }
        else { const int t2 = t_lin - nfull * band, rl = nrt_b - nfull * rb; rt = nfull * rb + t2 % rl; ct = t2 / rl; }
    }

    const int tid = threadIdx.x, wave = (tid >> 6) & 3, lane = tid & 63;
    const bool loader = tid >> 8;                          // waves 4..7 only move data, waves 0..3 only compute
    const int wm = wave >> 1, wn = wave & 1;
    const int r16 = lane & 15, g4 = lane >> 4;
    int32_t* pr = pruned + (size_t)b * max_V;
    const int32_t* kp = kept_idx + s.k0;
    const float* rn = rnorm + (size_t)b * max_V;
    const size_t base = (size_t)(s.tok0 + s.vs) * d;

    // byte offset of this lane inside the visual block for each of its direct loads (rows past the end
    // re-read row 0; masked later); the k-slice is added through the scalar offset
    const __amdgpu_buffer_rsrc_t rsrc = make_uniform_rsrc(f + base, (uint32_t)((size_t)s.V * d * sizeof(uint16_t)));
    // The A rows of a wave's loads: the first half (quarter) of its loads are the rows of the first half (quarter) of every computing
    // wave's 16-row blocks, so that a part of a row tile is the first part of everybody's work.
    auto a_row = [&](int i) { return (wave >> 1) * (BM / 2) + (i >> 1) * 32 + (wave & 1) * 16 + (i & 1) * 8; };
    // the sample's pruned row behind row `row` of the LDS tile, for the rows that a part has
    const int p0 = rt * BM + part * (BM >> cut);
    if (TM == 4)
        while (cut < 2 && s.M - p0 <= (BM / 2 >> cut)) ++cut;                   // few rows left: a smaller part has them
    auto pruned_row = [&](int row) { return p0 + row / (BM / 2) * (BM / 2 >> cut) + row % (BM / 2); };
    if (p0 >= s.M) return;
    int a_off[A_LD], b_off[B_LD];
    if (derive) {
        // the p-th pruned token is p + the number r of kept tokens in front of it: the first r with kept[r] - r > p
        int* kl = reinterpret_cast<int*>(ring);
        for (int t = tid; t < s.k; t += 512) kl[t] = min(max(kp[t], 0), s.V - 1);
        __syncthreads();
        if (loader) {
#pragma unroll
            for (int i = 0; i < A_LD; ++i) {
                const int row = a_row(i) + (lane >> 3);
                const int p = min(rt * BM + row, s.M - 1);
                int lo = 0, hi = s.k;
                while (lo < hi) { const int mid = (lo + hi) >> 1; if (kl[mid] - mid > p) hi = mid; else lo = mid + 1; }
                const int m = min(p + lo, s.V - 1);
                a_off[i] = m * d * 2 + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
                if (ct == 0 && blockIdx.y == 0 && (lane & 7) == 0 && rt * BM + row < s.M) pr[p] = m;
            }
        } else if (rt == 0 && blockIdx.y == 0) {
            for (int t = tid; t < BN; t += 256)
                if (ct * BN + t < s.k) table[(size_t)b * VP + kl[ct * BN + t]] = table_entry_kept(ct * BN + t);
        }
        __syncthreads();                                   // the ring is free for the tiles
    } else {
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            const int row = a_row(i) + (lane >> 3);
            const int cg = (lane & 7) ^ ((row >> 1) & 7);
            const int p = pruned_row(row);
            const int m = min(max((p < s.M) ? pr[p] : pr[0], 0), s.V - 1);
            a_off[i] = m * d * 2 + cg * 16;
        }
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        const int row = wave * (BN / 4) + i * 8 + (lane >> 3);
        const int cg = (lane & 7) ^ ((row >> 1) & 7);
        const int r = ct * BN + row;
        const int j = min(max(kp[(r < s.k) ? r : 0], 0), s.V - 1);
        b_off[i] = j * d * 2 + cg * 16;
    }
    if constexpr (!SPLIT)
        for (int t = tid; t < BN; t += 512) {
            const int r = ct * BN + t;
            // 1 / norm of the kept row in slot r: stored by slot, or by token when the selection launch computed them
            rnB[t] = (r < s.k) ? rn[prepared ? min(max(kp[r], 0), s.V - 1) : r] : 0.f;
        }
    // slice blockIdx.y of the contraction (ksplit slices of nkt stages each)
    const int nkt = SPLIT ? (d / COS_BK) / ksplit : d / COS_BK;
    const int kt0 = (int)blockIdx.y * nkt;
    // LDS destinations are wave-uniform: this wave's first row of the A (B) tile, made a scalar once so
    // that a load costs one scalar add for its M0 value and no vector instruction
    const uint32_t ring0 = (uint32_t)(size_t)(lds_ptr_t)ring;
    const uint32_t a_lds = __builtin_amdgcn_readfirstlane(ring0 + a_row(0) * 128);
    const uint32_t b_lds = __builtin_amdgcn_readfirstlane(ring0 + BM * 128 + wave * (BN / 4) * 128);
    auto issue = [&](int kt, int stage, auto rows) {
        constexpr int A_N = A_LD * decltype(rows)::value / (TM * 2);
#pragma unroll
        for (int i = 0; i < A_N; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(size_t)(a_lds + stage * STAGE + ((i >> 1) * 32 + (i & 1) * 8) * 128), 16,
                                                     a_off[i], (kt0 + kt) * (COS_BK * 2), 0, 0);
#pragma unroll
        for (int i = 0; i < B_LD; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_ptr_t)(size_t)(b_lds + stage * STAGE + i * 8 * 128), 16,
                                                     b_off[i], (kt0 + kt) * (COS_BK * 2), 0, 0);
    };

    constexpr int RBK = TM * 2;                         // 16-row blocks of a wave's (TM*32) x (CBK*16) tile
    f32x4 acc[RBK][CBK];
#pragma unroll
    for (int i = 0; i < RBK; ++i)
#pragma unroll
        for (int j = 0; j < CBK; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 bb[SPLIT ? CBK : 1];                           // SPLIT: B B^T of each column block
#pragma unroll
    for (int j = 0; j < (SPLIT ? CBK : 1); ++j) bb[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool squares = SPLIT && rt == 0 && wm == 0;    // uniform

    // a wave whose rows or columns all lie past the sample's only keeps step: its products would cost power, and clock with it
    // (with the smaller parts for few rows above: 80 samples of 300 .. 800 rows at d = 2048 118 -> 111 us, 32 of 600 .. 1200 at 4096 149 -> 148)
    const bool none = ct * BN + wn * (BN / 2) >= s.k || pruned_row(wm * (BM / 2)) >= s.M;

    // A wave that issues a direct load waits for room in the CU's vector-memory queue; in a computing wave
    // that wait stalls the MFMA stream, so the loads have waves of their own.  One s_barrier per stage:
    // the loaders arrive at the kt-th once stage kt has landed, the consumers once they have read stage kt-1 out of LDS,
    // whose slot the loaders then refill with stage kt+COS_NS-1.
    auto sweep = [&](auto rows) {
    constexpr int NR = decltype(rows)::value;              // 16-row blocks of a computing wave: all RBK, or the first of them
    if (loader) {
        constexpr int LPS = A_LD * NR / RBK + B_LD;         // loads per wave and stage
#pragma unroll
        for (int st = 0; st < COS_NS - 1; ++st)
            if (st < nkt) issue(st, st, rows);
        for (int kt = 0; kt < nkt; ++kt) {
            if (kt + COS_NS - 2 <= nkt - 1) wait_loads_and_barrier<(COS_NS - 2) * LPS>();
            else wait_loads_and_barrier<0>();
            if (kt + COS_NS - 1 < nkt) issue(kt + COS_NS - 1, (kt + COS_NS - 1) % COS_NS, rows);
        }
    } else {
        // A stage is two k-steps of 32.  The fragments of the next k-step are read behind the first MFMAs of this one, across
        // the barrier too (the one for stage kt+1 lies between the two k-steps of stage kt), so that neither LDS latency nor the
        // barrier leaves the matrix core idle.
        const int sw = (r16 >> 1) & 7;                  // rows 16 i + r16 all share it
        const int fa = (wm * (TM * 32) + r16) * 128, fb = BM * 128 + (wn * (BN / 2) + r16) * 128;
        const int ch0 = (g4 ^ sw) << 4, ch1 = ((4 + g4) ^ sw) << 4;
        bf16x8 fr[2][RBK + CBK];                        // [k-step][row blocks, column blocks]
        auto read_one = [&](const char* sb, int ks, int f) {
            fr[ks][f] = *reinterpret_cast<const bf16x8*>(sb + (f < RBK ? fa + f * 2048 : fb + (f - RBK) * 2048) + (ks ? ch1 : ch0));
        };
        auto multiply = [&](int ks, const char* next, bool read) {  // MFMAs of k-step ks; reads the other one's fragments from `next`
#pragma unroll
            for (int n = 0; n < NR * CBK; ++n) {
                const int i = n / CBK, j = n % CBK;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[ks][i], fr[ks][RBK + j], acc[i][j], 0, 0, 0);
                if (read && n < NR + CBK) {
                    __builtin_amdgcn_sched_barrier(0);
                    read_one(next, ks ^ 1, n < NR ? n : RBK + n - NR);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (squares) {
#pragma unroll
                for (int j = 0; j < (SPLIT ? CBK : 0); ++j) bb[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[ks][RBK + j], fr[ks][RBK + j], bb[j], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        wait_loads_and_barrier<0>();
        if (none) {
            for (int kt = 0; kt + 1 < nkt; ++kt) phase_barrier();
            return;
        }
#pragma unroll
        for (int f = 0; f < NR + CBK; ++f) read_one(ring, 0, f < NR ? f : RBK + f - NR);
        int slot = 0;
        for (int kt = 0; kt + 1 < nkt; ++kt) {
            const char* sb = ring + slot * STAGE;
            slot = slot + 1 == COS_NS ? 0 : slot + 1;
            multiply(0, sb, true);
            __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0): stage kt is in registers
            phase_barrier();
            multiply(1, ring + slot * STAGE, true);
        }
        multiply(0, ring + slot * STAGE, true);
        multiply(1, nullptr, false);
    }
    };
    if constexpr (TM == 4) {
        if (cut == 2) sweep(std::integral_constant<int, RBK / 4>{});
        else if (cut) sweep(std::integral_constant<int, RBK / 2>{});
        else sweep(std::integral_constant<int, RBK>{});
    } else sweep(std::integral_constant<int, RBK>{});

    if constexpr (SPLIT) {
        // partial products of this k-slice: block (slice, tile) of BM x 128 floats, summed by cos_reduce_argmax
        const int tile_id = (b * nrt_launch + rt) * nct_launch + ct;
        const int n_tiles = nB * nrt_launch * nct_launch;
        float* blk = dots + ((size_t)blockIdx.y * n_tiles + tile_id) * (BM * BN);
        if (loader) return;
        if (squares && (r16 >> 2) == g4) {
            float* sb = sq + (((size_t)blockIdx.y * nB + b) * nct_launch + ct) * 128 + wn * (BN / 2) + r16;
#pragma unroll
            for (int j = 0; j < (SPLIT ? CBK : 0); ++j) {
                const f32x4 v = bb[j];
                sb[j * 16] = (r16 & 2) ? ((r16 & 1) ? v[3] : v[2]) : ((r16 & 1) ? v[1] : v[0]);
            }
        }
#pragma unroll
        for (int i = 0; i < RBK; ++i)
#pragma unroll
            for (int j = 0; j < CBK; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    blk[(wm * (TM * 32) + i * 16 + g4 * 4 + e) * BN + wn * (BN / 2) + j * 16 + r16] = acc[i][j][e];
        return;
    }
    // epilogue: dot * rn_col (the cosine up to the row's own positive norm, which is the same for all of
    // its candidates); per row, best (value, slot) over this tile's columns.
    // The 32 candidates of a row (16 lanes x 2 wave columns) meet in LDS (the ring is free once all waves
    // are past the loop): every lane folds its four columns of a row into one candidate (branch-free; equal
    // values keep the lower slot) and stores it, then two threads per row scan 16 candidates each in
    // ascending slot order.  Rows are padded to 17 entries so that the scan of 32 different rows hits 32
    // different banks.
    __syncthreads();                                           // all waves are done with the ring
    float2* cand = reinterpret_cast<float2*>(ring);            // [BM][2][17]
    if (!loader) {
        float rn_col[CBK];                                     // read once: the compiler takes the stores below for possible changes
#pragma unroll
        for (int j = 0; j < CBK; ++j) rn_col[j] = rnB[wn * (BN / 2) + j * 16 + r16];
#pragma unroll
        for (int i = 0; i < RBK; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = wm * (TM * 32) + i * 16 + g4 * 4 + e;
                float best = -INFINITY; int bidx = 0x7FFFFFFF;
#pragma unroll
                for (int j = 0; j < CBK; ++j) {
                    const int col = wn * (BN / 2) + j * 16 + r16, slot = ct * BN + col;
                    const float v = (slot < s.k) ? acc[i][j][e] * rn_col[j] : -INFINITY;
                    const bool take = v > best;                // equal values: the lower slot stays
                    best = take ? v : best; bidx = take ? slot : bidx;
                }
                cand[(row * 2 + wn) * 17 + r16] = make_float2(best, __int_as_float(bidx));
            }
    }
    __syncthreads();
    for (int t = tid; t < BM * 2; t += 512) {
        const int row = t >> 1, side = t & 1;                  // side 0: slots of wave column 0 (lower slots)
        const float2* cr = cand + (row * 2 + side) * 17;
        float best = -INFINITY; int bidx = 0x7FFFFFFF;
#pragma unroll
        for (int q2 = 0; q2 < 16; ++q2) {
            const float2 a = cr[q2];
            const int ia = __float_as_int(a.y);
            const bool take = (a.x > best) | ((a.x == best) & (ia < bidx));
            best = take ? a.x : best; bidx = take ? ia : bidx;
        }
        const float ov = __shfl_xor(best, 1, WAVE);
        const int oi = __shfl_xor(bidx, 1, WAVE);
        const bool take = (ov > best) | ((ov == best) & (oi < bidx));
        best = take ? ov : best; bidx = take ? oi : bidx;
        const int p = pruned_row(row);
        if (side == 0 && p < s.M && row % (BM / 2) < (BM / 2 >> cut)) {
            const int tok = min(max(pr[p], 0), s.V - 1);
            atomicMax(table + (size_t)b * VP + tok, table_entry(best, bidx));
        }
    }
#endif
}

// ---- split-K second step: sum the k-slices, scale by the kept row's 1/norm, argmax over all slots ----
// Used when the similarity matrix has too few tiles to occupy the chip (short sequences): the GEMM is
// then cut along the contraction instead, and one, two or four waves per pruned row finish the job here, each taking every
// `wpr`-th column tile.  Slices are added in ascending order and ties go to the lowest slot, so the result is deterministic.
// Bound by the latency of its loads, so a wave should go round its loop once, and all loads of a turn (all slices of both halves of
// the tile, the norms) are requested together: without a branch around any of them, since each branch costs a wait and some tens
// of cycles.  (One wave per row, loads under conditions: 1400 rows x 600 slots x 2 slices 14.0 us, now 6.2; 486 x 243 x 4 slices
// 6.8 us, now 3.8; 921 x 103 x 16 4.5 us, 3.9 with norms read by token, then 4.4.)  No request waits for the sample's
// offsets either, which only say what of the answers counts (921 x 103 x 8 3.8 us, now 3.4; 486 x 243 x 4 3.6, 3.4).
template <int wpr, int SLICES>
__global__ __launch_bounds__(256) void cos_reduce_argmax(
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ vis_start, const int32_t* __restrict__ vis_count,
    const int32_t* __restrict__ kept_off,
    int max_V, int max_keep, const int32_t* __restrict__ pruned,
    const float* __restrict__ dots, int n_tiles, int nrt_launch, int nct_launch,
    table_t* __restrict__ table, int VP, const float* __restrict__ sq, int nB) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int BM = 64;
    extern __shared__ float rn_s[];             // [kept slots] 1 / norm, from the k-slices' sums of squares
    __shared__ float2 join[4];
    const int b = blockIdx.y;
    int t0 = seq_off[b], t1 = seq_off[b + 1], vs0 = vis_start[b], vc = vis_count[b], k0 = kept_off[b], k1 = kept_off[b + 1];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    constexpr int rows = 4 / wpr;
    const int p = blockIdx.x * rows + wave / wpr, part = wave % wpr;
    const int rt = p / BM, lr = p % BM;
    // Loads without branches: tiles beyond the launch's lie outside the buffer and read as 0 (what a tile holds beyond the sample's rows
    // and slots is not looked at).
    const uint32_t slice = (uint32_t)n_tiles * (BM * COS_BN * 4);
    const __amdgpu_buffer_rsrc_t dots_r = make_uniform_rsrc(dots, (uint32_t)SLICES * slice);
    float v[2][SLICES];
    auto request = [&](int ct) {
        const uint32_t tile_id = (uint32_t)((b * nrt_launch + rt) * nct_launch + ct);
        const uint32_t at = ct < nct_launch && rt < nrt_launch ? (tile_id * BM + lr) * (COS_BN * 4) + lane * 4 : 0xC0000000u;
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int ks = 0; ks < SLICES; ++ks)
                v[half][ks] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(dots_r, at + ks * slice + half * 256, 0, 0));
    };
    request(part);
    const int entry = pruned[(size_t)b * max_V + min(p, max_V - 1)];
    const __amdgpu_buffer_rsrc_t sq_r = make_uniform_rsrc(sq, (uint32_t)(SLICES * nB * nct_launch) * 512u);
    float sl[SLICES];
    auto squares = [&](int t) {
#pragma unroll
        for (int ks = 0; ks < SLICES; ++ks)
            sl[ks] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(sq_r, (((ks * nB + b) * nct_launch + t / COS_BN) * 128 + t % COS_BN) * 4, 0, 0));
    };
    squares(min((int)threadIdx.x, max_keep - 1));
    request_together(t0, t1, vs0, vc, k0, k1);
    const SampleGeom s = geom_of(t0, t1, vs0, vc, k0, k1, max_V, max_keep);
    if (s.k <= 0 || (int)blockIdx.x * rows >= s.M) return;
    const int nct = (p < s.M) ? (s.k + COS_BN - 1) / COS_BN : 0;
    const int tok = min(max(entry, 0), s.V - 1);
    for (int t = threadIdx.x; t < s.k;) {
        float ss = 0.f;
#pragma unroll
        for (int ks = 0; ks < SLICES; ++ks) ss += sl[ks];
        rn_s[t] = reciprocal_norm(ss);
        t += 256;
        if (t < s.k) squares(t);
    }
    __syncthreads();
    float best = -INFINITY; int bidx = 0x7FFFFFFF;
    for (int ct = part; ct < nct; ct += wpr) {
        if (ct != part) request(ct);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int slot = ct * COS_BN + half * 64 + lane;
            if (slot < s.k) {
                float sum = 0.f;
#pragma unroll
                for (int ks = 0; ks < SLICES; ++ks) sum += v[half][ks];        // ascending slices
                const float val = sum * rn_s[slot];
                if (val > best) { best = val; bidx = slot; }
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(best, o, WAVE);
        const int oi = __shfl_xor(bidx, o, WAVE);
        const bool take = (ov > best) | ((ov == best) & (oi < bidx));
        best = take ? ov : best; bidx = take ? oi : bidx;
    }
    if (wpr > 1) {
        if (lane == 0) join[wave] = make_float2(best, __int_as_float(bidx));
        __syncthreads();
        for (int w = 1; w < wpr; ++w) {
            const float2 o = join[(wave & ~(wpr - 1)) + w];
            const int oi = __float_as_int(o.y);
            const bool take = (o.x > best) | ((o.x == best) & (oi < bidx));
            best = take ? o.x : best; bidx = take ? oi : bidx;
        }
    }
    if (lane == 0 && part == 0 && p < s.M) table[(size_t)b * VP + tok] = table_entry(best, min(max(bidx, 0), s.k - 1));
#endif
}

// ---- cosine + argmax, generic: one workgroup per pruned row ---
// 16 groups of 16 lanes, each takes every 16th kept slot: 16-byte loads and a reduction inside a data-parallel row of
// 16 lanes (a whole wave per slot with scalar loads and a 64-lane reduction: 10 us at 108 x 36 rows of 256 floats, launch
// included; a slot at a time 5.9; four slots and four chunks of each at a time, which are requested together, 4.7).
template <typename T>
__global__ __launch_bounds__(256) void cos_argmax_generic(
    const T* __restrict__ f, int d, const int32_t* __restrict__ seq_off, const int32_t* __restrict__ vis_start,
    const int32_t* __restrict__ vis_count, const int32_t* __restrict__ kept_idx, const int32_t* __restrict__ kept_off,
    int max_V, int max_keep, const int32_t* __restrict__ pruned, const float* __restrict__ rnorm,
    table_t* __restrict__ table, int VP, int rn_by_token) {
    const int p = blockIdx.x, b = blockIdx.y;
    const SampleGeom s = sample_geom(b, seq_off, vis_start, vis_count, kept_off, max_V, max_keep);
    if (p >= s.M) return;
    __shared__ float2 red[16];
    const int grp = threadIdx.x >> 4, l16 = threadIdx.x & 15;
    const int m = min(max(pruned[(size_t)b * max_V + p], 0), s.V - 1);
    const int32_t* kp = kept_idx + s.k0;
    const float* rn = rnorm + (size_t)b * max_V;
    const T* xm = f + (size_t)(s.tok0 + s.vs + m) * d;
    const uint4* xc = reinterpret_cast<const uint4*>(xm);
    const int nch = d / (int)(16 / sizeof(T));
    float bv = -INFINITY; int bi = 0x7FFFFFFF;
    for (int r0 = grp; r0 < s.k; r0 += 64) {
        // four slots of a group at once: their tokens, then their rows and norms
        int tok[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) tok[i] = kp[min(r0 + 16 * i, s.k - 1)];
        const uint4* row[4];
        float scale[4], dot[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            tok[i] = min(max(tok[i], 0), s.V - 1);
            row[i] = reinterpret_cast<const uint4*>(f + (size_t)(s.tok0 + s.vs + tok[i]) * d);
            scale[i] = rn[rn_by_token ? tok[i] : min(r0 + 16 * i, s.k - 1)];      // the pruned row's own norm scales all its candidates alike
            dot[i] = 0.f;
        }
        for (int c0 = l16; c0 < nch; c0 += 64) {
            uint4 x[4], y[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int c = min(c0 + 16 * u, nch - 1);
                x[u] = xc[c];
#pragma unroll
                for (int i = 0; i < 4; ++i) y[i][u] = row[i][c];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = chunk_dot<T>(x[u], y[i][u], dot[i]);
                    dot[i] = c0 + 16 * u < nch ? v : dot[i];
                }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = row16_sum(dot[i]) * scale[i];
            if (r0 + 16 * i < s.k && v > bv) { bv = v; bi = r0 + 16 * i; }
        }
    }
    if (l16 == 0) red[grp] = make_float2(bv, __int_as_float(bi));
    __syncthreads();
    if (threadIdx.x == 0) {
        float2 a = red[0];
        for (int w = 1; w < 16; ++w) {
            const float2 c2 = red[w];
            if (c2.x > a.x || (c2.x == a.x && __float_as_int(c2.y) < __float_as_int(a.y))) a = c2;
        }
        table[(size_t)b * VP + m] = table_entry(a.x, min(max(__float_as_int(a.y), 0), s.k - 1));
    }
}

// ---- scatter-average + compaction ----------------------------------------------------------
// One workgroup per output row.  A caller who does not know the kept counts has only the longest sample for a bound, many times the rows that there
// are: the launch is then sized for the rows to expect, and the workgroups of a sample with more of them take the rest in further turns
// (one workgroup for every row that there could be: 231 of 1152 rows of 8 KB 7.3 -> 7.0 us, 493 of 3773 10.8 -> 10.4, 1951 of 3773
// 13.0 -> 12.3, 16 samples with 493 .. 1505 of 2688 90 -> 85).  A merged
// row first finds its members: the four waves scan the
// table of the sample (a quarter each, coalesced; the low word of an entry names the slot, and the kept
// token's own entry makes it a member like the others), keep the matches in ascending token
// order (ballot + popcount, no atomics) and the four pieces are joined into one list in LDS; the
// workgroup of a slot also writes the slot into `assign` for each of its members.  The member
// rows are then streamed four at a time so that eight 16-byte loads per thread are in flight;
// accumulation order is ascending token index, so the result does not depend on the unrolling.  A slot
// with more members than the LDS list holds is processed in windows of SCAT_LIST members (re-scan).
// Bound by its chain of trips to memory (the sample's offsets; table and kept position; rows) in small launches, by the rows' traffic
// in large ones.  No load is under a condition: each one that was cost a branch and often a wait (231 rows of 8 KB from
// 1024: 9.4 -> 7.5 us, 1951 from 3773: 16.5 -> 13.0, two payloads of 1040 from 3709: 20 -> 17.5).
constexpr int SCAT_LIST = 256;     // members staged per pass
[[maybe_unused]] constexpr int SCAT_WAVE = SCAT_LIST / 4;
template <typename T, int CPT>     // CPT: 16-byte chunks per thread per pass
__global__ __launch_bounds__(256, CPT == 2 ? 7 : 5) void merge_scatter_kernel(
    const T* __restrict__ x0, const T* __restrict__ x1, int d, const int32_t* __restrict__ seq_off, const int32_t* __restrict__ vis_start,
    const int32_t* __restrict__ vis_count, const int32_t* __restrict__ kept_idx, const int32_t* __restrict__ kept_off,
    int max_V, int max_keep, int max_out, int mode, const int32_t* __restrict__ out_off, const table_t* __restrict__ table, int VP,
    const int32_t* __restrict__ vis_off, T* __restrict__ y0, T* __restrict__ y1, int32_t* __restrict__ assign_out,
    int32_t* __restrict__ counts_out, int32_t* __restrict__ src_pos_out) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int EPC = 16 / sizeof(T);
    // a row may be cut into nslice column slices, one workgroup each (few output rows: more workgroups)
    constexpr int nslice = CPT == 1 ? 2 : 1;
    const int step = gridDim.x / nslice;
    for (int o = blockIdx.x / nslice;;) {
    int slice = blockIdx.x % nslice, b = blockIdx.y;
    asm volatile("" : "+s"(slice), "+s"(b), "+s"(o));      // a further turn reads everything anew: nothing is kept in registers for it
    // blockIdx.z selects the payload (a second one shares the routing: key and value caches); the
    // index outputs are written by the first payload's workgroups only
    const T* __restrict__ x = blockIdx.z ? x1 : x0;
    T* __restrict__ y = blockIdx.z ? y1 : y0;
    int32_t* counts = (blockIdx.z || slice) ? nullptr : counts_out;
    int32_t* src_pos = (blockIdx.z || slice) ? nullptr : src_pos_out;
    int vo0 = vis_off[b], oo0 = out_off[b];
    const SampleGeom s = sample_geom(b, seq_off, vis_start, vis_count, kept_off, max_V, max_keep, vo0, oo0);
    int32_t* assign = (blockIdx.z || slice || !assign_out) ? nullptr : assign_out + vo0;
    const int N_m = min(s.N - s.M, max_out);               // the caller's bound on the rows of y, whatever the sample's sizes say
    if (o >= N_m) return;
    __shared__ int list[SCAT_LIST];
    __shared__ int stage[4][SCAT_WAVE];
    __shared__ int wcnt[4];
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
    const int nch = d / EPC;
    const int c_per = (nch + nslice - 1) / nslice;
    const int c_lo = slice * c_per, c_hi = min(nch, c_lo + c_per);          // this workgroup's 16-byte chunks
    // table of this sample, read two entries (16 bytes) per lane; a wave takes a contiguous part of it
    // (a multiple of 128 entries so that every lane takes part in each ballot)
    const __amdgpu_buffer_rsrc_t tab = make_uniform_rsrc(table + (size_t)b * VP, (uint32_t)VP * 8u);
    const int part_len = ((s.V + 511) >> 9) << 7;
    const int e0 = wave * part_len;
    const int n_it = part_len >> 7;
    T* yrow = y + (size_t)(oo0 + o) * d;
    int src = -1, len = 1, r = 0;
    int wbase = 0;                                         // members found by the waves before this one
    bool fits = true;
    uint32_t want = 0;                                     // low word of the entries of this row's slot
    // scan this wave's part: fn(token, ordinal among this wave's matches) for every match, ascending
    auto scan = [&](auto&& fn) {
        int cnt = 0;
        for (int it0 = 0; it0 < n_it; it0 += 4) {
            uint4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = e0 + (it0 + u) * 128 + lane * 2;
                // beyond this wave's part: outside the buffer, reads as 0, which no slot's low word is
                v[u] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(tab, it0 + u < n_it ? (uint32_t)i * 8u : 0xFFFFFFF0u, 0, 0));
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = e0 + (it0 + u) * 128 + lane * 2;
                const bool m0 = (v[u].x == want) && (i < s.V), m1 = (v[u].z == want) && (i + 1 < s.V);
                const unsigned long long lt = (1ull << lane) - 1ull;
                const unsigned long long b0 = __builtin_amdgcn_ballot_w64(m0), b1 = __builtin_amdgcn_ballot_w64(m1);
                int ord = cnt + __popcll(b0 & lt) + __popcll(b1 & lt);
                if (m0) fn(i, ord++);
                if (m1) fn(i + 1, ord++);
                cnt += __popcll(b0) + __popcll(b1);
            }
        }
        return cnt;
    };
    if (o < s.vs) src = o;
    else if (o >= s.vs + s.k) src = o + s.M;
    else {
        r = o - s.vs;
        want = 0xFFFFFFFFu - (uint32_t)r;
        const int kept_tok = min(max(kept_idx[s.k0 + r], 0), s.V - 1);
        const int cnt = scan([&](int tok, int ord) {
            if (ord < SCAT_WAVE) stage[wave][ord] = tok;
            if (assign) assign[tok] = r;
        });
        if (lane == 0) wcnt[wave] = cnt;
        __syncthreads();
        len = wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3];
        fits = wcnt[0] <= SCAT_WAVE && wcnt[1] <= SCAT_WAVE && wcnt[2] <= SCAT_WAVE && wcnt[3] <= SCAT_WAVE;
        for (int w = 0; w < wave; ++w) wbase += wcnt[w];
        if (tid == 0) {
            if (src_pos) src_pos[oo0 + o] = s.vs + kept_tok;
            if (counts) counts[s.k0 + r] = len;
        }
        if (len <= 1) src = s.vs + kept_tok;               // nothing absorbed: bit-exact copy
        else if (fits) {
            if (lane < cnt) list[wbase + lane] = stage[wave][lane];
            __syncthreads();
        }
    }
    if (src >= 0) {
        if (tid == 0 && src_pos && (o < s.vs || o >= s.vs + s.k)) src_pos[oo0 + o] = src;
        const uint4* in = reinterpret_cast<const uint4*>(x + (size_t)(s.tok0 + src) * d);
        uint4* out = reinterpret_cast<uint4*>(yrow);
        for (int c = c_lo + tid; c < c_hi; c += 512) {
            const uint4 w0 = in[c], w1 = in[min(c + 256, c_hi - 1)];
            out[c] = w0;
            if (c + 256 < c_hi) out[c + 256] = w1;
        }
        o += step;
        if (o >= N_m) return;
        __syncthreads();                                   // a further turn writes the lists
        continue;
    }
    // members with ordinal in [win0, win0 + SCAT_LIST) -> list (only when the first scan did not fit)
    auto fill_window = [&](int win0) {
        scan([&](int tok, int ord) { const int pos = wbase + ord - win0; if (pos >= 0 && pos < SCAT_LIST) list[pos] = tok; });
    };
    const T* xv = x + (size_t)(s.tok0 + s.vs) * d;
    const float inv = (mode == D3TOM_MERGE_MEAN) ? (float)len : 1.0f;
    auto add_row = [&](float (&acc)[CPT][EPC], const uint4 (&w)[CPT]) {
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            if constexpr (sizeof(T) == 2) {
                acc[u][0] += bf16_lo(w[u].x); acc[u][1] += bf16_hi(w[u].x);
                acc[u][2] += bf16_lo(w[u].y); acc[u][3] += bf16_hi(w[u].y);
                acc[u][4] += bf16_lo(w[u].z); acc[u][5] += bf16_hi(w[u].z);
                acc[u][6] += bf16_lo(w[u].w); acc[u][7] += bf16_hi(w[u].w);
            } else {
                acc[u][0] += __uint_as_float(w[u].x); acc[u][1] += __uint_as_float(w[u].y);
                acc[u][2] += __uint_as_float(w[u].z); acc[u][3] += __uint_as_float(w[u].w);
            }
        }
    };
    for (int cb = c_lo; cb < c_hi; cb += 256 * CPT) {     // uniform trip count: the loop body has barriers
        const int c0 = cb + tid;
        int cc[CPT];                                       // chunks to read; what a thread beyond the slice's end adds up is not stored
#pragma unroll
        for (int u = 0; u < CPT; ++u) cc[u] = min(c0 + 256 * u, c_hi - 1);
        float acc[CPT][EPC];
#pragma unroll
        for (int u = 0; u < CPT; ++u)
#pragma unroll
            for (int e = 0; e < EPC; ++e) acc[u][e] = 0.f;
        for (int l0 = 0; l0 < len; l0 += SCAT_LIST) {
            const int ln = min(SCAT_LIST, len - l0);
            if (!fits) {                                   // uniform
                __syncthreads();
                fill_window(l0);
                __syncthreads();
            }
            // as many rows as registers allow requested together, the last ones (each of which would cost a trip of its own) too
            auto rows = [&](int t, auto n) {
                constexpr int R = decltype(n)::value;
                uint4 w[R][CPT];
#pragma unroll
                for (int m = 0; m < R; ++m) {
                    const uint4* row = reinterpret_cast<const uint4*>(xv + (size_t)list[t + m] * d);
#pragma unroll
                    for (int u = 0; u < CPT; ++u) w[m][u] = row[cc[u]];
                }
#pragma unroll
                for (int m = 0; m < R; ++m) add_row(acc, w[m]);
            };
            constexpr int NB = 8 / CPT;
            int t = 0;
            for (; t + NB <= ln; t += NB) rows(t, std::integral_constant<int, NB>());
            switch (ln - t) {
                case 1: rows(t, std::integral_constant<int, 1>()); break;
                case 2: rows(t, std::integral_constant<int, 2>()); break;
                case 3: rows(t, std::integral_constant<int, 3>()); break;
                case 4: if constexpr (NB > 4) rows(t, std::integral_constant<int, 4>()); break;
                case 5: if constexpr (NB > 4) rows(t, std::integral_constant<int, 5>()); break;
                case 6: if constexpr (NB > 4) rows(t, std::integral_constant<int, 6>()); break;
                case 7: if constexpr (NB > 4) rows(t, std::integral_constant<int, 7>()); break;
            }
        }
#pragma unroll
        for (int u = 0; u < CPT; ++u) {
            const int c = c0 + 256 * u;
            if (c < c_hi) {
                uint4 w;
                if constexpr (sizeof(T) == 2) {
                    // The quotients one by one: seen as pairs by the compiler, because the conversion takes two, all sums above became
                    // pairs of registers, with a wait at every row's addition (16 samples 86 -> 105 us, two payloads 18.3 -> 21.6).
                    float q[EPC];
#pragma unroll
                    for (int e = 0; e < EPC; ++e) {
                        q[e] = acc[u][e] / inv;
                        asm volatile("" : "+v"(q[e]));
                    }
                    w.x = pack_bf16x2(q[0], q[1]);
                    w.y = pack_bf16x2(q[2], q[3]);
                    w.z = pack_bf16x2(q[4], q[5]);
                    w.w = pack_bf16x2(q[6], q[7]);
                } else {
                    w.x = __float_as_uint(acc[u][0] / inv); w.y = __float_as_uint(acc[u][1] / inv);
                    w.z = __float_as_uint(acc[u][2] / inv); w.w = __float_as_uint(acc[u][3] / inv);
                }
                reinterpret_cast<uint4*>(yrow)[c] = w;
            }
        }
    }
    o += step;
    if (o >= N_m) return;
    __syncthreads();
    }
#endif
}

}  // namespace d3tom

using namespace d3tom;

// How the cosine kernel takes a batch: rows of a tile / 64, slices of the contraction; mfma: whether it is the MFMA kernel at all.
namespace {
struct CosPlan { bool mfma; int TM, ksplit; };
CosPlan cos_plan(int B, int max_V, int max_keep, int max_pruned, int d_sim, int dt) {
    const bool mfma = (dt == D3TOM_BF16) && (d_sim % COS_BK == 0) && ((size_t)max_V * d_sim * 2 < ((size_t)1 << 31));
    int TM = 1, ksplit = 1;
    if (mfma && max_pruned > 0) {
        const int nct = ceil_div(max_keep, COS_BN);
        // as long as the 64-row tiles still fit one round of the 256 CUs they finish sooner than half as many
        // 128-row tiles (a 64-row tile's k-loop is ~0.7 of a 128-row tile's); several rounds of 128-row tiles are 256-row tiles, which
        // move a third less operand data per flop and whose rests the kernel cuts (against 128-row tiles, merges at d = 4096: 4500 rows keeping
        // 0.2 .. 0.5 70 -> 59 us, 5 samples of 2304 90 -> 76, 9 of 1152 .. 2304 114 -> 83).  From 16 samples on, where the bounds that the
        // host has are far above what the samples need, they are also better above half a round: 450 drawn batches of 16 to 100 samples of 90 to
        // 900 rows at d = 1024 .. 4096, merges and whole merge layers, 1.04 x at 1024, 1.05 at 2048, 1.09 at 4096, 0.93 at the least; below half a
        // round (435 batches) 0.99, at the least 0.84.  Above half a round 14 and 15 samples gain 1.01, 5 to 7 0.99, and some lose 10 %.
        const long t64 = (long)nct * ceil_div(max_pruned, 64) * B, t128 = (long)nct * ceil_div(max_pruned, 128) * B;
        TM = t128 > (B >= 16 ? 128 : 256) ? 4 : t64 > 256 ? 2 : 1;
        // too few 64 x 128 tiles for 256 CUs (short sequences): cut the contraction into k-slices as well
        if (TM == 1) {
            const int stages = d_sim / COS_BK;
            // How many slices: one more stage of the contraction costs a workgroup 0.19 us, one more slice of a tile 0.022 us, most of it in
            // the launch that adds them.  (Merges of 100 to 2500 rows at d = 1024, 2048 and 4096, 1 and 3 samples, with 2, 4, 8 and 16 slices
            // each: the choice is within 2 % of the best.  As many slices as 256 compute units hold, and 16 of them requested in any case:
            // 1024 rows keeping 0.1 at 4096 18.1 -> 16.3 us, keeping half 20.3 -> 19.8, at 1024 16.2 -> 15.0 and 18.6 -> 15.9; 1600 keeping half
            // at 4096 28.6 -> 26.6; 3 samples of 105 to 150 rows 18.5 -> 15.0.)
            double least = 0.0;
            for (int s = 2; t64 <= COS_SPLIT_BLOCKS / 2 && s <= COS_MAX_SLICES; s *= 2) {
                if (t64 * s > COS_SPLIT_BLOCKS || stages % s || stages / s < cos_ring_stages(1)) break;
                const double cost = (double)(stages / s) + 0.114 * (double)(t64 * s);
                if (s == 2 || cost < least) { least = cost; ksplit = s; }
            }
        }
    }
    return {mfma, TM, ksplit};
}
}  // namespace
bool d3tom::merge_takes_norms(int B, int max_V, int max_keep, int max_pruned, int d_sim, int dt) {
    const CosPlan p = cos_plan(B, max_V, max_keep, max_pruned, d_sim, dt);
    return max_pruned > 0 && p.ksplit == 1;
}

// Both entry points: norms + pruned list, cosine argmax, token -> slot table, scatter of one or two
// payloads that share the routing.
int d3tom::merge_run(const void* x0, void* y0, const void* x1, void* y1, const void* sim, int d, int d_sim, int dt,
                     int B, const int32_t* seq_off, const int32_t* vis_start, const int32_t* vis_count,
                     const int32_t* vis_off, const int32_t* kept_idx, const int32_t* kept_off,
                     int max_N, int max_V, int max_keep, int max_pruned, int max_out, int mode,
                     const int32_t* out_off, int32_t* assign, int32_t* counts, int32_t* src_pos,
                     void* ws, size_t ws_bytes, void* stream, bool prepared, int out_rows_hint) {
    if (!x0 || !y0 || !seq_off || !vis_start || !vis_count || !vis_off || !kept_idx || !kept_off || !out_off)
        return D3TOM_ERR_INVALID_ARG;
    if ((x1 == nullptr) != (y1 == nullptr)) return D3TOM_ERR_INVALID_ARG;
    if (B < 1 || d < 1 || max_N < 1 || max_V < 1 || max_V > max_N || max_keep < 1 || max_keep > max_V ||
        max_pruned < 0 || max_pruned > max_V || max_out < 1 || max_out > max_N)
        return D3TOM_ERR_INVALID_ARG;
    if (dt != D3TOM_F32 && dt != D3TOM_BF16) return D3TOM_ERR_INVALID_ARG;
    if (mode != D3TOM_MERGE_MEAN && mode != D3TOM_MERGE_SUM) return D3TOM_ERR_INVALID_ARG;
    const int epc = (dt == D3TOM_BF16) ? 8 : 4;
    if (!sim) { sim = x0; d_sim = d; }
    if (d_sim < 1) return D3TOM_ERR_INVALID_ARG;
    if ((d % epc) || (d_sim % epc)) return D3TOM_ERR_UNSUPPORTED;
    if (!aligned16(x0) || !aligned16(sim) || !aligned16(y0) || !aligned16(x1) || !aligned16(y1)) return D3TOM_ERR_INVALID_ARG;
    if (max_V > D3TOM_MAX_VISUAL) return D3TOM_ERR_UNSUPPORTED;
    const MergeWs w = merge_ws_layout(B, max_V);
    if (!ws) return D3TOM_ERR_INVALID_ARG;
    if (ws_bytes < w.total || (((uintptr_t)ws) & 255u)) return D3TOM_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t st = (hipStream_t)stream;
    char* wsb = (char*)ws;
    int32_t* pruned = (int32_t*)(wsb + w.pruned_off);
    float* rnorm = (float*)(wsb + w.rnorm_off);
    table_t* table = (table_t*)(wsb + w.table_off);

    static PerDeviceOnce lds_setup;
    if (!lds_setup.run([] {
            return raise_dynamic_lds(cos_argmax_bf16<1, 4, true>, cos_ring_stages(1) * (64 + 128) * 128) &&
                   raise_dynamic_lds(cos_argmax_bf16<1, 4, false>, cos_ring_stages(1) * (64 + 128) * 128) &&
                   raise_dynamic_lds(cos_argmax_bf16<1, 3, false>, cos_ring_stages(1) * (64 + 96) * 128) &&
                   raise_dynamic_lds(cos_argmax_bf16<2, 4, false>, cos_ring_stages(2) * (128 + 128) * 128) &&
                   raise_dynamic_lds(cos_argmax_bf16<2, 3, false>, cos_ring_stages(2) * (128 + 96) * 128) &&
                   raise_dynamic_lds(cos_argmax_bf16<4, 4, false>, cos_ring_stages(4) * (256 + 128) * 128) &&
                   // the norms of every kept slot: above 16376 of them more than 64 KB with the kernel's own array
                   raise_dynamic_lds(cos_reduce_argmax<4, 2>, D3TOM_MAX_VISUAL * (int)sizeof(float)) &&
                   raise_dynamic_lds(cos_reduce_argmax<4, 4>, D3TOM_MAX_VISUAL * (int)sizeof(float)) &&
                   raise_dynamic_lds(cos_reduce_argmax<4, 8>, D3TOM_MAX_VISUAL * (int)sizeof(float)) &&
                   raise_dynamic_lds(cos_reduce_argmax<4, 16>, D3TOM_MAX_VISUAL * (int)sizeof(float));
        }))
        return D3TOM_ERR_DEVICE;

    const CosPlan plan = cos_plan(B, max_V, max_keep, max_pruned, d_sim, dt);
    const bool mfma = plan.mfma;
    const int TM = plan.TM, ksplit = plan.ksplit;
    // prepared: the selection launch has left 1 / norm of every visual row (by token), the pruned list and the
    // initial table in the workspace; a split contraction computes the norms itself, and without that launch the list as well
    const dim3 gn(ceil_div(max_keep, 4), B);
    if (prepared || ksplit > 1) {
    } else if (dt == D3TOM_BF16)
        D3TOM_LAUNCH(MERGE_NORMS, st, merge_norms_kernel<uint16_t><<<gn, 256, 0, st>>>(
            (const uint16_t*)sim, d_sim, seq_off, vis_start, vis_count, kept_idx, kept_off, max_V, max_keep, rnorm, pruned,
            table, w.VP));
    else
        D3TOM_LAUNCH(MERGE_NORMS, st, merge_norms_kernel<float><<<gn, 256, 0, st>>>(
            (const float*)sim, d_sim, seq_off, vis_start, vis_count, kept_idx, kept_off, max_V, max_keep, rnorm, pruned,
            table, w.VP));

    if (mfma && max_pruned > 0) {
        int nct = ceil_div(max_keep, COS_BN);
        const int BM = TM * 64;
        const int nrt = ceil_div(max_pruned, BM);
        // one round of workgroups with CUs to spare: tiles of 96 slots, if they still fit one round, spread the loads over more CUs
        // (3280 x 365 rows: 156 tiles of 24 KB a stage or 208 of 20 KB, 22.6 -> 20.1 us; 2733 x 912: 28.5 -> 26.4)
        const int nct96 = ceil_div(max_keep, 96);
        const bool narrow = ksplit == 1 && TM < 4 && (long)nrt * nct96 * B <= 256;
        if (narrow) nct = nct96;
        // tiles of a sample in 8 equal runs (one per XCD); bands about as high as a run's block is wide.  256-row tiles: the tiles of all
        // samples in 8 equal runs of whole tiles and parts of tiles behind them (a rest of 8 tiles, 32 parts, has the most workgroups more than tiles).
        const int per = TM == 4 ? ceil_div(nrt * nct * B, 8) + 24 : ceil_div(nrt * nct, 8);
        int RB = 1;
        while ((RB + 1) * (RB + 1) <= (TM == 4 ? 32 : per)) ++RB;
        if (RB > nrt) RB = nrt;
        const int tiles_launch = 8 * per * (TM == 4 ? 1 : B);
        // Without a selection launch in front that has read the rows, they may come from HBM (key and value caches: one of each per layer,
        // written a step ago).  A CU takes in 48 bytes per ns from there, 95 from the memory-side cache, and its tile waits for
        // the slowest row; CUs that a single round of tiles leaves idle then request rows ahead of the tiles.  Rows cold:
        // 3645 rows keeping 365 38.9 -> 33.6 us, 729 48.7 -> 41.4, 1822 52.0 -> 49.9; rows cached: within 1 % (without the test of the
        // first answers 0 to 4 % lost).  Not where a helper would have more rows than the 128 it can request at a time: helping
        // with part of the rows gains nothing (5600 rows, 32 idle CUs: 0 % cold, 1 % lost cached).
        const int idle = 256 - tiles_launch;
        const bool help = !prepared && ksplit == 1 && TM < 4 && idle > 0 && (long)max_pruned * B <= (long)idle * 128;
        const dim3 g((unsigned)(help ? 256 : tiles_launch), (unsigned)ksplit);
        float* dots = (float*)(wsb + w.dots_off);
        float* sq = (float*)(wsb + w.sq_off);
        const size_t lds = (size_t)cos_ring_stages(TM) * (BM + (narrow ? 96 : COS_BN)) * 128;
#define D3TOM_COS(TMV, CBKV, SPLITV)                                                                                        \
    D3TOM_LAUNCH(COS_ARGMAX, st, (cos_argmax_bf16<TMV, CBKV, SPLITV><<<g, 512, lds, st>>>(                                     \
        (const uint16_t*)sim, d_sim, seq_off, vis_start, vis_count, kept_idx, kept_off, max_V, max_keep, pruned, rnorm, table, \
        w.VP, per, RB, ksplit, dots, nrt, nct, prepared ? 1 : 0, B, sq)))
        if (TM == 4) D3TOM_COS(4, 4, false);
        else if (TM == 2) { if (narrow) D3TOM_COS(2, 3, false); else D3TOM_COS(2, 4, false); }
        else if (ksplit > 1) D3TOM_COS(1, 4, true);
        else { if (narrow) D3TOM_COS(1, 3, false); else D3TOM_COS(1, 4, false); }
#undef D3TOM_COS
        if (ksplit > 1) {
            const int wpr = nct >= 3 ? 4 : nct;            // waves per pruned row: one column tile each, as far as four go
            const dim3 gr(ceil_div(max_pruned, 4 / wpr), B);
#define D3TOM_REDUCE(WPRV, SLICESV)                                                                                     \
    D3TOM_LAUNCH(COS_REDUCE, st, (cos_reduce_argmax<WPRV, SLICESV><<<gr, 256, (size_t)max_keep * sizeof(float), st>>>(  \
        seq_off, vis_start, vis_count, kept_off, max_V, max_keep, pruned, dots, nrt * nct * B, nrt, nct, table, w.VP, sq, B)))
#define D3TOM_REDUCE_OF(SLICESV)                                                                                        \
    do { if (wpr == 1) D3TOM_REDUCE(1, SLICESV); else if (wpr == 2) D3TOM_REDUCE(2, SLICESV); else D3TOM_REDUCE(4, SLICESV); } while (0)
            if (ksplit == 2) D3TOM_REDUCE_OF(2); else if (ksplit == 4) D3TOM_REDUCE_OF(4); else if (ksplit == 8) D3TOM_REDUCE_OF(8); else D3TOM_REDUCE_OF(16);
#undef D3TOM_REDUCE_OF
#undef D3TOM_REDUCE
        }
    } else if (max_pruned > 0) {
        const dim3 g(max_pruned, B);
        if (dt == D3TOM_BF16)
            D3TOM_LAUNCH(COS_ARGMAX, st, cos_argmax_generic<uint16_t><<<g, 256, 0, st>>>(
                (const uint16_t*)sim, d_sim, seq_off, vis_start, vis_count, kept_idx, kept_off, max_V, max_keep, pruned,
                rnorm, table, w.VP, prepared ? 1 : 0));
        else
            D3TOM_LAUNCH(COS_ARGMAX, st, cos_argmax_generic<float><<<g, 256, 0, st>>>(
                (const float*)sim, d_sim, seq_off, vis_start, vis_count, kept_idx, kept_off, max_V, max_keep, pruned,
                rnorm, table, w.VP, prepared ? 1 : 0));
    }

    // few output rows (short sequences): two workgroups per row, half a row each, so that more CUs stream
    const int nch = d / epc;
    // (max_out bounds the rows; when it is only a loose bound, the launch is sized for the caller's expected row count)
    const int rows_expected = (out_rows_hint > 0 && out_rows_hint < max_out) ? out_rows_hint : max_out;
    const int nslice = ((long)rows_expected * B * (x1 ? 2 : 1) < 768 && nch >= 512) ? 2 : 1;
    const dim3 gs(rows_expected * nslice, B, x1 ? 2 : 1);    // output rows (x slices) per sample x payloads
#define D3TOM_SCATTER(TYPE, CPT)                                                                                        \
    D3TOM_LAUNCH(MERGE_SCATTER, st, merge_scatter_kernel<TYPE, CPT><<<gs, 256, 0, st>>>(                                \
        (const TYPE*)x0, (const TYPE*)x1, d, seq_off, vis_start, vis_count, kept_idx, kept_off, max_V, max_keep,         \
        max_out, mode, out_off, table, w.VP, vis_off, (TYPE*)y0, (TYPE*)y1, assign, counts, src_pos))
    if (dt == D3TOM_BF16) { if (nslice == 2) D3TOM_SCATTER(uint16_t, 1); else D3TOM_SCATTER(uint16_t, 2); }
    else                  { if (nslice == 2) D3TOM_SCATTER(float, 1); else D3TOM_SCATTER(float, 2); }
#undef D3TOM_SCATTER
    return D3TOM_OK;
}

extern "C" int d3tom_merge(const void* x, const void* sim, int d, int d_sim, int dt,
                           int B, const int32_t* seq_off, const int32_t* vis_start, const int32_t* vis_count,
                           const int32_t* vis_off, const int32_t* kept_idx, const int32_t* kept_off,
                           int max_N, int max_V, int max_keep, int max_pruned, int max_out, int mode,
                           const int32_t* out_off, void* y, int32_t* assign, int32_t* counts, int32_t* src_pos,
                           void* ws, size_t ws_bytes, void* stream) {
    return merge_run(x, y, nullptr, nullptr, sim, d, d_sim, dt, B, seq_off, vis_start, vis_count, vis_off, kept_idx,
                     kept_off, max_N, max_V, max_keep, max_pruned, max_out, mode, out_off, assign, counts, src_pos, ws,
                     ws_bytes, stream);
}

extern "C" int d3tom_merge_kv(const void* k_cache, const void* v_cache, int d, int dt,
                              int B, const int32_t* seq_off, const int32_t* vis_start, const int32_t* vis_count,
                              const int32_t* vis_off, const int32_t* kept_idx, const int32_t* kept_off,
                              int max_N, int max_V, int max_keep, int max_pruned, int max_out, int mode,
                              const int32_t* out_off, void* k_out, void* v_out, int32_t* assign, int32_t* counts,
                              int32_t* src_pos, void* ws, size_t ws_bytes, void* stream) {
    if (!k_cache || !v_cache || !k_out || !v_out) return D3TOM_ERR_INVALID_ARG;
    return merge_run(k_cache, k_out, v_cache, v_out, k_cache, d, d, dt, B, seq_off, vis_start, vis_count, vis_off,
                     kept_idx, kept_off, max_N, max_V, max_keep, max_pruned, max_out, mode, out_off, assign, counts,
                     src_pos, ws, ws_bytes, stream);
}
