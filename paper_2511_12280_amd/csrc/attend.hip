// d3tom_attend: bidirectional (unmasked) attention over the shortened sequence (Section 3.2: the
// shortened tensor runs through the later layers; Section 4.3: the 2 n^2 d term of FLOPs_layer).
//
// bf16 path — flash-style, MFMA 16x16x32, written "transposed" so that everything per query stays
// inside one lane column:
//     S^T = K Q^T      A = K tile (LDS, row-major), B = Q^T (registers, loaded once per workgroup)
//     P^T = exp2(S^T * scale*log2e - m)            in registers, the MFMA accumulator layout
//     O^T += V^T P^T   A = V^T, read from the row-major V tile in LDS with the transposing LDS read
//                      (ds_read_b64_tr_b16), B = P^T straight from the accumulator registers of the
//                      first product (no LDS round trip for P)
// In the accumulator layout lane (r, g) = (lane % 16, lane / 16) owns query column r and, of every 16 keys, keys
// 4g .. 4g + 3, so the running max / sum of the online softmax need exchanges between four lanes only, and
// the rescale of O^T is a per-lane scalar.  The contraction index of the second product (keys) is
// fed in the order the accumulator holds it; V^T is read from LDS in that same order.
//
// A workgroup has eight waves of 32 or 16 queries in two groups of four; wave i and wave i + 4 share a SIMD.  The groups
// alternate (ping-pong): while one issues the MFMAs of a 64-key tile (S of tile i + 1, O += V P of tile i: 64 of them, 1024
// clocks), the other does the softmax arithmetic of its tile.  That pays because the smaller MFMA shape lets another wave's vector
// instructions through: per tile 1058 clocks of MFMAs and 756 of softmax arithmetic (an fma, an exp2 and half a conversion per logit) of
// the other wave take 1250 clocks together, whereas beside MFMA 32x32x16 the exponentials do not issue at all (1029 + 756 -> 1780).
//
// Bound by the port of the vector instructions, which both waves of a SIMD share.  An MFMA of 17.4 clocks keeps the other wave's from it for 9.6, the
// softmax arithmetic of a tile takes 740 (an exp2 or a conversion of a pair 8 clocks, others 4) and 190 more for each block of 16 queries whose
// maximum moves.  What costs more than its share is an instruction of that kind in an MFMA phase: it waits behind the exponentials of the
// other wave, and the MFMAs behind it wait as well.  And a barrier makes four SIMDs wait for the one with the most to rescale.  So
//   - the fragments' addresses move on in the softmax phase, and are few: K and V tiles lie in LDS in parts of 64 dims, whose k-steps and blocks differ
//     by constants that go into the instructions, so that six addresses serve a stage;
//   - the loads' addresses are constants, the way from tile to tile is in the buffer descriptors and done by the scalar unit in the MFMA phase;
//   - the exponentials are held inside the phase (the compiler put them behind its end, out of its priority and behind a wait for loads);
//   - both blocks' maxima are there before the first branch on one, and those of four lanes are plain v_max (fmaxf also quiets each operand);
//   - a tile has one barrier, in front of group 0's softmax phase and group 1's MFMA phase: inside a tile the waves of a SIMD find
//     their turns by themselves (groups that share their queries have a ring each and need a barrier in front of either).
// 32 heads of 128 (four independent waves on the larger shape; two barriers a tile and addresses moved among the MFMAs; now): 3773 keys 240, 208 and 200 us = 1.17
// PFLOP/s, 1951 keys 71, 61.8 and 58.7.
//
// K and V tiles go HBM/L2 -> LDS with direct loads (buffer_load ... lds, no register staging; rows past the end of the sample
// load as zeros through the buffer bounds check) into a ring; rows are unpadded and their 16-byte chunks XOR-swizzled by the
// row index instead.  Loads are issued in the softmax phase, and the first K fragments of a tile are read there, so that the
// MFMA phase starts at once.
//
// The softmax arithmetic paces the loop, so its wave has the higher priority (against none, and the MFMAs before it: 8 heads, 900 keys 11.0, 12.0, 12.9 us;
// several rounds the same), and it is cut to what the results need: per logit one fma, one exp2, one addition and the packing to bf16, and
//   - the weights and the tail mask of the weighted form enter as the C operand of S^T (log2 w / scale2, -inf);
//   - the running maximum costs one max3 per two logits: a lane compares its own logits with the column's maximum, and only where one
//     of them exceeds it do the four lanes meet and the accumulators of that block of 16 queries get their new scale.
// What the exponents refer to is a matter of precision.  The probabilities are rounded to bf16, the largest ones carry most of
// that rounding, and relative to the running maximum the largest is exactly 1 and not rounded at all.  With the first tile's
// maximum as a fixed reference the kernel is a tenth faster, but its error against float64 (2-norm, relative) is 2.33e-3, 2.23e-3 and 1.92e-3 at 3773 keys and logit
// spreads of 1, 2 and 4 instead of 2.27e-3, 1.92e-3 and 1.74e-3.
// The row sums are float32 sums of the unrounded probabilities, as in the short-sample kernel.  The sums of the rounded ones
// (a fragment of ones times P^T, 2 % faster) are as near to float64, but they move whole rows by the rounding of
// their probabilities, so that the two kernels give a merge other near-ties.
//
// The generic path (float32 or any head size) is one workgroup per query, or in float32 per two queries, and head, with a chunked
// online softmax in plain float arithmetic.
#include "common.hpp"
#include "direct_load.hpp"
#include "internal.hpp"
#include <type_traits>

namespace d3tom {

constexpr int ATT_BK = 64;      // keys per tile
constexpr int ATT_SLOTS = 4;    // ring slots of one K tile and one V tile
constexpr int ATT_TURNS_WGS = 32;       // workgroups per XCD that take several tiles in turn: one per compute unit

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short att_short4;

// 4 keys x 16 dims of a row-major LDS tile, transposed on the way to the registers: within each group
// of 16 lanes, lanes 4j..4j+3 point at 4 x 4 consecutive elements of row j, and lane i receives
// column i of that 4 x 16 block (ds_read_b64_tr_b16).
template <typename P>           // a generic pointer into LDS or one of its address space
__device__ __forceinline__ att_short4 lds_read_tr16(P p) {
    typedef __attribute__((address_space(3))) att_short4* lp;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)p);
}

#if defined(__HIP_DEVICE_COMPILE__)
// the larger of two values that are no signalling NaN (fmaxf: two instructions more, which quiet its operands)
__device__ __forceinline__ float att_max(uint32_t a, uint32_t b) {
    float m;
    asm("v_max_f32 %0, %1, %2" : "=v"(m) : "v"(a), "v"(b));
    return m;
}
// the two lanes (l, l ^ 32) that share a query column combine their values: after the swap of the upper
// half of one copy with the lower half of the other, the two results hold {own, partner} in some order
__device__ __forceinline__ float att_pair_max(float x) {
    typedef unsigned att_u2 __attribute__((ext_vector_type(2)));
    const att_u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return att_max(r[0], r[1]);
}
__device__ __forceinline__ float att_pair_sum(float x) {
    typedef unsigned att_u2 __attribute__((ext_vector_type(2)));
    const att_u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// the four lanes (l, l ^ 16, l ^ 32, l ^ 48) that share a query column
__device__ __forceinline__ float att_quad_max(float x) {
    typedef unsigned att_u2 __attribute__((ext_vector_type(2)));
    const att_u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return att_pair_max(att_max(r[0], r[1]));
}
__device__ __forceinline__ float att_quad_sum(float x) {
    typedef unsigned att_u2 __attribute__((ext_vector_type(2)));
    const att_u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return att_pair_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}
#endif

// Size-weighted attention: key row j of sample b stands for w_j original tokens (the member counts of the
// merge); its logit gets + log2(w_j) in the base-2 softmax, which is attention over the sequence with the row
// written w_j times.  The weights are described the way the merge reports them: `counts` per kept slot; key
// rows vis_start[b] .. vis_start[b] + (kept_off[b+1] - kept_off[b]) - 1 are the merged rows, every other row
// weighs 1.
struct KeyWeights {
    const int32_t* counts;
    const int32_t* kept_off;
    const int32_t* vis_start;
};
__device__ __forceinline__ float key_log2_weight(const KeyWeights& kw, int b, int j) {
    const int r = j - kw.vis_start[b];
    const int k0 = kw.kept_off[b], kn = kw.kept_off[b + 1] - k0;
    return (r >= 0 && r < kn) ? __log2f((float)max(kw.counts[k0 + r], 1)) : 0.f;
}
constexpr int ATT_WKEYS = 3584;     // longest sample of the weighted tiled kernel: its log2 weights sit in LDS beside the ring

// SKIP: waves without queries skip their products.  Not in a single round of 128-query tiles, where the skipping gains nothing and the
// second loop costs 1 to 3 % (900 keys, 16 heads of 64 13.2 us without it, 13.6 with it; 775 keys, 8 heads of 128 15.5 and 15.7).
//
// SPLIT: the groups share their queries (64 of them) and take the tiles of keys in turn, each in its own half of the ring; at the end
// each hands half of the channels of its O^T to the other through LDS.  A launch that leaves compute units idle is one chain of
// phases per unit, and this is half as long a chain on twice as many units: 8 heads of 128, 775 keys 15.8 -> 11.3 us, 2000 keys 33.4 -> 23.1,
// 16 heads of 64, 1024 keys 13.9 -> 9.4.  No part of a phase bounds it (without loads, exponentials, rescaling or reads of V it is 3 to 8 %
// faster each).
//
// UNEVEN: 192 queries, 32 to a wave of group 0 and 16 to one of group 1.  Where 256 queries fill three quarters of a round of an XCD's compute units or less, or 128 need
// another round.  A round takes 0.87 to 0.94 of the time that one of 256 queries takes, not 0.75 (32 heads, 1100 and 1500 keys 27.1 and 31.1 us, 39.7 and 42.5): group 1's fragments feed one
// MFMA each, and four waves that read 32 KB of them keep the LDS busy as long as group 0's MFMAs take.  The sums of a row are those of the other two, bit by bit.
template <int DH, bool WGT, int NQ, bool TURNS, bool SKIP, bool SPLIT, bool UNEVEN>
__global__ __launch_bounds__(512, 2) void attend_bf16_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int32_t* __restrict__ cu, int H, int nB, int nqt, float scale2, uint16_t* __restrict__ o, KeyWeights kw) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int KS = DH / 32;                 // k-steps of the first product
    constexpr int DB = DH / 16;                 // 16-dim blocks of O^T
    constexpr int ROWB = DH * 2;                // bytes per row of q, k, v and o
    constexpr int NCHK = DH / 8;                // 16-byte chunks per row
    constexpr int RPI = 64 / NCHK;              // rows of q or o covered by one wave-wide access (1 KB)
    constexpr int HALVES = DH / 64, PARTB = 128;        // K and V tiles lie in LDS in parts of 64 dims: 64 rows of 128 bytes, unpadded, chunks swizzled
    constexpr int PART = ATT_BK * PARTB;
    constexpr int LROWS = SPLIT ? 2 : 1;        // groups of 8 rows that a wave loads of each part, one direct load (1 KB) each
    constexpr int LD = LROWS * HALVES;          // direct loads per wave and operand tile
    constexpr int TILE = ATT_BK * ROWB;         // bytes of one K (or V) tile
    constexpr int STAGE = 2 * TILE;             // stage j: K of tile j, V of tile j - 1
    constexpr int NS = ATT_SLOTS;
    constexpr int AHEAD = SPLIT ? 2 : NS - 1;   // the softmax phase of tile j fetches stage j + AHEAD
    constexpr int BQ = UNEVEN ? 192 : NQ * (SPLIT ? 64 : 128);          // queries of the workgroup: NQ blocks of 16 per wave
    static_assert(!UNEVEN || (NQ == 2 && !SPLIT), "group 1 has half of group 0's queries");
    constexpr int KPRE = 2 * KS;                // K fragments read ahead: the first 32 keys
    typedef unsigned att_u4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) char ring[];
    __shared__ __attribute__((aligned(16))) float w_s[WGT ? ATT_WKEYS : 4];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), grp = wave >> 2;
    const int wq = SPLIT ? wave & 3 : wave;                // SPLIT: waves i and i + 4 have the same queries
    auto tile_of = [&](int j) { return SPLIT ? 2 * j + grp : j; };     // the j-th tile of keys of this wave's group
    auto slot_of = [&](int j) { return SPLIT ? (j & 1) * 2 + grp : j % NS; };
    const int r = lane & 15, g = lane >> 4;
    const size_t rs = (size_t)H * DH;                      // token stride (elements)
    const int row_bytes = (int)(rs * 2);

    // An item is a tile of BQ queries of one head.  XCD x has the heads hb = x, x + 8, ... of hb = (the sample's place) * H + head, the
    // tiles of a head one after the other.  One item per workgroup (places = samples as they come), or (TURNS) workgroup li of the W of
    // an XCD takes its items li, 2 W - 1 - li, 2 W + li, ..., in order of falling time.  Up to 32 samples may have two places, one for the last
    // tile if that leaves half of the waves without a query (0.72 of the others' time) and one for the other tiles: where the tiles fill
    // the rounds better with the short ones behind all others (48 heads, 1290 keys 71 -> 63 us, 40 heads, 1540 78 -> 75, 64 heads, 4098 527 -> 513; 3 x 650 at 32 heads 40.9 -> 39.8; some ragged
    // batches lose, 32 drawn samples of 1 .. 520 at 13 heads 30.6 -> 32.9: the estimate counts passes as equal, whatever the lengths of the samples in them).
    // Apart from its head's other tiles a short one does not find K and V in the XCD's L2: always behind the others, 6 x 800 keys take 87 instead of 78.
    const int xcd = blockIdx.x & 7, li = blockIdx.x >> 3;
    constexpr int W = ATT_TURNS_WGS;
    __shared__ int4 tab[TURNS ? WAVE : 1];                 // by place: first token, tokens, sample (its complement: the last tile only), tiles
    __shared__ int ends[TURNS ? WAVE : 1];                 // by place: items up to and with this one
    int tok0, n, h, b, qt;
    auto item = [&](int pass) {
        const int idx = pass * W + ((pass & 1) ? W - 1 - li : li);
        const int end = ends[TURNS ? lane : 0];
        const int place = __popcll(__builtin_amdgcn_ballot_w64(end <= idx));
        if (place >= WAVE) return false;
        const int rem = idx - (place ? __builtin_amdgcn_readlane(end, place - 1) : 0);
        const int4 e = tab[place];
        tok0 = __builtin_amdgcn_readfirstlane(e.x);
        n = __builtin_amdgcn_readfirstlane(e.y);
        const int smp = __builtin_amdgcn_readfirstlane(e.z), tiles = __builtin_amdgcn_readfirstlane(e.w);
        b = smp < 0 ? ~smp : smp;
        h = ((xcd - place * H) & 7) + 8 * (rem / tiles);
        qt = smp < 0 ? (n - 1) / BQ : rem % tiles;
        return true;
    };
    if constexpr (TURNS) {
        if (wave == 0) {
            const bool two = nB <= WAVE / 2, is_last = two && lane >= WAVE / 2;
            const int smp = two ? lane & (WAVE / 2 - 1) : lane;
            const int c0 = cu[min(smp, nB - 1)], c1 = cu[min(smp + 1, nB)];
            const int len = smp < nB ? max(min(c1 - c0, WGT ? ATT_WKEYS : 0x7FFFFFFF), 0) : 0;
            const int left = len % BQ, all = (len + BQ - 1) / BQ;
            int lone = !UNEVEN && two && left > 0 && left <= BQ / 2;
            {
                // passes over the XCD's units with the last tiles among the others, and with them behind all others, as if all samples were of one length
                const int sum = is_last ? 0 : all, sum_lone = is_last ? 0 : lone;
                const int P = __builtin_amdgcn_readlane(wave_incl_scan(sum), 63) * H / 8, S = __builtin_amdgcn_readlane(wave_incl_scan(sum_lone), 63) * H / 8;
                const int among = (P + W - 1) / W, full = (P - S + W - 1) / W, free = full * W - (P - S);
                const float t0 = (float)among * ((float)P - 0.28f * (float)S) / (float)max(P, 1);
                const float t1 = (float)full + 0.72f * (float)(S > free ? (S - free + W - 1) / W : 0);
                if (t1 > 0.99f * t0) lone = 0;
            }
            const int others = all - lone;
            const int mine = is_last ? lone : others;
            const float time = mine > 0 ? (float)len * (is_last ? 0.72f : 1.f) : -1.f;
            int rank = 0;
            for (uint64_t m = __builtin_amdgcn_ballot_w64(mine > 0); m; m &= m - 1) {
                const int j = __builtin_ctzll(m);
                const float other = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(time), j));
                rank += (other > time) || (other == time && j < lane);
            }
            tab[lane].w = 0;
            if (mine > 0) tab[rank] = make_int4(c0, len, is_last ? ~smp : smp, mine);
            asm volatile("" ::: "memory");                  // what follows reads what other lanes have written
            const int h0 = (xcd - lane * H) & 7;
            const int heads = h0 < H ? (H - h0 + 7) >> 3 : 0;
            ends[lane] = wave_incl_scan(heads * tab[lane].w);
        }
        __syncthreads();
        if (!item(0)) return;
    } else {
        const int hb = (li / nqt) * 8 + xcd;
        if (hb >= H * nB) return;
        h = hb % H; b = hb / H; qt = li % nqt;
        tok0 = cu[b];
        n = min(cu[b + 1] - tok0, WGT ? ATT_WKEYS : 0x7FFFFFFF);
        if (qt * BQ >= n) return;
    }
    // what the logits start from; -inf past the end of the sample: those keys then need no other mask
    constexpr int KROUND = SPLIT ? 2 * ATT_BK : ATT_BK;
    static_assert(ATT_WKEYS % KROUND == 0, "the weights of the last tiles fit");
    auto write_weights = [&] {
        for (int j = tid; j < ((n + KROUND - 1) / KROUND) * KROUND; j += 512)
            w_s[j] = (j < n) ? key_log2_weight(kw, b, j) / scale2 : -INFINITY;
    };
    if constexpr (WGT) write_weights();
    // this head's rows of this sample; a row index >= n is past the end and loads as zeros
    auto rows_of = [&](const uint16_t* p) {
        return make_uniform_rsrc(p + (size_t)tok0 * rs + (size_t)h * DH, (uint32_t)(((size_t)(n - 1) * rs + DH) * 2));
    };
    __amdgpu_buffer_rsrc_t rq = rows_of(q);
    // this head's first byte in q, k, v and o, and the bytes from there to its end in the sample's last row
    size_t head_at;
    uint32_t head_bytes;
    auto place_head = [&] { head_at = ((size_t)tok0 * rs + (size_t)h * DH) * 2; head_bytes = (uint32_t)(((size_t)(n - 1) * rs + DH) * 2); };
    place_head();

    auto first_query = [&] { return qt * BQ + (UNEVEN && grp ? 64 + wq * 16 : wq * NQ * 16); };
    int q0 = first_query();                     // this wave's first query
    bf16x8 qf[NQ][KS];
    f32x4 ot[DB][NQ];
    // m_run: running maximum of the RAW logits; ms: what the exponents subtract; l_run: this lane's part of the column's sum
    float m_run[NQ], ms[NQ], l_run[NQ];
    auto clear = [&] {
#pragma unroll
        for (int t = 0; t < DB; ++t)
#pragma unroll
            for (int qb = 0; qb < NQ; ++qb) ot[t][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) { m_run[qb] = -INFINITY; ms[qb] = 0.f; l_run[qb] = 0.f; }
    };
    clear();

    // direct loads: lane -> (row, chunk position).  The chunk fetched into position p of row x is p ^ f(x): K fragments are 16
    // consecutive rows of one chunk, transposing reads of V four consecutive rows (per 16 lanes) of one 32-byte piece.
    int k_off[LROWS], v_off[LROWS];             // byte offsets inside the head's K / V for key0 = 0; the second part of a row lies 128 bytes on
#pragma unroll
    for (int i = 0; i < LROWS; ++i) {
        const int x = (wq * LROWS + i) * 8 + (lane >> 3), pos = lane & 7;
        k_off[i] = x * row_bytes + ((pos ^ ((x >> 1) & 7)) << 4);
        v_off[i] = x * row_bytes + ((pos ^ (((x >> 1) & 3) << 1)) << 4);
    }
    const uint32_t ring0 = (uint32_t)(size_t)(lds_ptr_t)ring;
    const uint32_t wave_lds = ring0 + wq * LROWS * 1024;
    // The tiles of the next stage to be requested, as buffers that begin with them and end with the sample's rows (stage 0 has no V tile).
    __amdgpu_buffer_rsrc_t rk, rv;
    int tile_at;                                // of that stage's K tile: bytes behind the head's first one
    const int tile_step = (SPLIT ? 2 : 1) * ATT_BK * row_bytes;
    auto first_tile = [&] {
        tile_at = (SPLIT ? grp : 0) * ATT_BK * row_bytes;
        rk = make_uniform_rsrc((const char*)k + head_at + tile_at, (uint32_t)max((int)head_bytes - tile_at, 0));
        rv = make_uniform_rsrc((const char*)v + head_at, 0);
    };
    auto next_tile = [&] {
        rv = make_uniform_rsrc((const char*)v + head_at + tile_at, (uint32_t)max((int)head_bytes - tile_at, 0));
        tile_at += tile_step;
        rk = make_uniform_rsrc((const char*)k + head_at + tile_at, (uint32_t)max((int)head_bytes - tile_at, 0));
    };
    first_tile();
    auto issue_one = [&](int j, int i) {        // one of the 2 LD loads of stage j
        const int u = i >> 1, row = u / HALVES, half = u % HALVES;
        const uint32_t dst = wave_lds + slot_of(j) * STAGE + half * PART + row * 1024 + (i & 1) * TILE;
        if (half) direct_load_16<128>((i & 1) ? rv : rk, ((i & 1) ? v_off : k_off)[row], dst);
        else direct_load_16((i & 1) ? rv : rk, ((i & 1) ? v_off : k_off)[row], dst);
    };
    auto issue = [&](int j) {
#pragma unroll
        for (int i = 0; i < 2 * LD; ++i) issue_one(j, i);
        next_tile();
    };
    // LDS addresses of the fragments in the stage that the next MFMA phase reads: two k-steps of K, four blocks of V; the others lie in the next part
    // of the tile.  V's move on in the softmax phase, K's, which are wanted at its start, at the end of the MFMA phase.
    constexpr int KA = 2, VA = 4;
    uint32_t ka[KA], va[VA];
    auto first_addresses = [&] {
        // the lane's number anew, so that nothing of this is kept in a register from one item to the next
        int l = threadIdx.x;
        asm volatile("" : "+v"(l));
        l &= 63;
        const int lr = l & 15, lg = l >> 4;
        const int k0 = lr * PARTB + ((lg ^ ((lr >> 1) & 7)) << 4);               // rows 0..15, chunk 4 ks + g
        // transposing read: row 4 g + tj, 4-dim quad tq of a 16-dim block; the block number goes in by exclusive or (32-byte pieces)
        const int tj = lr >> 2, tq = l & 3, tx = 4 * lg + tj;
        const int v0 = TILE + tx * PARTB + (((tq >> 1) ^ (((tx >> 1) & 3) << 1)) << 4) + (tq & 1) * 8;
        const uint32_t base = ring0 + slot_of(0) * STAGE;
#pragma unroll
        for (int i = 0; i < KA; ++i) ka[i] = base + (k0 ^ (i << 6));
#pragma unroll
        for (int i = 0; i < VA; ++i) va[i] = base + (v0 ^ (i << 5));
    };
    auto step_to = [&](int j) { return (uint32_t)__builtin_amdgcn_readfirstlane((slot_of(j) - slot_of(j - 1)) * STAGE); };     // from stage j - 1 to j
    auto move = [](uint32_t& a, uint32_t step) { asm volatile("v_add_u32 %0, %1, %0" : "+v"(a) : "s"(step)); };
    typedef __attribute__((address_space(3))) const char* lds_bytes_t;
    auto k_fragment = [&](int ks, int kb) {
        typedef __attribute__((address_space(3))) const bf16x8* lp;
        return *(lp)((lds_bytes_t)(size_t)ka[ks % KA] + ks / KA * PART + kb * 16 * PARTB);
    };

    bf16x8 kf[KPRE];                            // the first 32 keys' fragments of the next tile
    auto read_first = [&](int f) { kf[f] = k_fragment(f / 2, f % 2); };
    f32x4 st[4][NQ];                            // S^T: [16-key block][query block]
    bf16x8 pf[2][NQ];                           // P^T: [32-key half][query block]
    // S of tile j (QK) and O += V P of tile j - 1 (PV).  A wave that issues LDS reads back to back waits for the CU's one LDS at each
    // of them while the matrix core idles; every fragment of what comes next is therefore read right behind the MFMAs that used
    // up the registers it goes into (a bunch of reads in front of each part: 1710 clocks per phase; dealt: 1350).
    static_assert(KPRE == DB, "a V fragment follows every K fragment");
    uint32_t step = 0;                          // from the stage of the last MFMA phase to the next one
    auto mfma_phase = [&](int j, auto qk_c, auto pv_c, auto blocks) {
        constexpr int NB = decltype(blocks)::value;         // query blocks of this wave: NQ, or (UNEVEN, group 1) one
        constexpr bool QK = decltype(qk_c)::value, PV = decltype(pv_c)::value;
        typedef __attribute__((__vector_size__(8 * sizeof(short)))) short att_short8;
        att_short8 vf[DB];                      // V^T of 32 keys, 16 dims each
        auto read_v = [&](int kt, int t) {
            const lds_bytes_t p = (lds_bytes_t)(size_t)va[t % VA] + t / VA * PART + kt * 32 * PARTB;
            vf[t] = __builtin_shufflevector(lds_read_tr16(p), lds_read_tr16(p + 16 * PARTB), 0, 1, 2, 3, 4, 5, 6, 7);
        };
        auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
        fence();
        if constexpr (QK) {
            f32x4 c0[4];                        // what S^T starts from, per 16-key block
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) {
                if constexpr (WGT) c0[kb] = *reinterpret_cast<const f32x4*>(&w_s[tile_of(j) * ATT_BK + kb * 16 + g * 4]);
                else c0[kb] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int i = 0; i < 2 * KPRE; ++i) {
                const int f = i % KPRE, ks = f / 2, kb = (i / KPRE) * 2 + f % 2;
#pragma unroll
                for (int qb = 0; qb < NB; ++qb)
                    st[kb][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[f], qf[qb][ks], ks ? st[kb][qb] : c0[kb], 0, 0, 0);
                fence();
                if (PV && i == KPRE) next_tile();
                if (i == KPRE) step = step_to(j + 1);
                if (i < KPRE) kf[f] = k_fragment(ks, kb + 2);
                else if constexpr (PV) read_v(0, f);
                fence();
            }
        } else {
#pragma unroll
            for (int t = 0; t < DB; ++t) read_v(0, t);
        }
        if constexpr (PV) {
#pragma unroll
            for (int i = 0; i < 2 * DB; ++i) {
                const int kt = i / DB, t = i % DB;
#pragma unroll
                for (int qb = 0; qb < NB; ++qb)
                    ot[t][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[t]), pf[kt][qb], ot[t][qb], 0, 0, 0);
                fence();
                if (kt == 0) read_v(1, t);
                fence();
            }
        }
        fence();
        if constexpr (QK) {
#pragma unroll
            for (int i = 0; i < KA; ++i) move(ka[i], step);
        }
    };
    auto softmax_phase = [&](int j, auto last_c, auto blocks) {
        constexpr int NB = decltype(blocks)::value;
        constexpr bool LAST = decltype(last_c)::value;
        if (LAST && !WGT && (tile_of(j) + 1) * ATT_BK > n) {
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int qb = 0; qb < NB; ++qb)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (tile_of(j) * ATT_BK + kb * 16 + g * 4 + e >= n) st[kb][qb][e] = -INFINITY;
        }
        // The first fragments of tile j + 1 and the loads of stage j + AHEAD in turns, in front of the arithmetic (clocks per tile and
        // pair of groups, measured without maximum and sums: so 2960, reads first and then loads 3190, spread among the exponentials 3420).
        // SPLIT, with twice as many loads in a phase: half of them behind the maximum (64 to 500 keys 2 % faster).
        constexpr int LATER = SPLIT ? LD : 0;
        if constexpr (!LAST) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
#pragma unroll
                for (int f = i * KPRE / 8; f < (i + 1) * KPRE / 8; ++f) read_first(f);
#pragma unroll
                for (int f = i * (2 * LD - LATER) / 8; f < (i + 1) * (2 * LD - LATER) / 8; ++f) issue_one(j + AHEAD, f);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int i = 0; i < VA; ++i) move(va[i], step);
        // The running maximum.  A lane sees its own 16 of a column's 64 logits; only if one of them exceeds the column's maximum do
        // the four lanes meet and the accumulators get their new scale.
        float peak[NB];
        uint64_t above[NB];
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) {
            peak[qb] = m_run[qb];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int e = 0; e < 4; ++e) peak[qb] = fmaxf(peak[qb], st[kb][qb][e]);
            above[qb] = __builtin_amdgcn_ballot_w64(peak[qb] > m_run[qb]);
        }
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) {
            if (above[qb] != 0) {
                const float m_new = att_quad_max(peak[qb]);    // finite: every tile holds at least one key of the sample
                const float alpha = __builtin_amdgcn_exp2f((m_run[qb] - m_new) * scale2);
                ms[qb] = m_new * scale2;
                m_run[qb] = m_new;
                l_run[qb] *= alpha;
#pragma unroll
                for (int x = 0; x < DB; ++x)
#pragma unroll
                    for (int e = 0; e < 4; ++e) ot[x][qb][e] *= alpha;
            }
        }
        if constexpr (!LAST && LATER > 0) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 2 * LD - LATER; f < 2 * LD; ++f) issue_one(j + AHEAD, f);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int qb = 0; qb < NB; ++qb)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                {
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(st[kb][qb][e], scale2, -ms[qb]));
                    pf[kb >> 1][qb][(kb & 1) * 4 + e] = (__bf16)p;
                    l_run[qb] += p;
                }
        // (all of it here, not behind what ends the phase)
#pragma unroll
        for (int qb = 0; qb < NB; ++qb) asm volatile("" : "+v"(pf[0][qb]), "+v"(pf[1][qb]), "+v"(l_run[qb]));
    };

    int ntile = (n + KROUND - 1) / KROUND;      // tiles of a group (SPLIT: the last one may lie past the end in part or, of group 1, in full)
    // The queries go through the ring's last two slots, each wave's rows in its own part: whole lines, and in flight together with
    // the first tiles.  Every wave has read them when stage 2 is started.
    constexpr int QROWS = NQ * 16, QLD = QROWS / RPI;
    auto row_swizzle = [](int x) { return DH == 128 ? (x & 15) : ((x >> 1) & 7); };
    if constexpr (SPLIT) {
        // (Half of the rows of a pair of waves from each of them, in the place of the V tile that stage 0 has not.)
        constexpr int HROWS = QROWS / 2;
        static_assert(4 * HROWS * ROWB <= TILE && HROWS % RPI == 0, "the queries fit beside the first tile");
        const int q_lds = TILE + wq * HROWS * ROWB;
#pragma unroll
        for (int i = 0; i < HROWS / RPI; ++i) {
            const int x = grp * HROWS + i * RPI + lane / NCHK;
            direct_load_16(rq, (q0 + x) * row_bytes + (((lane % NCHK) ^ row_swizzle(x)) << 4), ring0 + grp * STAGE + q_lds + i * 1024);
        }
#pragma unroll
        for (int i = 0; i < 2 * LD; i += 2) issue_one(0, i);
        next_tile();
        issue(1);
        wait_loads<2 * LD>();
        if constexpr (WGT) __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0): the weights are written
        phase_barrier();
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int x = qb * 16 + r;
                qf[qb][ks] = *reinterpret_cast<const bf16x8*>(ring + (x / HROWS) * STAGE + q_lds + (x % HROWS) * ROWB + (((ks * 4 + g) ^ row_swizzle(x)) << 4));
            }
        __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0): read before the other group loads into their place
    } else {
        static_assert(8 * QROWS * ROWB <= 2 * STAGE, "the queries fit into two slots");
        const int q_lds = 2 * STAGE + wave * QROWS * ROWB;
#pragma unroll
        for (int i = 0; i < QLD; ++i) {
            const int x = i * RPI + lane / NCHK;
            direct_load_16(rq, (q0 + x) * row_bytes + (((lane % NCHK) ^ row_swizzle(x)) << 4), ring0 + q_lds + i * 1024);
        }
        issue(0);
        issue(1);
        wait_loads<2 * LD>();
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) qf[qb][ks] = *reinterpret_cast<const bf16x8*>(ring + q_lds + (qb * 16 + r) * ROWB + (((ks * 4 + g) ^ row_swizzle(r)) << 4));
        __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0): the queries are there (and the weights written)
        phase_barrier();
    }
    static_assert(SPLIT || AHEAD == 3, "three stages are under way when the loop starts");
    using yes = std::integral_constant<bool, true>;
    using no = std::integral_constant<bool, false>;
    constexpr int KEEP = SPLIT ? 0 : (NS - 3) * 2 * LD;
    bool first = true;
    // all tiles of keys; LIVE = false for a wave whose queries all lie past the end of the sample, which only requests its part of the
    // tiles and keeps step: in a last tile of at most 128 queries a SIMD has one wave to serve instead of two, in others the card has
    // less to do.  (Last tiles computed in full before: 16 samples of 614 .. 1536 keys 346 -> 332 us, 64 of 300 .. 1000 at 8
    // heads 166 -> 155, 12 of 270 .. 800 84.6 -> 82.3, one of 1951 61.4 -> 60.5, of 3700 203 -> 201; 8 of 1000, 232 queries in the last, 133.)
    auto sweep = [&](auto live_c, auto blocks) {
        constexpr bool LIVE = decltype(live_c)::value;
        if constexpr (!SPLIT) issue(2);
        if constexpr (LIVE) {
            first_addresses();
#pragma unroll
            for (int f = 0; f < KPRE; ++f) read_first(f);
        }
        // Stage j + 1 has to have landed when the softmax phase of tile j begins (its first fragments are read there), and stage j - 1, whose slot the
        // loads of that phase fill, has to have been read.  Groups that share the ring: both wait for their loads before the one barrier of tile j, which ends
        // group 0's MFMA phase of tile j and group 1's softmax phase of tile j - 1.  Stages behind j + 1 stay in flight.  SPLIT: a group has a ring of two slots of its own, and stage j + 1, requested in the softmax phase of tile j - 1,
        // is all that is on its way; the group waits for it before the barrier that ends its own MFMA phase of tile j.
        if (grp == 1) { if (!SPLIT && first) wait_loads<KEEP>(); phase_barrier(); }
        bool wait0 = SPLIT || (grp == 0 && first);         // (behind another item the first two stages have landed, and its stores may still be on their way)
        if constexpr (LIVE) mfma_phase(0, yes(), no(), blocks);
        // The last tile is peeled off: a loop left in its middle keeps both the accumulators before and after the MFMA phase alive.
        // (The weighted form with heads of 128 gets its trip count in a scalar register by force: the compiler counted in a vector register and
        // branched on vcc, 0.5 % of single rounds of 128-query tiles.  The others are 0.2 to 0.5 % faster as they are.)
        constexpr bool COUNTED = WGT && DH == 128;
        const int last = COUNTED ? __builtin_amdgcn_readfirstlane(ntile - 1) : 0;
#pragma unroll 1
        for (int j = 0; COUNTED ? j < last : j + 1 < ntile; ++j) {
            if (wait0) wait_loads<KEEP>();
            wait0 = SPLIT || grp == 0;
            if (SPLIT || grp == 0) phase_barrier();
            if constexpr (LIVE) {
                __builtin_amdgcn_s_setprio(2);
                softmax_phase(j, no(), blocks);
                __builtin_amdgcn_s_setprio(0);
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0): the fragments are there (a wait the compiler knows of)
            } else {
                issue(j + AHEAD);
            }
            if (!SPLIT && grp == 1) wait_loads<KEEP>();
            if (SPLIT || grp == 1) phase_barrier();
            if constexpr (LIVE) mfma_phase(j + 1, yes(), yes(), blocks);
        }
        if (SPLIT || grp == 0) { wait_loads<0>(); phase_barrier(); }
        if constexpr (LIVE) softmax_phase(ntile - 1, yes(), blocks);
        if (grp == 1) wait_loads<0>();
        if (SPLIT || grp == 1) phase_barrier();
        if constexpr (LIVE) mfma_phase(ntile, no(), yes(), blocks);
    };
    // SPLIT: the two parts of the keys meet.  A wave gives the channels that it does not finish to the wave with the same queries (group 0
    // finishes the first half of them), takes that wave's part of its own, and stores its half rows through LDS.
    auto join_groups = [&](auto grp_c) {
        constexpr int HALF = DB / 2, KEPT = decltype(grp_c)::value * HALF, GIVEN = HALF - KEPT;
        constexpr int XCH = NQ * HALF * 1024, HROWB = ROWB / 2, HCHK = NCHK / 2;
        static_assert(!SPLIT || 8 * (XCH + NQ * 128 + QROWS * HROWB) <= NS * STAGE, "what is exchanged, the sums and the rows fit into the ring");
        f32x4* mine = reinterpret_cast<f32x4*>(ring + wave * XCH);
        const f32x4* theirs = reinterpret_cast<const f32x4*>(ring + (wave ^ 4) * XCH);
        float* sums = reinterpret_cast<float*>(ring + 8 * XCH);         // [wave][query block]: maximum of 16 queries, sum of 16 queries
        char* rows = ring + 8 * (XCH + NQ * 128) + wave * QROWS * HROWB;
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) {
            l_run[qb] = att_quad_sum(l_run[qb]);
            if (g == 0) { sums[(wave * NQ + qb) * 32 + r] = m_run[qb]; sums[(wave * NQ + qb) * 32 + 16 + r] = l_run[qb]; }
#pragma unroll
            for (int t = 0; t < HALF; ++t) mine[(qb * HALF + t) * 64 + lane] = ot[GIVEN + t][qb];
        }
        wait_lds();
        phase_barrier();
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) {
            const float m1 = sums[((wave ^ 4) * NQ + qb) * 32 + r], l1 = sums[((wave ^ 4) * NQ + qb) * 32 + 16 + r];
            const float m = fmaxf(m_run[qb], m1);
            const float f0 = __builtin_amdgcn_exp2f((m_run[qb] - m) * scale2), f1 = __builtin_amdgcn_exp2f((m1 - m) * scale2);    // 0 for a part without keys
            const float inv = 1.0f / (l_run[qb] * f0 + l1 * f1);
#pragma unroll
            for (int t = 0; t < HALF; ++t) {
                const f32x4 a = ot[KEPT + t][qb], c = theirs[(qb * HALF + t) * 64 + lane];
                uint2 w;
                w.x = pack_bf16x2((a[0] * f0 + c[0] * f1) * inv, (a[1] * f0 + c[1] * f1) * inv);
                w.y = pack_bf16x2((a[2] * f0 + c[2] * f1) * inv, (a[3] * f0 + c[3] * f1) * inv);
                *reinterpret_cast<uint2*>(rows + (qb * 16 + r) * HROWB + (((t * 2 + (g >> 1)) ^ (r & (HCHK - 1))) << 4) + (g & 1) * 8) = w;
            }
        }
        wait_lds();
        const __amdgpu_buffer_rsrc_t ro = rows_of(o);
#pragma unroll
        for (int i = 0; i < QROWS * HCHK / 64; ++i) {
            const int x = i * (64 / HCHK) + lane / HCHK;
            const uint4 w = *reinterpret_cast<const uint4*>(rows + x * HROWB + (((lane % HCHK) ^ (x & (HCHK - 1))) << 4));
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(att_u4, w), ro, (q0 + x) * row_bytes + KEPT * 32 + (lane % HCHK) * 16, 0, 0);
        }
    };
    for (int pass = 1;; ++pass) {
        using all = std::integral_constant<int, NQ>;
        using one = std::integral_constant<int, 1>;
        if (SKIP && q0 >= n) sweep(no(), all());
        else if (UNEVEN && grp == 1) sweep(yes(), one());
        else sweep(yes(), all());
        wait_loads<0>();                        // nothing may be in flight into LDS when the workgroup ends
        if (grp == 0) phase_barrier();
        if constexpr (SPLIT) {
            phase_barrier();                    // everybody is done with the ring
            if (grp == 0) join_groups(std::integral_constant<int, 0>()); else join_groups(std::integral_constant<int, 1>());
            break;
        }

        // O^T lies in the registers as 4 dims of a row per lane; through LDS the rows are stored in whole lines.  Slot ntile % NS may
        // still be read by group 1 (V of its last tile); the two behind the next one are free.
        const __amdgpu_buffer_rsrc_t ro = rows_of(o);
        // the lane's number anew, so that no address of this part is kept in a register through the loop above
        int el = threadIdx.x;
        asm volatile("" : "+v"(el));
        el &= 63;
        const int er = el & 15, eg = el >> 4;
        const int o0 = q0;
        int slot = (ntile + 2 + grp) % NS;
        bool more = false;
        if constexpr (TURNS) {
            // The next item's first stages and queries are requested in front of this one's epilogue.  (The next workgroup on a CU
            // starts 2 us after the one before has ended, and waits another 2.8 .. 4.5 us for its first loads.)
            const int before = b;
            more = item(pass);
            if (more) {
                phase_barrier();                // everybody is done with the ring and the weights
                rq = rows_of(q);
                place_head();
                first_tile();
                q0 = first_query();
                ntile = (n + ATT_BK - 1) / ATT_BK;
                issue(0);
                issue(1);
                slot = 2 + grp;
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
                        qf[qb][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rq, (q0 + qb * 16 + er) * row_bytes + ks * 64 + eg * 16, 0, 0));
                if constexpr (WGT) { if (b != before) write_weights(); }
            }
        }
        char* ow = ring + slot * STAGE + (wave & 3) * QROWS * ROWB;
        static_assert(4 * QROWS * ROWB <= STAGE, "a group's rows fit into a slot");
        const int blocks = UNEVEN && grp == 1 ? 1 : NQ;
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) {
            if (qb >= blocks) break;
            const float inv = 1.0f / att_quad_sum(l_run[qb]);
#pragma unroll
            for (int t = 0; t < DB; ++t) {
                uint2 w;
                w.x = pack_bf16x2(ot[t][qb][0] * inv, ot[t][qb][1] * inv);
                w.y = pack_bf16x2(ot[t][qb][2] * inv, ot[t][qb][3] * inv);
                *reinterpret_cast<uint2*>(ow + (qb * 16 + er) * ROWB + (((t * 2 + (eg >> 1)) ^ row_swizzle(er)) << 4) + (eg & 1) * 8) = w;
            }
        }
        wait_lds();
#pragma unroll
        for (int i = 0; i < QLD; ++i) {
            if (i * RPI >= blocks * 16) break;
            const int x = i * RPI + el / NCHK;
            const uint4 w = *reinterpret_cast<const uint4*>(ow + x * ROWB + (((el % NCHK) ^ row_swizzle(x)) << 4));
            // rows past the end of the sample lie outside the buffer and are not written
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(att_u4, w), ro, (o0 + x) * row_bytes + (el % NCHK) * 16, 0, 0);
        }
        if (!more) break;
        clear();
        first = false;
        wait_loads<UNEVEN ? QLD / 2 : QLD>();   // all loads have landed; the stores (UNEVEN: of group 1, half as many) may be on their way
        __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0): the rows are out of the slots, the weights are written
        phase_barrier();
    }
#endif
}
// ---- short sequences: the keys are split across four waves -------------------------------------
// With a few hundred keys the kernel above is one short serial chain per workgroup (8 stages at 493 keys)
// on half of the CUs.  Here a workgroup owns 32 or 64 queries (QH halves of 32) of one head.  The waves of a half take the 32-key
// tiles w, w + 4, w + 8, ... with the same transposed products as above, and at the end the four partial results
// (running max, sum, O^T) of a half meet in LDS, rows of queries, from where eight threads to a row store whole lines.  A step is four tiles, one for
// each wave of a half.  K and V go to LDS by direct loads, the queries in front of them take the same way.  With one half nobody else reads a
// wave's tiles, and each has one place: K of the next step is requested behind the first product, V in front of the second one, and two workgroups of heads of 128 (four
// of 64) fit on a unit, which hide each other's waits.  The waves of two halves share their tile, load half of it each and meet at one barrier a step, with a second place for
// the step ahead.
// Bound by the chain of trips to memory where workgroups are few (the sample's offsets; queries and tiles: 1080 and some 2500 clocks), and by what a
// compute unit takes in where they are many, four times the K and V per query of the kernel above with 32 queries, twice with 64.
// With 32 queries, against two places for a wave's tiles, one workgroup to a unit with heads of 128, and 64 queries wherever 32 need more than a round (the same
// bits): 32 heads of 128, 16 x 8 rows 7.1 -> 4.6 us, 8 x 65 9.4 -> 7.8, 9 x 100 13.0 -> 11.0, one sample of 100 rows 4.2 -> 4.1, of 200 5.4 -> 5.2, of 300 7.6 -> 7.4; 8 heads of 128, one of 512
// 7.15 -> 6.3, 9 x 200 11.7 -> 6.8; 32 heads of 64, 16 x 21 .. 65 8.3 -> 5.5; 887 calls of up to 512 tiles of 128 queries 1.066 in the mean.
constexpr int ATS_BK = 32;      // keys per wave tile
constexpr int ATS_MAX_KEYS = 512;

template <int DH, int QH> struct AtsLds {
    static constexpr int ROWB = DH * 2, TILE = ATS_BK * ROWB, REGION = 2 * TILE, BUF = 4 * REGION;     // a wave's K and V tile; four of them a step
    static constexpr int PITCH = DH + 4;                                                                // floats of a row of a partial O
    static constexpr int BUFS = QH == 1 ? 1 : 2;                                                        // steps with a place of their own
    static constexpr int STEPS = BUFS * BUF + QH * 32 * ROWB, PARTS = 4 * QH * 32 * PITCH * 4;
    static constexpr int BYTES = STEPS > PARTS ? STEPS : PARTS;
};
template <int DH, bool WGT, int QH>
__global__ __launch_bounds__(256 * QH, 2) void attend_bf16_short_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const int32_t* __restrict__ cu, int H, int nB, int nqt, float scale2, uint16_t* __restrict__ o, KeyWeights kw) {
#if defined(__HIP_DEVICE_COMPILE__)
    using C = AtsLds<DH, QH>;
    constexpr int KS = DH / 16;
    constexpr int DT = DH / 32;
    constexpr int ROWB = C::ROWB, TILE = C::TILE;
    constexpr int NCHK = DH / 8;
    constexpr int RPI = 64 / NCHK;              // rows per wave-wide direct load
    constexpr int LD = ATS_BK / RPI / QH;       // direct loads per wave and operand tile
    constexpr int QLD = 32 / RPI / 4;           // of the queries
    constexpr bool ALONE = QH == 1;             // nobody else reads or loads a wave's tiles
    extern __shared__ __attribute__((aligned(16))) char ring[];
    __shared__ float part_m[4 * QH][32], part_l[4 * QH][32];
    __shared__ __attribute__((aligned(16))) float lw_s[WGT ? ATS_MAX_KEYS : 4];

    const int xcd = blockIdx.x & 7, li = blockIdx.x >> 3;
    const int hb = (li / nqt) * 8 + xcd, qt = li % nqt;
    if (hb >= H * nB) return;
    const int h = hb % H, b = hb / H;
    const int tok0 = cu[b];
    const int n = min(cu[b + 1] - tok0, ATS_MAX_KEYS);
    const int q0 = qt * 32 * QH;
    if (q0 >= n) return;

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int kg = wave & 3, qh = wave >> 2;               // which tiles of keys, which half of the queries
    const int c = lane & 31, g = lane >> 5;
    const size_t rs = (size_t)H * DH;
    const int row_bytes = (int)(rs * 2);
    const size_t head = (size_t)tok0 * rs + (size_t)h * DH;
    const uint32_t span = (uint32_t)(((size_t)(n - 1) * rs + DH) * 2);      // rows past the end load as zeros
    const __amdgpu_buffer_rsrc_t rq = make_uniform_rsrc(q + head, span), rk = make_uniform_rsrc(k + head, span), rv = make_uniform_rsrc(v + head, span);

    // direct loads: same chunk swizzles as in the kernel above
    const int ld_pos = lane % NCHK, ld_row = lane / NCHK;
    const uint32_t ring0 = (uint32_t)(size_t)(lds_ptr_t)ring;
    constexpr int Q_LDS = C::BUFS * C::BUF;
#pragma unroll
    for (int i = 0; i < QLD; ++i) {
        const int x = wave * QLD * RPI + i * RPI + ld_row;
        direct_load_16(rq, (q0 + x) * row_bytes + (((ld_pos ^ (x & 15)) & (NCHK - 1)) << 4), ring0 + Q_LDS + (wave * QLD + i) * 1024);
    }
    int k_off[LD], v_off[LD];
#pragma unroll
    for (int i = 0; i < LD; ++i) {
        const int r = (qh * LD + i) * RPI + ld_row;
        k_off[i] = (kg * ATS_BK + r) * row_bytes + (((ld_pos ^ (r & 15)) & (NCHK - 1)) << 4);
        v_off[i] = (kg * ATS_BK + r) * row_bytes + (((ld_pos ^ ((r & 3) * 4)) & (NCHK - 1)) << 4);
    }
    auto place = [&](int step) { return (C::BUFS == 2 ? (step & 1) * C::BUF : 0) + kg * C::REGION; };
    auto issue_k = [&](int step) {
#pragma unroll
        for (int i = 0; i < LD; ++i) direct_load_16(rk, k_off[i] + step * 4 * ATS_BK * row_bytes, ring0 + place(step) + (qh * LD + i) * 1024);
    };
    auto issue_v = [&](int step) {
#pragma unroll
        for (int i = 0; i < LD; ++i) direct_load_16(rv, v_off[i] + step * 4 * ATS_BK * row_bytes, ring0 + place(step) + TILE + (qh * LD + i) * 1024);
    };
    auto issue = [&](int step) { issue_k(step); issue_v(step); };
    const int ntile = (n + ATS_BK - 1) / ATS_BK, nstep = (ntile + 3) / 4;
    issue(0);
    if constexpr (WGT)
        for (int j = tid; j < ATS_MAX_KEYS; j += 256 * QH) lw_s[j] = (j < n) ? key_log2_weight(kw, b, j) : 0.f;

    int k_addr[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) k_addr[kk] = c * ROWB + ((((kk * 2 + g) ^ (c & 15)) & (NCHK - 1)) << 4);
    const int tr_j = (lane & 15) >> 2, tr_t = lane & 3, tr_half = (lane >> 4) & 1;
    int v_addr[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) {
        const int chunk = t * 4 + tr_half * 2 + (tr_t >> 1);
        v_addr[t] = TILE + (g * 4 + tr_j) * ROWB + (tr_t % 2) * 8 + (((chunk ^ (tr_j * 4)) & (NCHK - 1)) << 4);
    }
    f32x16 ot[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) ot[t][e] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    bf16x8 qf[KS];
    const bool live = q0 + qh * 32 < n;         // uniform
    for (int step = 0; step < nstep; ++step) {
        // This step's tiles (and the queries, the weights) are there.  ALONE: behind the first step a wave waits for nobody; otherwise
        // everybody is done with the step before, whose place the next one's tiles take.
        if (ALONE && step > 0) wait_loads<0>();
        else wait_loads_and_barrier<0>();
        const bool more = step + 1 < nstep;
        if (step == 0) {
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(ring + Q_LDS + qh * TILE + k_addr[kk]);
        }
        if (step * 4 + kg >= ntile || !live) {
            if (!ALONE && more) issue(step + 1);            // (ALONE: no tile, no later one)
            continue;
        }
        const int key0 = (step * 4 + kg) * ATS_BK;
        const char* wreg = ring + place(step);
        bf16x8 kf[KS];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) kf[kk] = *reinterpret_cast<const bf16x8*>(wreg + k_addr[kk]);
        __builtin_amdgcn_sched_barrier(0);
        f32x16 st;
#pragma unroll
        for (int e = 0; e < 16; ++e) st[e] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) st = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], st, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (more) { if (ALONE) issue_k(step + 1); else issue(step + 1); }        // (ALONE: the products above have taken the K fragments)
        __builtin_amdgcn_sched_barrier(0);
        att_short4 vf[2][DT][2];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                const char* pa = wreg + v_addr[t] + hh * 16 * ROWB;
                vf[hh][t][0] = lds_read_tr16(pa);
                vf[hh][t][1] = lds_read_tr16(pa + 8 * ROWB);
            }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (WGT) {
            // weighted: maximum and exponent on scale2 * logit + log2 w (m_run lives in that scaled domain)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                const f32x4 w4 = *reinterpret_cast<const f32x4*>(&lw_s[min(key0 + e4 * 8 + g * 4, ATS_MAX_KEYS - 4)]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int key = key0 + e4 * 8 + g * 4 + e;
                    const float t = __builtin_fmaf(st[e4 * 4 + e], scale2, w4[e]);
                    st[e4 * 4 + e] = (key < n) ? t : -INFINITY;
                }
            }
        } else if (key0 + ATS_BK > n) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int key = key0 + (e >> 2) * 8 + g * 4 + (e & 3);
                if (key >= n) st[e] = -INFINITY;
            }
        }
        float tmax = st[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) tmax = fmaxf(tmax, st[e]);
        tmax = att_pair_max(tmax);
        const float m_new = fmaxf(m_run, tmax);                // finite: every tile holds >= 1 valid key
        const float ms = m_new * scale2;
        float psum = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float p = __builtin_amdgcn_exp2f(WGT ? st[e] - m_new : __builtin_fmaf(st[e], scale2, -ms));
            st[e] = p;
            psum += p;
        }
        if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {
            const float alpha = __builtin_amdgcn_exp2f(WGT ? m_run - m_new : (m_run - m_new) * scale2);
            l_run *= alpha;
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) ot[t][e] *= alpha;
        }
        l_run += psum;
        m_run = m_new;
        __builtin_amdgcn_sched_barrier(0);
        if (ALONE && more) {
            __builtin_amdgcn_s_waitcnt(0xC07F);             // lgkmcnt(0): the V fragments are in registers
            issue_v(step + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            bf16x8 pf;
#pragma unroll
            for (int j = 0; j < 8; ++j) pf[j] = (__bf16)st[hh * 8 + j];
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                typedef __attribute__((__vector_size__(8 * sizeof(short)))) short att_short8;
                const att_short8 v8 = __builtin_shufflevector(vf[hh][t][0], vf[hh][t][1], 0, 1, 2, 3, 4, 5, 6, 7);
                ot[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v8), pf, ot[t], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // the four partial results of a half meet in LDS, rows of queries
    __syncthreads();                            // everybody is done with the tiles
    float* part = reinterpret_cast<float*>(ring);
    if (live) {
        l_run = att_pair_sum(l_run);
        float* mine = part + (wave * 32 + c) * C::PITCH + g * 4;
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4)
                *reinterpret_cast<f32x4*>(mine + t * 32 + e4 * 8) = f32x4{ot[t][e4 * 4], ot[t][e4 * 4 + 1], ot[t][e4 * 4 + 2], ot[t][e4 * 4 + 3]};
        if (g == 0) { part_m[wave][c] = m_run; part_l[wave][c] = l_run; }
    }
    __syncthreads();
    // eight threads to a row, an eighth of its channels each
    constexpr int CH = DH / 8;
    const int row = tid >> 3, w0 = (row >> 5) * 4, x = row & 31, ch = (tid & 7) * CH;
    if (q0 + row >= n) return;
    float m = part_m[w0][x];
#pragma unroll
    for (int w2 = 1; w2 < 4; ++w2) m = fmaxf(m, part_m[w0 + w2][x]);
    float f[4], l = 0.f;
#pragma unroll
    for (int w2 = 0; w2 < 4; ++w2) {
        const float mw = part_m[w0 + w2][x];
        f[w2] = (mw == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((mw - m) * (WGT ? 1.0f : scale2));
        l += part_l[w0 + w2][x] * f[w2];
    }
    const float inv = 1.0f / l;
    uint16_t* op = o + (size_t)(tok0 + q0 + row) * rs + (size_t)h * DH + ch;
#pragma unroll
    for (int e8 = 0; e8 < CH; e8 += 8) {
        float acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) {
            const f32x4* p = reinterpret_cast<const f32x4*>(part + ((w0 + w2) * 32 + x) * C::PITCH + ch + e8);
            const f32x4 lo = p[0], hi = p[1];
#pragma unroll
            for (int e = 0; e < 4; ++e) { acc[e] += lo[e] * f[w2]; acc[4 + e] += hi[e] * f[w2]; }
        }
        uint4 w;
        w.x = pack_bf16x2(acc[0] * inv, acc[1] * inv);
        w.y = pack_bf16x2(acc[2] * inv, acc[3] * inv);
        w.z = pack_bf16x2(acc[4] * inv, acc[5] * inv);
        w.w = pack_bf16x2(acc[6] * inv, acc[7] * inv);
        *reinterpret_cast<uint4*>(op + e8) = w;
    }
#endif
}

// generic: one workgroup per (Q queries, head), keys in chunks of 256, plain float online softmax.  A wave forms the logits of 64 keys, 16 lanes
// to a key; for the output a thread takes one 16-byte chunk of the channels and every G-th key (G = 256 / chunks), and the
// G partial rows meet in LDS at the end.  The first values are requested with the keys.  (A single row of dh threads walking all keys is one
// chain of n dependent loads: 8.1 us at 100 keys, launch included; split over the groups, a key to a thread 5.8 us; now 5.0.)
template <typename T, int Q>                   // Q: queries of a workgroup
__global__ __launch_bounds__(256) void attend_generic_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, const int32_t* __restrict__ cu,
    int H, int dh, float scale2, T* __restrict__ o, KeyWeights kw) {
    constexpr int EPC = 16 / sizeof(T);
    const int i0 = blockIdx.x * Q, h = blockIdx.y, b = blockIdx.z;
    const int tok0 = cu[b];
    const int n = cu[b + 1] - tok0;
    if (i0 >= n) return;
    __shared__ float ps[Q][256];
    __shared__ float red[Q][8];
    __shared__ float part[256][EPC + 1];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const size_t rs = (size_t)H * dh;
    const T* qr[Q];
#pragma unroll
    for (int x = 0; x < Q; ++x) qr[x] = q + (size_t)(tok0 + min(i0 + x, n - 1)) * rs + (size_t)h * dh;
    const int nch = dh / EPC, G = 256 / nch;
    const int grp = tid / nch, ch = tid - grp * nch;           // threads beyond G * nch take no keys
    float m_run[Q], l_run[Q], acc[Q][EPC];
#pragma unroll
    for (int x = 0; x < Q; ++x) {
        m_run[x] = -INFINITY; l_run[x] = 0.f;
#pragma unroll
        for (int e = 0; e < EPC; ++e) acc[x][e] = 0.f;
    }
    for (int j0 = 0; j0 < n; j0 += 256) {
        const int cnt = (grp < G) ? min(256, n - j0) : 0;
        const T* vr = v + (size_t)(tok0 + j0) * rs + (size_t)h * dh + ch * EPC;
        uint4 w[8];
        auto values = [&](int t0) {
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u] = *reinterpret_cast<const uint4*>(vr + (size_t)min(t0 + u * G, max(cnt - 1, 0)) * rs);
        };
        values(grp);                               // before the logits, whose keys arrive with them
        const int first = j0 + wave * 64, j = first + wave_dots_row(lane);
        float s2[Q];
#pragma unroll
        for (int x = 0; x < Q; ++x) s2[x] = -INFINITY;
        if (first < n) {
            float dot[Q];
            wave_row_dots<T, Q>(qr, k + (size_t)(tok0 + first) * rs + (size_t)h * dh, rs, n - first, dh, lane, dot);
            if (j < n) {
                const float weight = kw.counts ? key_log2_weight(kw, b, j) : 0.f;
#pragma unroll
                for (int x = 0; x < Q; ++x) s2[x] = kw.counts ? dot[x] * scale2 + weight : dot[x] * scale2;
            }
        }
#pragma unroll
        for (int x = 0; x < Q; ++x) {
            const float wm = wave_max(s2[x]);
            if (lane == 0) red[x][wave] = wm;
        }
        __syncthreads();
        float alpha[Q];
#pragma unroll
        for (int x = 0; x < Q; ++x) {
            const float cmax = fmaxf(fmaxf(red[x][0], red[x][1]), fmaxf(red[x][2], red[x][3]));
            const float m_new = fmaxf(m_run[x], cmax);
            alpha[x] = exp2f(m_run[x] - m_new);
            const float p = (j < n) ? exp2f(s2[x] - m_new) : 0.f;
            ps[x][wave * 64 + wave_dots_row(lane)] = p;
            const float wsum = wave_sum(p);
            if (lane == 0) red[x][4 + wave] = wsum;
            m_run[x] = m_new;
        }
        __syncthreads();
#pragma unroll
        for (int x = 0; x < Q; ++x) {
            l_run[x] = l_run[x] * alpha[x] + (red[x][4] + red[x][5] + red[x][6] + red[x][7]);
#pragma unroll
            for (int e = 0; e < EPC; ++e) acc[x][e] *= alpha[x];
        }
        for (int t0 = grp; t0 < cnt; t0 += 8 * G) {
            if (t0 != grp) values(t0);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (t0 + u * G >= cnt) break;
                const uint32_t ww[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
#pragma unroll
                for (int x = 0; x < Q; ++x) {
                    const float pt = ps[x][t0 + u * G];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (sizeof(T) == 2) {
                            acc[x][2 * e] += pt * bf16_lo(ww[e]); acc[x][2 * e + 1] += pt * bf16_hi(ww[e]);
                        } else {
                            acc[x][e] += pt * __uint_as_float(ww[e]);
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int x = 0; x < Q; ++x) {
        if (x) __syncthreads();
#pragma unroll
        for (int e = 0; e < EPC; ++e) part[tid][e] = acc[x][e];
        __syncthreads();
        if (tid < dh && i0 + x < n) {
            const int c0 = tid / EPC, e = tid - c0 * EPC;
            float sum = 0.f;
            for (int g = 0; g < G; ++g) sum += part[g * nch + c0][e];      // groups in ascending order
            Elem<T>::store(o + (size_t)(tok0 + i0 + x) * rs + (size_t)h * dh + tid, sum / l_run[x]);
        }
    }
}

}  // namespace d3tom

using namespace d3tom;

// Which kernel takes a call, and how many queries a workgroup of it has.
namespace {
enum { ATT_GENERIC = 0, ATT_SHORT = 1, ATT_TILES = 2 };
struct AttendPlan {
    int kernel, queries;                // of a workgroup
    int nqt;                            // such tiles of the longest sample
    bool turns, skip;                   // ATT_TILES: a workgroup takes several tiles in turn; waves without queries skip their products
    size_t lds;                         // dynamic
};
// whole: without the 64-query tiles (the blocks of a stack in front of its merge), see attend_whole_run
AttendPlan attend_plan(int dt, int B, int max_seqlen, int H, int dh, bool whole) {
    AttendPlan p{ATT_GENERIC, 1, max_seqlen, false, false, 0};
    // the tiled kernel addresses one sample's K / V rows with 32-bit byte offsets
    const bool fits32 = ((size_t)max_seqlen + 8 * ATT_BK) * (size_t)H * (size_t)dh * 2 < ((size_t)1 << 31);
    const long heads = (long)H * B;
    if (dt != D3TOM_BF16 || (dh != 128 && dh != 64) || !fits32) {
        // float32 is bound by reading each query its keys and values.  With two queries to a workgroup a round of workgroups reads half of that, but two
        // fit on a unit for three, and the round takes up to 1.3 times as long: taken where it saves enough rounds.  (One query and two; 4 heads of 64:
        // 160 rows 6.1 and 6.5 us, 200 rows 8.6 and 6.8, 300 rows 13.4 and 15.6, 400 rows 21.2 and 19.3, 700 rows 46.9 and 42.1; 16 heads of 64, 100 rows
        // 9.6 and 9.6, 300 rows 42.7 and 40.8; 8 heads of 36, 200 rows 11.2 and 11.6; 4 heads of 256, 200 rows 20.9 and 13.8.)
        const long one = (max_seqlen * heads + 767) / 768, two = (ceil_div(max_seqlen, 2) * heads + 511) / 512;
        if (dt == D3TOM_F32 && 13 * two < 10 * one) { p.queries = 2; p.nqt = ceil_div(max_seqlen, 2); }
        return p;
    }
    // Short samples, up to two rounds of 128-query tiles: keys split across the waves.  The tiles below are faster for some of them (493 keys, 32 heads of
    // 128 10.1 us here, 8.5 with 64-query tiles), but this kernel has four running maxima a row, over tiles of 32 keys, relative to which the probabilities are rounded.  Error against
    // float64 (2-norm, relative, output rounded to bf16) at logit spreads of 1 and 2, 493 keys: 2.10e-3, 1.77e-3 here; 2.16e-3, 1.82e-3 with 64-query
    // tiles; 2.19e-3, 1.86e-3 with wider ones.  66 to 512 keys, weighted or not, heads of 64 and 128: 2.2 to 4.9 % more with any of the tiles.
    if (max_seqlen <= ATS_MAX_KEYS && ceil_div(max_seqlen, 128) * heads <= 512) {
        // 32 queries to a workgroup, of which two with heads of 128 and four with heads of 64 fit on a unit, and 64 only for one sample of more than 256 keys whose
        // tiles fill the rounds of an XCD's units, one or two workgroups to each, by nine tenths: there they read half of the K and V that 32 queries read.
        // (32 and 64; one sample at 32 heads of 128, 200 rows 5.2 and 6.3 us, 300 7.4 and 7.6, 512 9.9 and 9.4; 8 heads of 128, 9 x 200 rows 6.8 and 11.7, 9 x 75 .. 200 6.5
        // and 8.8; 32 heads of 128, 16 x 8 rows 4.6 and 7.1, 8 x 30 .. 65 5.6 and 8.9; 32 heads of 64, 16 x 21 .. 65 5.5 and 8.4.  Over 880 single samples the choice is
        // 0.997 of the better one's speed.  Batches, of which the host knows the longest sample only, lose most where they are of one length that fills the rounds,
        // 8 x 512 rows at 8 heads of 128 17.7 and 17.5, weighted 20.1 and 19.1, 32 heads of 64, 4 x 256 7.1 and 6.8; 4 x 106 .. 256 6.3 and 6.7.)
        const int tiles = ceil_div(H, 8) * ceil_div(max_seqlen, 64), round = dh == 64 ? 64 : 32;
        p.queries = B == 1 && max_seqlen > 256 && 10 * tiles >= 9 * round * ceil_div(tiles, round) ? 64 : 32;
        p.kernel = ATT_SHORT;
        p.nqt = ceil_div(max_seqlen, p.queries);
        p.lds = dh == 128 ? (p.queries == 64 ? AtsLds<128, 2>::BYTES : AtsLds<128, 1>::BYTES) : (p.queries == 64 ? AtsLds<64, 2>::BYTES : AtsLds<64, 1>::BYTES);
        return p;
    }
    // 64-query tiles whose groups share the keys, where they fill one round of compute units at most: half as long a chain as 128-query
    // tiles on twice as many units, and two running maxima a row instead of one (error against float64 0.98 of theirs).  Two workgroups of heads of
    // 64 fit on a unit, and of ragged batches fewer tiles are real than the longest
    // sample lets the host expect.  Means over 697 drawn calls (1 to 16 samples of 513 to 2400 keys), the other widths' choice against this, by the
    // number of 64-query tiles: heads of 128, up to 128 tiles 1.37, 129 to 256 1.25 (0.81 where an XCD has more than 32 of them), 257 to 384 0.82; heads of 64, up to 256 tiles
    // 1.32, 257 to 512 0.98, 513 to 640 1.05, 641 to 768 0.97.
    // whole: the blocks of a stack in front of its merge do without these tiles, see attend_whole_run.
    const bool split = !whole && max_seqlen > ATS_MAX_KEYS && ceil_div(max_seqlen, 64) * heads <= (dh == 64 ? 640 : 256);
    // Rounds: an XCD has the tiles of an eighth of the heads and 32 compute units.  (Counted over the whole card, one sample at 12 heads of 128, 3227 keys, took 17 tiles of
    // 192 queries for each head, of which four XCDs have two heads: 145 us, with 256 queries 91; 28 heads, 1710 keys 77 and 51; 20 heads of 64, 2687 keys 83 with
    // 256, 54 with 128.)
    // With heads of 128 a round of 128-query tiles costs 0.63 to 0.72 of one of 256-query tiles (every fragment read from LDS feeds one MFMA instead of two), one of
    // 192 queries 0.87 to 0.94; with heads of 64 two workgroups of 128 queries share a CU, and a round of half of them costs 0.52.  (128, 192 and 256 queries; 32 heads of 128:
    // 1024 keys 19.8, 24.1 and 27.6 us, 1100 39.7, 27.1 and 31.1, 1500 52.0, 39.7 and 42.5, 1600 54.0, 72.2 and 43.5, 2060 94.5, 93.8 and 94.9, 2400 117.6, 107.1 and 123.7, 3000 153.5,
    // 139.2 and 154.2, 3773 240, 240 and 200, 4500 354, 298 and 338; weighted, 1100 42.8, 29.7 and 32.8; 16 heads, 2200 70.6, 48.0 and 53.2.)  Last 128-query tiles that
    // leave half of the waves without a query are items of their own behind the others (see the kernel) and count for less where the others leave room for most of them: 40 heads, 1538 keys 65.1,
    // 71.9 and 71.2, 1566 69.3, 71.9 and 74.2, 48 heads, 1282 57.0, 63.0 and 61.3; with no or little room 24 heads, 2690 117, 115 and 130, 56 heads, 1182 59.7, 56.9 and 67.1.
    // That holds for one sample (of 541 at 4 to 64 heads of 128 and 379 of 64 the choice is 0.9995 and 0.9998 of the best one's speed; counted over the card 0.964 and 0.986).  Of a batch the host
    // knows the longest sample only.  192 queries are for what is one round of them on every XCD whatever the others' lengths are (all tiles run side by side, the longest sample's
    // decide; 2 x 700 28.3, 21.6 and 22.5); for 128 or 256 its rounds are those of the card: where the longest sample's length makes a round of 128 overfull on some XCDs, the others' often
    // does not (12 heads, 834, 738 and 350 keys 15.9, 21.3 and 23.5; over 800 drawn batches by XCD 1.096 times as fast as with 128 and 256 by card alone, but 0.81 at
    // the least, so 1.093 and 0.98).  A batch with heads of 64 takes 128-query tiles always: its samples may all but one be shorter than the bound, and neither the rounds nor the bound say
    // by how much.  6028 drawn batches (2 to 48 samples, the longest of 170 to 8000 keys, the others as long, or from a half, a third or an
    // eighth of it on, 8 to 32 heads): 0.993 of the better width's speed, 0.75 at the least; by rounds, as for one sample, 0.955 and 0.58.  Where
    // the rounds speak for 256 queries, wide against narrow in the mean: samples of one length 0.95 to 1.01, ragged ones 0.71 to 1.02 (above
    // 1.00 from 13 rounds on).
    const int per_xcd = ceil_div(H * B, 8);
    auto rounds_of = [](long tiles) { return (tiles + 31) / 32; };
    auto rounds = [&](int queries) { return rounds_of((long)per_xcd * ceil_div(max_seqlen, queries)); };
    auto rounds_for = [&](int queries) { return B == 1 ? rounds(queries) : (ceil_div(max_seqlen, queries) * heads + 255) / 256; };
    // in hundredths of a round of 256-query tiles
    const long wide = 100 * rounds_for(256), mid = 90 * rounds(192);
    long narrow = (dh == 128 ? 66 : 55) * rounds_for(128);
    const int left = max_seqlen % 128;
    if (dh == 128 && B == 1 && left > 0 && left <= 64) {
        // last tiles that find no place in the rounds of the others
        const long full = (long)per_xcd * (max_seqlen / 128), r = rounds_of(full), behind = max(per_xcd - (r * 32 - full), 0L);
        if (2 * behind <= per_xcd) narrow = 66 * r + 47 * rounds_of(behind);
    }
    const bool small = (dh == 64 && B > 1) || narrow < wide;
    const bool uneven = dh == 128 && (B == 1 || rounds(192) == 1) && mid < (small ? narrow : wide);
    p.kernel = ATT_TILES;
    p.queries = split ? 64 : uneven ? 192 : small ? 128 : 256;
    p.nqt = ceil_div(max_seqlen, p.queries);
    p.lds = (size_t)ATT_SLOTS * 2 * ATT_BK * dh * 2;
    // Several rounds of workgroups that have a compute unit to themselves: one per unit, which takes its tiles in turn, samples by
    // falling length (one tile per workgroup / in turn, 32 heads of 128: 16 x 700 .. 1505 keys 386 / 375 us, 4 x 575 .. 1951 126 / 119, 12 x 270 .. 800
    // 103 / 82, 8 x 1000 140.5 / 138.7, one sample of 3773 206 / 206; 8 heads, 64 x 300 .. 1000 179 / 156; one sample in tiles of 192 queries 0.98, 2400 keys 108.6 / 110.7).
    p.turns = !split && p.nqt * heads > 256 && !(dh == 64 && p.queries == 128) && B <= WAVE;
    p.skip = p.nqt * heads > (dh == 64 ? 512 : 256);                   // more than one round (two workgroups of 128 queries with heads of 64 to a unit)
    return p;
}
}  // namespace

static int attend_any(const void* q, const void* k, const void* v, int dt, int B, const int32_t* cu_seqlens, int max_seqlen, int H, int dh,
                      float scale, const int32_t* counts, const int32_t* kept_off, const int32_t* vis_start, void* o, void* stream, bool whole = false) {
    if (!q || !k || !v || !o || !cu_seqlens) return D3TOM_ERR_INVALID_ARG;
    if (B < 1 || max_seqlen < 1 || H < 1 || dh < 1) return D3TOM_ERR_INVALID_ARG;
    if (!(scale > 0.f) || !(scale < 3.0e38f)) return D3TOM_ERR_INVALID_ARG;      // the running max is taken on raw logits
    if (dt != D3TOM_F32 && dt != D3TOM_BF16) return D3TOM_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return D3TOM_ERR_INVALID_ARG;
    if (dh > 256 || (dt == D3TOM_BF16 ? (dh % 8) : (dh % 4))) return D3TOM_ERR_UNSUPPORTED;
    const bool wgt = counts != nullptr;
    const KeyWeights kw{counts, kept_off, vis_start};
    hipStream_t st = (hipStream_t)stream;
    const float scale2 = scale * LOG2E;
    const AttendPlan p = attend_plan(dt, B, max_seqlen, H, dh, whole);
    // the weighted MFMA kernels keep a sample's weights in LDS
    if (wgt && p.kernel != ATT_GENERIC && max_seqlen > ATT_WKEYS) return D3TOM_ERR_UNSUPPORTED;
    const int nqt = p.nqt;
    const dim3 g(p.turns ? 8u * ATT_TURNS_WGS : 8u * (unsigned)ceil_div(H * B, 8) * (unsigned)nqt);
    if (p.kernel == ATT_SHORT) {
#define D3TOM_ATT_SHORT(DHV, WGTV, QHV)                                                                                         \
    do {                                                                                                                        \
        static PerDeviceOnce lds_setup;                                                                                         \
        if (!lds_setup.run([] { return raise_dynamic_lds(attend_bf16_short_kernel<DHV, WGTV, QHV>, AtsLds<DHV, QHV>::BYTES); })) return D3TOM_ERR_DEVICE; \
        D3TOM_LAUNCH(ATTEND, st, (attend_bf16_short_kernel<DHV, WGTV, QHV><<<g, 256 * QHV, p.lds, st>>>((const uint16_t*)q, (const uint16_t*)k, \
                                                               (const uint16_t*)v, cu_seqlens, H, B, nqt, scale2, (uint16_t*)o, kw))); \
    } while (0)
#define D3TOM_ATT_SHORT2(DHV, WGTV) do { if (p.queries == 32) D3TOM_ATT_SHORT(DHV, WGTV, 1); else D3TOM_ATT_SHORT(DHV, WGTV, 2); } while (0)
        if (dh == 128) { if (wgt) D3TOM_ATT_SHORT2(128, true); else D3TOM_ATT_SHORT2(128, false); }
        else           { if (wgt) D3TOM_ATT_SHORT2(64, true);  else D3TOM_ATT_SHORT2(64, false); }
#undef D3TOM_ATT_SHORT2
#undef D3TOM_ATT_SHORT
    } else if (p.kernel == ATT_TILES) {
#define D3TOM_ATT(KERNEL)                                                                                            \
    D3TOM_LAUNCH(ATTEND, st, (KERNEL<<<g, 512, p.lds, st>>>((const uint16_t*)q, (const uint16_t*)k, (const uint16_t*)v, \
                                                           cu_seqlens, H, B, nqt, scale2, (uint16_t*)o, kw)))
#define D3TOM_ATT8(DHV, WGTV, NQV, TURNSV, SKIPV, SPLITV, UNEVENV)                                                           \
    do {                                                                                                                    \
        static PerDeviceOnce lds_setup;                                                                                     \
        if (!lds_setup.run([] { return raise_dynamic_lds(attend_bf16_kernel<DHV, WGTV, NQV, TURNSV, SKIPV, SPLITV, UNEVENV>, ATT_SLOTS * 2 * ATT_BK * DHV * 2); })) \
            return D3TOM_ERR_DEVICE;                                                                                        \
        D3TOM_ATT((attend_bf16_kernel<DHV, WGTV, NQV, TURNSV, SKIPV, SPLITV, UNEVENV>));                                                     \
    } while (0)
#define D3TOM_ATT8_2(DHV, WGTV) do { if (p.turns) D3TOM_ATT8(DHV, WGTV, 2, true, true, false, false); else D3TOM_ATT8(DHV, WGTV, 2, false, true, false, false); } while (0)
#define D3TOM_ATT8_1(DHV, WGTV) do { if (p.skip) D3TOM_ATT8(DHV, WGTV, 1, false, true, false, false); else D3TOM_ATT8(DHV, WGTV, 1, false, false, false, false); } while (0)
#define D3TOM_ATT8_U(WGTV) do { if (p.turns) D3TOM_ATT8(128, WGTV, 2, true, true, false, true); else D3TOM_ATT8(128, WGTV, 2, false, false, false, true); } while (0)
#define D3TOM_ATT8_128(WGTV) do { if (p.queries == 192) D3TOM_ATT8_U(WGTV); else if (p.queries == 256) D3TOM_ATT8_2(128, WGTV); else if (p.turns) D3TOM_ATT8(128, WGTV, 1, true, true, false, false); else D3TOM_ATT8_1(128, WGTV); } while (0)
#define D3TOM_ATT8_64(WGTV) do { if (p.queries == 256) D3TOM_ATT8_2(64, WGTV); else D3TOM_ATT8_1(64, WGTV); } while (0)
        if (p.queries == 64) {
            if (dh == 128) { if (wgt) D3TOM_ATT8(128, true, 1, false, false, true, false); else D3TOM_ATT8(128, false, 1, false, false, true, false); }
            else           { if (wgt) D3TOM_ATT8(64, true, 1, false, false, true, false);  else D3TOM_ATT8(64, false, 1, false, false, true, false); }
        } else if (dh == 128) { if (wgt) D3TOM_ATT8_128(true); else D3TOM_ATT8_128(false); }
        else           { if (wgt) D3TOM_ATT8_64(true);  else D3TOM_ATT8_64(false); }
#undef D3TOM_ATT8_64
#undef D3TOM_ATT8_128
#undef D3TOM_ATT8_U
#undef D3TOM_ATT8_1
#undef D3TOM_ATT8_2
#undef D3TOM_ATT8
#undef D3TOM_ATT
    } else {
#define D3TOM_ATT_GENERIC(T, Q)                                                                                             \
    D3TOM_LAUNCH(ATTEND, st, (attend_generic_kernel<T, Q><<<dim3(nqt, H, B), 256, 0, st>>>(             \
        (const T*)q, (const T*)k, (const T*)v, cu_seqlens, H, dh, scale2, (T*)o, kw)))
        if (dt == D3TOM_F32) { if (p.queries == 2) D3TOM_ATT_GENERIC(float, 2); else D3TOM_ATT_GENERIC(float, 1); }
        else D3TOM_ATT_GENERIC(uint16_t, 1);
#undef D3TOM_ATT_GENERIC
    }
    return D3TOM_OK;
}

int d3tom::attend_whole_run(const void* q, const void* k, const void* v, int B, const int32_t* cu_seqlens, int max_seqlen, int H, int dh, float scale,
                            void* o, void* stream) {
    return attend_any(q, k, v, D3TOM_BF16, B, cu_seqlens, max_seqlen, H, dh, scale, nullptr, nullptr, nullptr, o, stream, true);
}

extern "C" int d3tom_attend(const void* q, const void* k, const void* v, int dt,
                            int B, const int32_t* cu_seqlens, int max_seqlen, int H, int dh, float scale,
                            void* o, void* ws, size_t ws_bytes, void* stream) {
    (void)ws; (void)ws_bytes;
    return attend_any(q, k, v, dt, B, cu_seqlens, max_seqlen, H, dh, scale, nullptr, nullptr, nullptr, o, stream);
}

extern "C" int d3tom_attend_weighted(const void* q, const void* k, const void* v, int dt,
                                     int B, const int32_t* cu_seqlens, int max_seqlen, int H, int dh, float scale,
                                     const int32_t* counts, const int32_t* kept_off, const int32_t* vis_start,
                                     void* o, void* ws, size_t ws_bytes, void* stream) {
    (void)ws; (void)ws_bytes;
    if (!counts || !kept_off || !vis_start) return D3TOM_ERR_INVALID_ARG;
    return attend_any(q, k, v, dt, B, cu_seqlens, max_seqlen, H, dh, scale, counts, kept_off, vis_start, o, stream);
}

// ---- for tuning and tests: which kernel takes a call: {generic, short samples, tiles}, queries of a workgroup, whether a workgroup takes
// several tiles in turn, dynamic LDS bytes; whole: as the blocks of a stack in front of its merge call it
extern "C" int d3tom_attend_plan(int dt, int B, int max_seqlen, int H, int dh, int whole, int32_t* plan) {
    if (!plan || B < 1 || max_seqlen < 1 || H < 1 || dh < 1) return D3TOM_ERR_INVALID_ARG;
    const AttendPlan p = attend_plan(dt, B, max_seqlen, H, dh, whole != 0);
    plan[0] = p.kernel;
    plan[1] = p.queries;
    plan[2] = p.turns;
    plan[3] = (int32_t)p.lds;
    return D3TOM_OK;
}
