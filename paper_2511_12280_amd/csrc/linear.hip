// d3tom_linear: out = a w^T for the projections of a transformer block (the per-layer 4 n d^2 and 3 n d m
// terms of the cost model in Section 4.3), bf16 operands, float32 accumulation on MFMA 16x16x32, with the
// element-wise tail of the projection folded into the epilogue:
//   PLAIN     out = a w^T, optionally written as several [rows, out_chunk] matrices (q | k | v)
//   RESIDUAL  out = residual + a w^T                      (the block's two skip connections)
//   SWIGLU    out = silu(a w_gate^T) * (a w_up^T)         (w holds the F gate rows, then the F up rows)
//   ROPE      (inside the stack only) PLAIN for the stacked q | k | v weight with the rotary embedding of the q and k
//             sections folded in; the projection is rounded to bf16 first (the value the separate rotary kernel would have
//             read), turned by the token's angle from a per-step table, and rounded again
//   PARTIAL   (inside the stack only) the contraction is cut into gridDim.y slices and every slice writes
//             its float32 products to its own [rows, n] matrix; the row-wise kernel that follows adds the
//             slices, the residual, rounds once and normalises.  Used where a short sequence leaves the
//             output and down projections with too few tall tiles to fill the chip.
// One rounding to bf16, at the store (ROPE: one for the projection, one for the rotated value).
//
// One workgroup per tile of BM x BN, eight waves, in one of two forms.
// Ping-pong (WC = 4): two groups of four.  Group i owns rows i*BM/2 .. of the tile, its four
// waves a quarter of the columns each; wave i and wave i + 4 share a SIMD.  The groups alternate: in one phase a
// group reads the operand fragments of a whole 64-element k-stage from LDS into registers (and issues direct loads) while
// the other group issues nothing but the MFMAs of the stage it holds; a barrier ends the phase.  Measured on gfx950 with
// 256 x 256 tiles (clocks of a k-stage; the MFMAs alone are 2048): all waves on one schedule 3270, phases of 32 elements
// 2570, phases of 64 2307.  MFMA streams of two waves of one SIMD slow each other down, hence the phases.
// Loading waves (WC = 2): four waves compute a quarter of the tile each, their fragments read one k-step ahead, four only issue the
// direct loads; one barrier a k-stage.  For small tiles, whose phases above would be mostly latency: 2048 x 2048 weights, 493 rows
// 14.9 -> 9.3 us, 11008 channels into 4096 at 1400 rows 127 -> 107 us.  Such a tile is bound by what a compute unit takes in, 62 to 77
// bytes per ns of rows that no other one has had (a deeper ring does not help, and loads that touch the rows ahead of time cost more
// than they give); large tiles are bound by the MFMAs and by power, for which the first form is the better one.
//
// MFMA 16x16x32 and not 32x32x16: at full load the card is power bound (it clocks down to 1.5 GHz), and the smaller shape
// moves fewer accumulator bytes per flop: 2.09 against 1.86 PFLOP/s with operands in registers and random data, 1.24 against
// 1.10 in this loop.  It adds the products in the same order as two 32x32x16 steps; the results are the same bits.
//
// Both operands are contraction-contiguous, so both tiles travel HBM/L2 -> LDS with direct loads (16 bytes per lane, no
// register staging), 128 bytes of every row per stage (a whole cache line: half lines halve the rate of a compute unit's load
// path).  In the first form group 0 fetches the rows of a, group 1 the rows of w; two rings fill the 160 KB of LDS, and the one of w is
// the deeper one, its rows come cold from HBM.  The 16-byte chunk stored at position p of tile row r is chunk p ^ f(r), with f
// such that the 16 rows of a fragment read hit all 64 banks.
//
// The product is formed as w a^T, so that a lane ends up with one row of out and 4 * TN consecutive columns of it: the
// epilogue works on registers and stores 16 bytes per lane, no LDS pass.  For SWIGLU and ROPE rows of w are laid out in the
// tile so that both partners of a pair (gate and up of one output; channels c and c + dh/2) land in the same lane.
//
// Tiles are numbered band by band and cut into 8 equal runs, one per XCD (see linear_tile), so that the 32 workgroups that run
// together on an XCD form a compact block and its private L2 sees few operand rows.
#include <cstdio>
#include <type_traits>
#include "common.hpp"
#include "direct_load.hpp"

namespace d3tom {

enum { LIN_PLAIN = 0, LIN_RESIDUAL = 1, LIN_SWIGLU = 2, LIN_PARTIAL = 3, LIN_ROPE = 4 };
constexpr int LIN_BK = 64;

// A tile of BM x BN.  WC = 4: two groups of four waves in turn, 2 x 4 waves over the tile; WC = 2: four computing waves, 2 x 2, and
// four that load.  TM, TN: 16-row and 16-column fragments of a computing wave.
template <int TM, int TN, int WC> struct LinCfg {
    static constexpr int BM = 32 * TM, BN = 16 * TN * WC;
    static constexpr int A_BYTES = BM * 128, W_BYTES = BN * 128;       // one k-stage of either operand
    // ring depths within 160 KB.  WC = 4: that of w first (deeper); WC = 2: a stage is one thing, at most six of them
    static constexpr int NS_MAX = 163840 / (A_BYTES + W_BYTES), NS = NS_MAX > 6 ? 6 : NS_MAX;
    static constexpr int NW = WC == 2 ? NS : (TN == 4) ? (TM >= 3 ? 3 : 4) : (TN == 3) ? 4 : (TM == 2 ? 6 : TM <= 5 ? 5 : 4);
    static constexpr int NA_MAX = (163840 - NW * W_BYTES) / A_BYTES;
    static constexpr int NA = WC == 2 ? NS : NA_MAX > 6 ? 6 : NA_MAX;
    static constexpr int LDS = NA * A_BYTES + NW * W_BYTES;
    static_assert(NA >= 2 && NW >= 2 && LDS <= 163840 && (WC == 4 || NS >= 3), "rings must fit");
};

// The tiles that there are.  uses: taken for whole projections, for slices of a contraction, or only where d3tom_linear_tile asks for it.  (Of
// 20000 shapes, 1 .. 12000 rows, each tile is the estimate's choice for 20 or more in each of the uses that it is built for.)
enum { LIN_WHOLE = 1, LIN_SLICES = 2, LIN_ASKED = 4 };
struct LinTile { int bm, bn, wc, uses; };
constexpr LinTile LIN_TILES[] = {
    {64, 64, 2, LIN_WHOLE | LIN_SLICES}, {64, 96, 2, LIN_WHOLE | LIN_SLICES}, {64, 128, 2, LIN_WHOLE | LIN_SLICES}, {64, 256, 4, LIN_ASKED},
    {96, 128, 2, LIN_WHOLE | LIN_SLICES}, {128, 128, 4, LIN_WHOLE | LIN_SLICES}, {128, 192, 2, LIN_WHOLE}, {128, 256, 4, LIN_WHOLE},
    {160, 128, 2, LIN_WHOLE | LIN_SLICES}, {160, 256, 4, LIN_WHOLE}, {192, 128, 2, LIN_WHOLE | LIN_SLICES}, {192, 256, 4, LIN_WHOLE},
    {224, 256, 4, LIN_WHOLE}, {256, 128, 4, LIN_SLICES | LIN_ASKED}, {256, 128, 2, LIN_WHOLE}, {256, 192, 4, LIN_WHOLE}, {256, 256, 4, LIN_WHOLE}};
constexpr int LIN_NTILES = sizeof(LIN_TILES) / sizeof(LIN_TILES[0]);
// the uses for which a tile is built with an epilogue
constexpr int linear_uses(int epi) { return epi == LIN_PARTIAL ? LIN_SLICES : epi == LIN_ROPE ? LIN_WHOLE : LIN_WHOLE | LIN_ASKED; }

// Tile (rt, ct) of workgroup id.  Ids are dealt round-robin to the 8 XCDs; the tiles are numbered in bands of RB row tiles,
// column-major inside a band, and that sequence is cut into 8 runs of `per` tiles, one per XCD.
__device__ __forceinline__ bool linear_tile(int id, int per, int RB, int NRT, int NCT, int& rt, int& ct) {
    const int t = (id & 7) * per + (id >> 3);
    if (t >= NRT * NCT) return false;
    const int band = RB * NCT, nfull = NRT / RB;
    if (t < nfull * band) { const int rem = t % band; rt = (t / band) * RB + rem % RB; ct = rem / RB; }
    else { const int t2 = t - nfull * band, rl = NRT - nfull * RB; rt = nfull * RB + t2 % rl; ct = t2 / rl; }
    return true;
}

template <int TM, int TN, int WC, int EPI>
__global__ __launch_bounds__(512, 2) void linear_bf16_kernel(
    const uint16_t* __restrict__ a, const uint16_t* __restrict__ w, int M, int N, int K,
    const uint16_t* residual, uint16_t* out, int out_chunk, int NRT, int NCT, int per, int RB, int col0, int col_end,
    const float2* __restrict__ rope_cs, int rope_dh) {
#if defined(__HIP_DEVICE_COMPILE__)
    using C = LinCfg<TM, TN, WC>;
    constexpr int BM = C::BM, BN = C::BN, NA = C::NA, NW = C::NW;
    constexpr int LA = BM / 32, LW = BN / 32;           // direct loads per loading wave and stage (8 rows each)
    constexpr bool PAIR = EPI == LIN_SWIGLU || EPI == LIN_ROPE;
    extern __shared__ __attribute__((aligned(16))) char ring[];     // NA stages of a, then NW stages of w

    int rt, ct;
    if (!linear_tile(blockIdx.x, per, RB, NRT, NCT, rt, ct)) return;

    const int tid = threadIdx.x, lane = tid & 63;
    // (the wave's number is kept in a scalar register where the tile needs every vector register: 256 x 128 with loading waves spilled one)
    const int half_wg = __builtin_amdgcn_readfirstlane(tid >> 8), wn = (WC == 2 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6) & 3;
    const int r = lane & 15, g = lane >> 4;
    // a computing wave's part of the tile: rows grp * BM/2 .., columns wcol * BN/WC ..
    const int grp = WC == 4 ? half_wg : wn >> 1, wcol = WC == 4 ? wn : wn & 1;
    const int n_out = (EPI == LIN_SWIGLU) ? N / 2 : N;  // SWIGLU: N counts gate and up rows
    // What a tile's columns are: plain columns, or pairs (SWIGLU: output o = rows o and o + F of w; ROPE: channels c, c + dh/2)
    constexpr int UNITS = PAIR ? BN / 2 : BN;
    const int unit0 = ((EPI == LIN_ROPE) ? col0 / 2 : col0) + ct * UNITS;
    const int unit_end = (EPI == LIN_ROPE) ? col_end / 2 : col_end;
    const int half = rope_dh >> 1;

    // rows past the end re-read row 0 (their results are never stored); the k-stage moves through the scalar offset
    auto a_offset = [&](int i) {
        const int row = wn * (BM / 4) + i * 8 + (lane >> 3), m = rt * BM + row;
        return (m < M ? m : 0) * K * 2 + (((lane & 7) ^ ((row >> 1) & 7)) << 4);
    };
    auto w_offset = [&](int i) {
        const int row = wn * (BN / 4) + i * 8 + (lane >> 3);
        const int part = row / (16 * TN), q = row - part * 16 * TN, qg = q / (4 * TN);
        int n, ok;
        if constexpr (PAIR) {
            const int u = unit0 + part * 8 * TN + qg * 2 * TN + ((q - qg * 4 * TN) >> 2) * 2 + (q & 1);
            const int second = (q >> 1) & 1;
            ok = u < unit_end;
            if constexpr (EPI == LIN_SWIGLU) n = u + second * n_out;
            else { const int h = u / half; n = h * rope_dh + (u - h * half) + second * half; }
        } else {
            n = unit0 + row;
            ok = n < unit_end;
        }
        return (ok ? n : 0) * K * 2 + (((lane & 7) ^ (((q >> 1) & 1) | (qg << 1))) << 4);
    };
    const int nst = (K / LIN_BK) / (int)gridDim.y;         // k-stages of this workgroup's slice of the contraction
    const int st0 = (int)blockIdx.y * nst;
    const uint32_t ring0 = (uint32_t)(size_t)(lds_ptr_t)ring;
    const uint32_t a_lds = __builtin_amdgcn_readfirstlane(ring0 + wn * (BM / 4) * 128);
    const uint32_t w_lds = __builtin_amdgcn_readfirstlane(ring0 + NA * C::A_BYTES + wn * (BN / 4) * 128);

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // fragment addresses inside a stage: a fragment of a is 16 consecutive rows; row x of w fragment j is tile row
    // (x / 4) * 4 TN + 4 j + x % 4 of the wave's part
    int a_addr[2], w_addr[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const int ra = grp * (BM / 2) + r, q = (r >> 2) * 4 * TN + (r & 3);
        a_addr[kk] = ra * 128 + (((kk * 4 + g) ^ ((ra >> 1) & 7)) << 4);
        w_addr[kk] = NA * C::A_BYTES + (wcol * 16 * TN + q) * 128 + (((kk * 4 + g) ^ (((q >> 1) & 1) | ((r >> 2) << 1))) << 4);
    }
    // The columns of a fragment row are taken there and those of the next one back, so that every MFMA has an operand in common with the one
    // before it: less switching, and the card is power bound (3773 rows, 256 x 256 tiles, 12288 columns of 4096 279.6 -> 276.1 us, 4096
    // of 11008 242.2 -> 238.5, with 256 x 128 tiles and loading waves 268.6 -> 265.7; 160 x 256 at 2100 rows 166.1 -> 165.6, as much as two runs
    // differ; short launches -0.4 to 0.9 %).  Where a wave holds both k-steps of a stage, they follow one another in each accumulator: the second
    // product takes the sum where the first has just left it.  MFMAs alone, random data: 2.08 -> 2.20 PFLOP/s; 3773 rows, 12288 columns of 4096
    // 273.3 -> 265.7 us, gate | up of 11008 498.2 -> 487.8, 2100 rows 296.9 -> 291.5, 493 rows 84.3 -> 83.2 (fragments of a row and not of a column
    // held in between: the same).
    auto there_and_back = [](int i, int j) { return (i & 1) ? TN - 1 - j : j; };
    bf16x8 af[2][TM], wf[2][TN];
    if constexpr (WC == 4) {
        auto read = [&](int sa, int sw) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const char* pw = ring + sw * C::W_BYTES + w_addr[kk];
                const char* pa = ring + sa * C::A_BYTES + a_addr[kk];
#pragma unroll
                for (int j = 0; j < TN; ++j) wf[kk][j] = *reinterpret_cast<const bf16x8*>(pw + j * 4 * 128);
#pragma unroll
                for (int i = 0; i < TM; ++i) af[kk][i] = *reinterpret_cast<const bf16x8*>(pa + i * 16 * 128);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto compute = [&]() {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int n = 0; n < TM * TN; ++n)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    const int i = n / TN, j = there_and_back(i, n % TN);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[kk][j], af[kk][i], acc[i][j], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
        };
        auto next = [](int slot, int n) { return slot + 1 == n ? 0 : slot + 1; };
        // Stage s sits in slot s mod NA (NW).  Group 0 reads it in phase 2s, group 1 in phase 2s + 1; from phase 2s + 2 on its
        // slots may be refilled, which group 0 does for a in that phase and group 1 for w one later.  Before the barrier that ends
        // phase 2s + 1 both groups wait for their own loads of stage s + 1.
        if (half_wg == 0) {
            int off[LA];
#pragma unroll
            for (int i = 0; i < LA; ++i) off[i] = a_offset(i);
            const __amdgpu_buffer_rsrc_t rs = make_uniform_rsrc(a, (uint32_t)((size_t)M * K * 2));
            auto issue = [&](int s, int slot) {
#pragma unroll
                for (int i = 0; i < LA; ++i)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(size_t)(a_lds + slot * C::A_BYTES + i * 1024), 16, off[i], (st0 + s) * 128, 0, 0);
            };
#pragma unroll
            for (int s = 0; s < NA; ++s) if (s < nst) issue(s, s);
            if (nst >= NA) wait_loads<(NA - 1) * LA>(); else wait_loads<0>();
            phase_barrier();
            int sa = 0, sw = 0, fill = NA - 1;
#pragma unroll 1
            for (int s = 0; s < nst; ++s) {
                const bool more = s + NA - 1 < nst;
                read(sa, sw);
                if (s > 0 && more) issue(s + NA - 1, fill);
                wait_lds();
                phase_barrier();
                compute();
                if (more) wait_loads<(NA - 2) * LA>(); else wait_loads<0>();
                phase_barrier();
                fill = sa; sa = next(sa, NA); sw = next(sw, NW);
            }
            phase_barrier();
        } else {
            int off[LW];
#pragma unroll
            for (int i = 0; i < LW; ++i) off[i] = w_offset(i);
            const __amdgpu_buffer_rsrc_t rs = make_uniform_rsrc(w, (uint32_t)((size_t)N * K * 2));
            auto issue = [&](int s, int slot) {
#pragma unroll
                for (int i = 0; i < LW; ++i)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t)(size_t)(w_lds + slot * C::W_BYTES + i * 1024), 16, off[i], (st0 + s) * 128, 0, 0);
            };
#pragma unroll
            for (int s = 0; s < NW; ++s) if (s < nst) issue(s, s);
            if (nst >= NW) wait_loads<(NW - 1) * LW>(); else wait_loads<0>();
            phase_barrier();
            phase_barrier();
            int sa = 0, sw = 0, fill = NW - 1;
#pragma unroll 1
            for (int s = 0; s < nst; ++s) {
                const bool more = s + NW - 1 < nst;
                read(sa, sw);
                if (s > 0 && more) issue(s + NW - 1, fill);
                wait_lds();
                if (more) wait_loads<(NW - 2) * LW>(); else wait_loads<0>();
                phase_barrier();
                compute();
                phase_barrier();
                fill = sw; sa = next(sa, NA); sw = next(sw, NW);
            }
        }
    } else if (half_wg == 1) {
        // the loading waves: stage s + NA - 1 goes into the slot of stage s - 1 once the computing waves have that in registers
        const __amdgpu_buffer_rsrc_t ra = make_uniform_rsrc(a, (uint32_t)((size_t)M * K * 2)), rw = make_uniform_rsrc(w, (uint32_t)((size_t)N * K * 2));
        int off_a[LA], off_w[LW];
#pragma unroll
        for (int i = 0; i < LA; ++i) off_a[i] = a_offset(i);
#pragma unroll
        for (int i = 0; i < LW; ++i) off_w[i] = w_offset(i);
        auto issue = [&](int s, int slot) {
#pragma unroll
            for (int i = 0; i < LW; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_ptr_t)(size_t)(w_lds + slot * C::W_BYTES + i * 1024), 16, off_w[i], (st0 + s) * 128, 0, 0);
#pragma unroll
            for (int i = 0; i < LA; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr_t)(size_t)(a_lds + slot * C::A_BYTES + i * 1024), 16, off_a[i], (st0 + s) * 128, 0, 0);
        };
#pragma unroll
        for (int s = 0; s < NA - 1; ++s) if (s < nst) issue(s, s);
        int fill = NA - 1;
#pragma unroll 1
        for (int s = 0; s < nst; ++s) {
            if (s + NA - 2 < nst) wait_loads_and_barrier<(NA - 2) * (LA + LW)>(); else wait_loads_and_barrier<0>();
            if (s + NA - 1 < nst) issue(s + NA - 1, fill);
            fill = fill + 1 == NA ? 0 : fill + 1;
        }
        return;
    } else {
        // the computing waves: the fragments of the next k-step of 32 are read behind the first MFMAs of this one, across the
        // barrier too (the one for stage s + 1 lies between the two k-steps of stage s)
        auto read_one = [&](int slot, int kk, int f) {
            if (f < TN) wf[kk][f] = *reinterpret_cast<const bf16x8*>(ring + slot * C::W_BYTES + w_addr[kk] + f * 4 * 128);
            else af[kk][f - TN] = *reinterpret_cast<const bf16x8*>(ring + slot * C::A_BYTES + a_addr[kk] + (f - TN) * 16 * 128);
        };
        auto multiply = [&](int kk, int slot, bool read) {     // MFMAs of k-step kk; the other one's fragments from `slot`
#pragma unroll
            for (int n = 0; n < TM * TN; ++n) {
                const int i = n / TN, j = there_and_back(i, n % TN);
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[kk][j], af[kk][i], acc[i][j], 0, 0, 0);
                if (read && n < TM + TN) {
                    __builtin_amdgcn_sched_barrier(0);
                    read_one(slot, kk ^ 1, n);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        static_assert(TM * TN >= TM + TN, "a fragment is read behind every MFMA");
        wait_loads_and_barrier<0>();
#pragma unroll
        for (int f = 0; f < TM + TN; ++f) read_one(0, 0, f);
        int slot = 0;
#pragma unroll 1
        for (int s = 0; s + 1 < nst; ++s) {
            multiply(0, slot, true);
            __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0): stage s is in registers
            phase_barrier();
            slot = slot + 1 == NA ? 0 : slot + 1;
            multiply(1, slot, true);
        }
        multiply(0, slot, true);
        multiply(1, slot, false);
    }

    // epilogue, in registers: lane (r, g) holds row r of every 16-row fragment and, over the TN fragments, 4 TN consecutive
    // values of its part: plain columns, or (PAIR) 2 TN consecutive outputs with their partners in elements 2 and 3
    const int u0 = unit0 + wcol * (UNITS / WC) + g * (UNITS / (4 * WC));
    // values per store (plain columns: never across an out_chunk, a multiple of 8), and where they go from the start of a row of the output's first
    // section: worked out once for all rows
    constexpr int V = !PAIR ? ((TN % 2 == 0) ? 8 : 4) : (TN % 4 == 0) ? 8 : (TN % 2 == 0) ? 4 : 2, NV = (PAIR ? 2 : 4) * TN / V;
    const int row_width = EPI == LIN_PARTIAL ? N : out_chunk;
    size_t at[NV];
    int c[EPI == LIN_ROPE ? NV : 1];                    // ROPE: the first channel's place in its half of the head
#pragma unroll
    for (int x = 0; x < NV; ++x) {
        int col = min(u0 + x * V, unit_end - V);        // past the end: loaded from there, not stored
        if constexpr (EPI == LIN_ROPE) { const int h = col / half; c[x] = col - h * half; col = h * rope_dh + c[x]; }
        const int section = col / row_width;
        at[x] = (size_t)section * M * row_width + (col - section * row_width);
    }
    auto row_of = [&](int i) { return rt * BM + grp * (BM / 2) + i * 16 + r; };
    if constexpr (EPI == LIN_PARTIAL) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (row_of(i) >= M) continue;
            float* po = reinterpret_cast<float*>(out) + ((size_t)blockIdx.y * M + row_of(i)) * N + u0;
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (u0 + j * 4 < unit_end) *reinterpret_cast<f32x4*>(po + j * 4) = acc[i][j];
        }
    } else if constexpr (!PAIR) {
        // all of the residual is requested before the first of it is used (it may be the output: nobody else writes these elements)
        uint32_t rr[EPI == LIN_RESIDUAL ? TM : 1][NV][V / 2];
        if constexpr (EPI == LIN_RESIDUAL) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int x = 0; x < NV; ++x)
                    __builtin_memcpy(rr[i][x], __builtin_assume_aligned(residual + at[x] + (size_t)min(row_of(i), M - 1) * row_width, V * 2), V * 2);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int x = 0; x < NV; ++x) {
                float v[V];
#pragma unroll
                for (int e = 0; e < V; ++e) v[e] = acc[i][(x * V + e) >> 2][e & 3];
                if constexpr (EPI == LIN_RESIDUAL) {
#pragma unroll
                    for (int e = 0; e < V / 2; ++e) { v[2 * e] += bf16_lo(rr[i][x][e]); v[2 * e + 1] += bf16_hi(rr[i][x][e]); }
                }
                if (row_of(i) < M && u0 + x * V < unit_end) store_bf16<V>(out + at[x] + (size_t)row_of(i) * row_width, v);
            }
    } else {
        // ROPE: (cos, sin) of channels 2 e and 2 e + 1 of the next row are requested in front of a row's arithmetic, also by tiles of the v section, which use
        // none (under a condition, 55 shapes of 16 to 3773 rows 0.994 in the mean, 3773 rows of 512 channels 12.2 -> 13.4 us)
        float4 cs[2][EPI == LIN_ROPE ? NV : 1][V / 2];
        auto request = [&](int i) {
#pragma unroll
            for (int n = 0; n < NV; ++n)
#pragma unroll
                for (int e = 0; e < V / 2; ++e)
                    cs[i & 1][n][e] = reinterpret_cast<const float4*>(rope_cs + (size_t)min(row_of(i), M - 1) * half + c[n])[e];
        };
        if constexpr (EPI == LIN_ROPE) request(0);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if constexpr (EPI == LIN_ROPE) if (i + 1 < TM) request(i + 1);
#pragma unroll
            for (int n = 0; n < NV; ++n) {
                float x[V], y[V];
#pragma unroll
                for (int e = 0; e < V; ++e) { x[e] = acc[i][(n * V + e) >> 1][e & 1]; y[e] = acc[i][(n * V + e) >> 1][2 + (e & 1)]; }
                uint16_t* o = out + at[n] + (size_t)row_of(i) * row_width;
                const bool in = row_of(i) < M && u0 + n * V < unit_end;
                if constexpr (EPI == LIN_SWIGLU) {
#pragma unroll
                    for (int e = 0; e < V; ++e) x[e] = x[e] / (1.f + expf(-x[e])) * y[e];
                    if (in) store_bf16<V>(o, x);
                } else {
                    const int h = (u0 + n * V) / half;
                    if (h * rope_dh + c[n] < 2 * out_chunk) {          // q and k sections; v passes through
#pragma unroll
                        for (int e = 0; e < V / 2; ++e) {
                            const float4 t = cs[i & 1][n][e];
                            // both channels as the stored bf16 projection, then the rotation in float32
#pragma unroll
                            for (int f = 0; f < 2; ++f) {
                                const float x0 = bf16_bits_to_f32(f32_to_bf16_bits(x[2 * e + f])), x1 = bf16_bits_to_f32(f32_to_bf16_bits(y[2 * e + f]));
                                rope_rotate(x0, x1, f ? t.z : t.x, f ? t.w : t.y, x[2 * e + f], y[2 * e + f]);
                            }
                        }
                    }
                    if (in) { store_bf16<V>(o, x); store_bf16<V>(o + half, y); }
                }
            }
        }
    }
#endif
}

namespace {
template <int TM, int TN, int WC, int EPI>
int launch_linear(const void* a, const void* w, int M, int N, int K, const void* residual, void* out, int out_chunk,
                  int ksplit, int col0, int col_end, hipStream_t st, const float2* rope_cs = nullptr, int rope_dh = 0) {
    using C = LinCfg<TM, TN, WC>;
    static PerDeviceOnce lds_setup;      // per instantiation
    if (!lds_setup.run([] { return raise_dynamic_lds(linear_bf16_kernel<TM, TN, WC, EPI>, C::LDS); })) return D3TOM_ERR_DEVICE;
    const int out_bn = (EPI == LIN_SWIGLU) ? C::BN / 2 : C::BN;
    const int NRT = ceil_div(M, C::BM), NCT = ceil_div(col_end - col0, out_bn);
    const int per = ceil_div(NRT * NCT, 8);
    // the (at most) 32 workgroups that run together on an XCD: a block of RB row tiles whose operand rows are as few as
    // possible, i.e. RB * BM close to (32 / RB) * BN
    const int conc = per < 32 ? per : 32;
    int RB = 1;
    while ((RB + 1) * (RB + 1) * C::BM <= conc * C::BN) ++RB;
    if (RB > NRT) RB = NRT;
    D3TOM_LAUNCH(LINEAR, st, (linear_bf16_kernel<TM, TN, WC, EPI><<<dim3(8u * (unsigned)per, (unsigned)ksplit), 512, C::LDS, st>>>(
        (const uint16_t*)a, (const uint16_t*)w, M, N, K, (const uint16_t*)residual, (uint16_t*)out, out_chunk,
        NRT, NCT, per, RB, col0, col_end, rope_cs, rope_dh)));
    return D3TOM_OK;
}

// the kernel of entry `cfg` of LIN_TILES
template <int EPI, int C = 0>
int launch_linear_cfg(int cfg, const void* a, const void* w, int M, int N, int K, const void* residual, void* out, int out_chunk,
                      int ksplit, int col0, int col_end, hipStream_t st, const float2* rope_cs = nullptr, int rope_dh = 0) {
    if constexpr (C < LIN_NTILES) {
        if (cfg != C) return launch_linear_cfg<EPI, C + 1>(cfg, a, w, M, N, K, residual, out, out_chunk, ksplit, col0, col_end, st, rope_cs, rope_dh);
        constexpr LinTile t = LIN_TILES[C];
        if constexpr ((t.uses & linear_uses(EPI)) != 0)
            return launch_linear<t.bm / 32, t.bn / (16 * t.wc), t.wc, EPI>(a, w, M, N, K, residual, out, out_chunk, ksplit, col0, col_end, st, rope_cs, rope_dh);
    }
    return D3TOM_ERR_UNSUPPORTED;
}
}  // namespace

// ---- choice of the tile -----------------------------------------------------------------------------
// A grid runs in rounds of 256 workgroups, one per compute unit, and a mostly empty last round costs as much time as a full one: hence
// tiles of many heights.  What a launch takes, in microseconds:
//   rounds * (stages * (rows a tile takes in of either operand) + epilogue and ring) + tiles / 256 * stages * products + launch
// The rows count however few tiles there are; the products count by how full the chip is (above all power).  The two forms have constants of
// their own, tiles of the same form share them; a wave whose fragments are three columns wide stores 8 bytes at a time instead of 16.
// Cut contractions besides: what a million values of a partial matrix take to write (by eight waves or by four, whose fragments fill the
// lines they store, or are more than three columns wide and leave gaps between the lanes) and to read again.
// Fitted to the times within 1.3 of a shape's best of 782 shapes, 259 of them with cut contractions too (16 .. 4600 rows; q | k | v, output,
// gate | up and down projections of 512 .. 5632 channels; weights cold in HBM): there the choice is 0.7 % behind the best built tile on
// average.  On 654 shapes that the fit has not seen it is 0.8 % behind, 3.8 % at the 90th percentile, 9.8 % at the 99th, 19.6 % at most.  (A
// table of five constants for each of the 17 tiles: 0.9 %, 3.8, 10.9 and 24.7 %.)  profiles/projection_tiles.txt has the times.
static double linear_estimate(int cfg, int M, int cols, int nst, int ksplit) {
    struct Form { double a_rows, w_rows, products, round; };
    constexpr Form PING_PONG = {0.50, 0.40, 0.36, 9.31}, LOADERS = {0.36, 0.54, 0.32, 4.02};       // of 256 rows, 256 x 256 tiles
    constexpr double LAUNCH = 2.18, NARROW_STORES = 1.85, PART_PING_PONG = 0.54, PART_LOADERS = 0.90, PART_GAPS = 1.45, PART_READ = 0.45;
    const LinTile& t = LIN_TILES[cfg];
    const Form& f = t.wc == 4 ? PING_PONG : LOADERS;
    const int tn = t.bn / (16 * t.wc);
    const long tiles = (long)ceil_div(M, t.bm) * ceil_div(cols, t.bn) * ksplit;
    const double area = (double)(t.bm * t.bn) / 65536.0, stages = nst / ksplit;
    double us = (double)((tiles + 255) / 256) * (stages * (f.a_rows * t.bm + f.w_rows * t.bn) / 256.0 + (f.round + (tn == 3 ? NARROW_STORES : 0.0)) * area);
    us += (double)tiles / 256.0 * stages * f.products * area + LAUNCH;
    if (ksplit > 1) us += (double)M * cols * ksplit * 1e-6 * ((tn > 3 ? PART_GAPS : t.wc == 4 ? PART_PING_PONG : PART_LOADERS) + PART_READ);
    return us;
}
// the best tile for a projection in one launch (`cols` counts rows of w; SWIGLU: gate and up); bm: of that height
static int linear_pick(int M, int cols, int nst, int bm, double* est) {
    int best = -1;
    double best_t = 0.0;
    for (int c = 0; c < LIN_NTILES; ++c) {
        if (!(LIN_TILES[c].uses & LIN_WHOLE) || (bm && LIN_TILES[c].bm != bm)) continue;
        const double t = linear_estimate(c, M, cols, nst, 1);
        if (best < 0 || t < best_t) { best = c; best_t = t; }
    }
    *est = best_t;
    return best;
}
// A last round that is mostly empty can be cut off: the leading columns that fill whole rounds go in one launch, the
// remaining ones in a second launch with whatever tile suits them (4600 rows x 22016 x 4096: 1548 tiles of 256 x 256 are six full rounds
// and twelve, 627 us in one launch, 599 in two).  `cols` in rows of w; *cols_a: rows of w of the first launch (all of them: one launch), a
// multiple of its tile width.
constexpr double LIN_SECOND_US = 4.0;       // the first launch drains and the second fills its rings
struct LinPlan { int cfg_a, cols_a, cfg_b; double est; };
static LinPlan linear_plan(int M, int cols, int nst) {
    LinPlan p;
    p.cfg_a = linear_pick(M, cols, nst, 0, &p.est);
    p.cols_a = cols;
    p.cfg_b = 0;
    const double single = p.est;
    for (int c = 0; c < LIN_NTILES; ++c) {
        if (!(LIN_TILES[c].uses & LIN_WHOLE)) continue;
        const int nrt = ceil_div(M, LIN_TILES[c].bm), nct = ceil_div(cols, LIN_TILES[c].bn);
        const int rounds = (int)((long)nrt * nct / 256);
        const int lead = rounds > 0 ? rounds * 256 / nrt : 0;
        if (lead < 1 || lead >= nct) continue;
        double rest;
        const int cb = linear_pick(M, cols - lead * LIN_TILES[c].bn, nst, 0, &rest);
        const double t = linear_estimate(c, M, lead * LIN_TILES[c].bn, nst, 1) + rest + LIN_SECOND_US;
        if (t < p.est && t < 0.95 * single) { p.cfg_a = c; p.cols_a = lead * LIN_TILES[c].bn; p.cfg_b = cb; p.est = t; }
    }
    return p;
}

// Contraction slices for a projection whose result goes through the row-wise add-and-normalise kernel anyway: cutting the
// contraction fills the chip where the tiles of a short sequence do not, at the price of writing `ksplit` float32 matrices and of the row
// kernel reading them (0.45 us per million values more than without).  Returns 1 (no split), 2 or 4; *cfg is the tile.
// max_floats bounds the partial matrices together.
int linear_split_plan(int M, int N, int K, size_t max_floats, int* cfg) {
    const int nst = K / LIN_BK;
    const LinPlan whole = linear_plan(M, N, nst);
    int best = 1;
    double best_t = whole.est;
    *cfg = whole.cfg_a;
    if (K % LIN_BK != 0 || N % 8 != 0) return 1;
    for (int ks = 2; ks <= 4; ks <<= 1) {
        if (nst % ks || nst / ks < 8 || (size_t)M * N * ks > max_floats) continue;
        for (int c = 0; c < LIN_NTILES; ++c) {
            if (!(LIN_TILES[c].uses & LIN_SLICES)) continue;
            const double t = linear_estimate(c, M, N, nst, ks);
            if (t < best_t) { best = ks; best_t = t; *cfg = c; }
        }
    }
    return best;
}

// a w^T as `ksplit` float32 partial matrices [ksplit][M][N]
int linear_partial_run(const void* a, const void* w, int M, int N, int K, int ksplit, int cfg, float* partial, hipStream_t st) {
    if (!a || !w || !partial || M < 1 || N < 1 || K < 1 || ksplit < 1 || cfg < 0 || cfg >= LIN_NTILES) return D3TOM_ERR_INVALID_ARG;
    if (!aligned16(a) || !aligned16(w) || !aligned16(partial)) return D3TOM_ERR_INVALID_ARG;
    if (K % (LIN_BK * ksplit) != 0 || N % 8 != 0) return D3TOM_ERR_UNSUPPORTED;
    if ((size_t)M * K * 2 >= (1ull << 31) || (size_t)N * K * 2 >= (1ull << 31)) return D3TOM_ERR_UNSUPPORTED;
    return launch_linear_cfg<LIN_PARTIAL>(cfg, a, w, M, N, K, nullptr, partial, N, ksplit, 0, N, st);
}

// tile: 0 the estimate's choice, (1 + c) * LIN_PIN entry c of LIN_TILES, otherwise height and width as in d3tom_linear_tile.
constexpr int LIN_PIN = 256;
// rope_cs != nullptr (PLAIN only, stacked q | k | v weight with out_chunk = d, head size rope_dh of 64 or 128): the
// rotary embedding of the q and k sections is applied in the epilogue; rope_cs[row * rope_dh / 2 + c] = (cos, sin)
int linear_run(const void* a, const void* w, int M, int N, int K, int epilogue, const void* residual, void* out,
               int out_chunk, int tile, hipStream_t st, const float2* rope_cs, int rope_dh) {
    if (!a || !w || !out || M < 1 || N < 1 || K < 1) return D3TOM_ERR_INVALID_ARG;
    if (epilogue < LIN_PLAIN || epilogue > LIN_SWIGLU) return D3TOM_ERR_INVALID_ARG;
    if (rope_cs && (epilogue != LIN_PLAIN || (rope_dh != 64 && rope_dh != 128) || out_chunk <= 0 || out_chunk % rope_dh != 0 ||
                    N != 3 * out_chunk))
        return D3TOM_ERR_INVALID_ARG;
    if (epilogue == LIN_RESIDUAL && !residual) return D3TOM_ERR_INVALID_ARG;
    if (!aligned16(a) || !aligned16(w) || !aligned16(out) || (residual && !aligned16(residual))) return D3TOM_ERR_INVALID_ARG;
    if (K % LIN_BK != 0) return D3TOM_ERR_UNSUPPORTED;
    const int n_out = (epilogue == LIN_SWIGLU) ? N / 2 : N;
    if (epilogue == LIN_SWIGLU && (N % 2 != 0)) return D3TOM_ERR_INVALID_ARG;
    if (n_out % 8 != 0) return D3TOM_ERR_UNSUPPORTED;
    if (out_chunk <= 0) out_chunk = n_out;
    if (out_chunk % 8 != 0 || n_out % out_chunk != 0) return D3TOM_ERR_INVALID_ARG;
    if (epilogue != LIN_PLAIN && out_chunk != n_out) return D3TOM_ERR_INVALID_ARG;
    // 32-bit byte offsets inside each operand
    if ((size_t)M * K * 2 >= (1ull << 31) || (size_t)N * K * 2 >= (1ull << 31)) return D3TOM_ERR_UNSUPPORTED;
    // from here on columns are counted in rows of w; SWIGLU stores half as many columns
    const int per_col = (epilogue == LIN_SWIGLU) ? 2 : 1;
    auto launch = [&](int cfg, int c0, int c1) {
        c0 /= per_col; c1 /= per_col;
        switch (epilogue) {
            case LIN_PLAIN:
                if (rope_cs) return launch_linear_cfg<LIN_ROPE>(cfg, a, w, M, N, K, residual, out, out_chunk, 1, c0, c1, st, rope_cs, rope_dh);
                return launch_linear_cfg<LIN_PLAIN>(cfg, a, w, M, N, K, residual, out, out_chunk, 1, c0, c1, st);
            case LIN_RESIDUAL: return launch_linear_cfg<LIN_RESIDUAL>(cfg, a, w, M, N, K, residual, out, out_chunk, 1, c0, c1, st);
            default: return launch_linear_cfg<LIN_SWIGLU>(cfg, a, w, M, N, K, residual, out, out_chunk, 1, c0, c1, st);
        }
    };
    if (tile >= LIN_PIN) return (tile / LIN_PIN > LIN_NTILES) ? D3TOM_ERR_INVALID_ARG : launch(tile / LIN_PIN - 1, 0, N);
    if (tile) {
        const int bm = (tile & 15) * 64, bn = (tile >> 4) * 64;
        for (int c = 0; c < LIN_NTILES; ++c)
            if (LIN_TILES[c].bm == bm && LIN_TILES[c].bn == bn) return launch(c, 0, N);
        if (bn) return D3TOM_ERR_INVALID_ARG;
        double est;
        return launch(linear_pick(M, N, K / LIN_BK, bm, &est), 0, N);
    }
    const LinPlan p = linear_plan(M, N, K / LIN_BK);
    const int status = launch(p.cfg_a, 0, p.cols_a);
    return (status != D3TOM_OK || p.cols_a >= N) ? status : launch(p.cfg_b, p.cols_a, N);
}

}  // namespace d3tom

extern "C" int d3tom_linear(const void* a, const void* w, int rows, int n_w_rows, int K, int epilogue,
                            const void* residual, void* out, int out_chunk, void* stream) {
    return d3tom::linear_run(a, w, rows, n_w_rows, K, epilogue, residual, out, out_chunk, 0, (hipStream_t)stream, nullptr, 0);
}

// Same as d3tom_linear with the tile fixed: its height (64, 128 or 256 rows: low four bits 1, 2, 4) and, unless zero, its width in
// rows of w (128, 192 or 256: the bits above 2, 3, 4; 64 x 192 is not built); for tuning and tests.
extern "C" int d3tom_linear_tile(const void* a, const void* w, int rows, int n_w_rows, int K, int epilogue,
                                 const void* residual, void* out, int out_chunk, int tile, void* stream) {
    const int h = tile & 15, wd = tile >> 4;
    if (tile < 0 || (h != 1 && h != 2 && h != 4) || (wd != 0 && (wd < 2 || wd > 4))) return D3TOM_ERR_INVALID_ARG;
    return d3tom::linear_run(a, w, rows, n_w_rows, K, epilogue, residual, out, out_chunk, tile, (hipStream_t)stream, nullptr, 0);
}

// ---- for tuning and tests: the tiles by index, with every epilogue, and what the estimate chooses ----
extern "C" const char* d3tom_linear_tile_name(int index) {
    using namespace d3tom;
    struct Names {
        char text[LIN_NTILES][16];
        Names() { for (int c = 0; c < LIN_NTILES; ++c) snprintf(text[c], sizeof text[c], "%dx%d%s", LIN_TILES[c].bm, LIN_TILES[c].bn, LIN_TILES[c].wc == 2 ? " loaders" : ""); }
    };
    static const Names names;
    return index < 0 || index >= LIN_NTILES ? nullptr : names.text[index];
}

extern "C" int d3tom_linear_plan(int rows, int n_w_rows, int K, size_t partial_floats, int32_t* plan) {
    using namespace d3tom;
    if (!plan || rows < 1 || n_w_rows < 1 || K < LIN_BK || K % LIN_BK != 0) return D3TOM_ERR_INVALID_ARG;
    const LinPlan p = linear_plan(rows, n_w_rows, K / LIN_BK);
    int cfg = p.cfg_a;
    plan[3] = partial_floats ? linear_split_plan(rows, n_w_rows, K, partial_floats, &cfg) : 1;
    const bool two = plan[3] == 1 && p.cols_a < n_w_rows;
    plan[0] = cfg;
    plan[1] = two ? p.cols_a : n_w_rows;
    plan[2] = two ? p.cfg_b : -1;
    return D3TOM_OK;
}

extern "C" int d3tom_linear_pinned(const void* a, const void* w, int rows, int n_w_rows, int K, int epilogue, const void* extra, void* out,
                                   int out_chunk, int index, int slices, int rope_dh, void* stream) {
    using namespace d3tom;
    hipStream_t st = (hipStream_t)stream;
    if (index < 0 || index >= LIN_NTILES) return D3TOM_ERR_INVALID_ARG;
    if (epilogue == LIN_PARTIAL) return linear_partial_run(a, w, rows, n_w_rows, K, slices, index, (float*)out, st);
    const int tile = (1 + index) * LIN_PIN;
    if (epilogue != LIN_ROPE) return linear_run(a, w, rows, n_w_rows, K, epilogue, extra, out, out_chunk, tile, st, nullptr, 0);
    if (!extra) return D3TOM_ERR_INVALID_ARG;
    return linear_run(a, w, rows, n_w_rows, K, LIN_PLAIN, nullptr, out, out_chunk, tile, st, (const float2*)extra, rope_dh);
}
