// Internal helpers shared by the gfx950 kernels of libd3tom (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <mutex>
#include "../../include/d3tom.h"

namespace d3tom {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int WAVE = 64;
constexpr float LOG2E = 1.4426950408889634f;

// ---- bf16 <-> f32 -------------------------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
// round-to-nearest-even, v_cvt_pk_bf16_f32: one instruction for two values (by shifts and adds it is nine)
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)lo, (__bf16)hi});
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// V values rounded to bf16 and stored in one piece (p aligned to V elements)
template <int V>
__device__ __forceinline__ void store_bf16(uint16_t* p, const float (&v)[V]) {
    uint32_t w[V / 2];
#pragma unroll
    for (int e = 0; e < V / 2; ++e) w[e] = pack_bf16x2(v[2 * e], v[2 * e + 1]);
    __builtin_memcpy(__builtin_assume_aligned(p, V * 2), w, V * 2);
}

// element load as float for the generic (untuned) kernels
template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float load(const float* p) { return *p; }
    static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct Elem<uint16_t> {   // bf16 storage
    static __device__ __forceinline__ float load(const uint16_t* p) { return bf16_bits_to_f32(*p); }
    static __device__ __forceinline__ void store(uint16_t* p, float v) { *p = f32_to_bf16_bits(v); }
};

// Dot product of two rows of n elements (16-byte aligned, n a multiple of the elements per 16 bytes):
// 16-byte loads, eight chunks requested before the first is used, float32 accumulation.  For the
// generic kernels, whose time is load latency: one scalar load per multiply made them 10-50 times slower.
template <typename T>
__device__ __forceinline__ float chunk_dot(const uint4& a, const uint4& b, float acc) {
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if constexpr (sizeof(T) == 2) {
            acc = __builtin_fmaf(bf16_lo(aw[e]), bf16_lo(bw[e]), acc);
            acc = __builtin_fmaf(bf16_hi(aw[e]), bf16_hi(bw[e]), acc);
        } else {
            acc = __builtin_fmaf(__uint_as_float(aw[e]), __uint_as_float(bw[e]), acc);
        }
    }
    return acc;
}
// The products are added as wave_row_dots adds them: sixteen chains over chunks u, u + 16, ..., then neighbours, pairs, quads and eights.
template <typename T>
__device__ __forceinline__ float row_dot(const T* __restrict__ a, const T* __restrict__ b, int n) {
    const uint4* pa = reinterpret_cast<const uint4*>(a);
    const uint4* pb = reinterpret_cast<const uint4*>(b);
    const int nch = n / (int)(16 / sizeof(T));
    float acc[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) acc[u] = 0.f;
    for (int c0 = 0; c0 < nch; c0 += 16) {
#pragma unroll
        for (int half = 0; half < 16; half += 8) {
            const int c = c0 + half;
            uint4 x[8], y[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) { x[u] = pa[min(c + u, nch - 1)]; y[u] = pb[min(c + u, nch - 1)]; }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float v = chunk_dot<T>(x[u], y[u], acc[half + u]);
                acc[half + u] = c + u < nch ? v : acc[half + u];
            }
        }
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1)
#pragma unroll
        for (int u = 0; u < 16; u += 2 * o) acc[u] += acc[u + o];
    return acc[0];
}

// Makes a kernel hold all of these wave-uniform values at one point, so that they are read together.  A sample's offsets written one
// after the other are otherwise scheduled each behind the wait for the one before it: three trips to memory instead of one
// before a merge kernel knows its sample.
__device__ __forceinline__ void request_together(int& v0, int& v1, int& v2, int& v3) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(v0), "+s"(v1), "+s"(v2), "+s"(v3));
#endif
}
__device__ __forceinline__ void request_together(int& v0, int& v1, int& v2, int& v3, int& v4) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(v0), "+s"(v1), "+s"(v2), "+s"(v3), "+s"(v4));
#endif
}
__device__ __forceinline__ void request_together(int& v0, int& v1, int& v2, int& v3, int& v4, int& v5) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(v0), "+s"(v1), "+s"(v2), "+s"(v3), "+s"(v4), "+s"(v5));
#endif
}
__device__ __forceinline__ void request_together(int& v0, int& v1, int& v2, int& v3, int& v4, int& v5, int& v6) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(v0), "+s"(v1), "+s"(v2), "+s"(v3), "+s"(v4), "+s"(v5), "+s"(v6));
#endif
}
__device__ __forceinline__ void request_together(int& v0, int& v1, int& v2, int& v3, int& v4, int& v5, int& v6, int& v7) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(v0), "+s"(v1), "+s"(v2), "+s"(v3), "+s"(v4), "+s"(v5), "+s"(v6), "+s"(v7));
#endif
}

// ---- wave / block reductions ----------------------------------------------------------------
// Reductions over the 16 lanes of a DPP row (lanes 16 i .. 16 i + 15), every lane ends with the result.
// Four data-parallel-primitive steps inside the vector ALU (no LDS traffic): swap neighbours, swap
// pairs, mirror inside each half row, mirror the whole row.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float row16_max(float v) {
    v = fmaxf(v, dpp_move<0xB1>(v));     // quad_perm [1,0,3,2]
    v = fmaxf(v, dpp_move<0x4E>(v));     // quad_perm [2,3,0,1]
    v = fmaxf(v, dpp_move<0x141>(v));    // row_half_mirror
    v = fmaxf(v, dpp_move<0x140>(v));    // row_mirror
    return v;
}
__device__ __forceinline__ float row16_sum(float v) {
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    v += dpp_move<0x141>(v);
    v += dpp_move<0x140>(v);
    return v;
}
// The four lanes (l, l ^ 16, l ^ 32, l ^ 48): after the swap of halves of two copies the two results hold {own, partner}.
template <typename F>
__device__ __forceinline__ float quad_combine(float v, F&& f) {
#if defined(__HIP_DEVICE_COMPILE__)
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = f(__uint_as_float(r[0]), __uint_as_float(r[1]));
    r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return f(__uint_as_float(r[0]), __uint_as_float(r[1]));
#else
    return v;
#endif
}
// All 64 lanes.  The sum combines lanes 32, 16, 8, 4, 2 and 1 apart, in this order (near-ties of two cosines go by the last bits of the
// norms): rotations by 8 and 4 inside a row of 16 are what 8 and 4 apart are, once the lanes 8 apart agree.
__device__ __forceinline__ float wave_sum(float v) {
    v = quad_combine(v, [](float a, float b) { return a + b; });
    v += dpp_move<0x128>(v);             // row_ror:8
    v += dpp_move<0x124>(v);             // row_ror:4
    v += dpp_move<0x4E>(v);
    v += dpp_move<0xB1>(v);
    return v;
}
__device__ __forceinline__ float wave_max(float v) { return quad_combine(row16_max(v), [](float a, float b) { return fmaxf(a, b); }); }

// Dot products of a row with `count` rows (at least one) that lie `stride` elements apart, up to 64 of them, by one wave: lane l gets the one
// with row wave_dots_row(l).  16 lanes to a row, so that a load takes in whole lines; all rows of a pass are requested at once, behind
// them the row `a`, whose place may be the last thing to be known.  (A row to a lane: every load touches 64 lines.)
// 64 rows span less than 4 GB (65535 heads of 256 float32 channels at most).
__device__ __forceinline__ int wave_dots_row(int lane) { return (lane & 15) * 4 + (lane >> 4); }
// Q rows `a`: the same rows with each of them.
template <typename T, int Q>
__device__ __forceinline__ void wave_row_dots(const T* const (&a)[Q], const T* __restrict__ rows, size_t stride, int count, int n, int lane, float (&r)[Q]) {
    const int l = lane & 15, g = lane >> 4, nch = n / (int)(16 / sizeof(T));
    const uint32_t step = (uint32_t)(stride * sizeof(T));
    const char* base = reinterpret_cast<const char*>(rows);
    float d[Q][16];
#pragma unroll
    for (int u = 0; u < 16; ++u)
#pragma unroll
        for (int q = 0; q < Q; ++q) d[q][u] = 0.f;
    for (int c0 = 0; c0 < nch; c0 += 16) {
        const uint32_t at = (uint32_t)min(c0 + l, nch - 1) * 16u;
        uint4 y[16], x[Q];
#pragma unroll
        for (int u = 0; u < 16; ++u) y[u] = *reinterpret_cast<const uint4*>(base + ((uint32_t)min(u * 4 + g, count - 1) * step + at));
#pragma unroll
        for (int q = 0; q < Q; ++q) x[q] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(a[q]) + at);
#pragma unroll
        for (int u = 0; u < 16; ++u)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const float v = chunk_dot<T>(x[q], y[u], d[q][u]);
                d[q][u] = c0 + l < nch ? v : d[q][u];
            }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        r[q] = 0.f;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const float v = row16_sum(d[q][u]);
            r[q] = l == u ? v : r[q];
        }
    }
}

#if defined(__HIP_DEVICE_COMPILE__)
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ int dpp_move_i(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, ROWS == 0xF); }
// inclusive prefix sum over the 64 lanes of a wave: inside rows of 16, then the last lane of row 0 (2) to row 1 (3), of row 1 to rows 2, 3
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += dpp_move_i<0x111>(v);
    v += dpp_move_i<0x112>(v);
    v += dpp_move_i<0x114>(v);
    v += dpp_move_i<0x118>(v);
    v += dpp_move_i<0x142, 0xA>(v);
    v += dpp_move_i<0x143, 0xC>(v);
    return v;
}
#endif

// Combine two (running max, running sum of exp2) pairs.  -inf max means "empty".
__device__ __forceinline__ void lse2_combine(float& m, float& z, float m2, float z2) {
    float mn = fmaxf(m, m2);
    float a = (m == -INFINITY) ? 0.f : z * exp2f(m - mn);
    float b = (m2 == -INFINITY) ? 0.f : z2 * exp2f(m2 - mn);
    m = mn; z = a + b;
}

// One rotary pair (a, b) turned by the angle with cosine c and sine s.  The fused multiply-adds are spelled out so
// that every kernel that rotates (the rotary kernel, the q | k | v projection's epilogue) rounds the same way.
__device__ __forceinline__ void rope_rotate(float a, float b, float c, float s, float& ra, float& rb) {
    ra = __builtin_fmaf(a, c, -(b * s));
    rb = __builtin_fmaf(b, c, a * s);
}

// (cos, sin) of the rotary angle p * theta^(-2c/dh), evaluated in double precision (positions reach the thousands, where a float32
// angle is already off by 1e-4) and rounded to float32.
__device__ __forceinline__ float2 rope_cos_sin(int p, int c, int dh, double log2_theta) {
    const double inv_freq = exp2(-2.0 * (double)c / (double)dh * log2_theta);
    double s, co;
    sincos((double)p * inv_freq, &s, &co);
    return make_float2((float)co, (float)s);
}

// The same with the hardware exponential (one instruction, about 1 ulp, results below the normal range flush to
// zero): for the MFMA kernels, whose workgroups combine hundreds of pairs each.
__device__ __forceinline__ void lse2_combine_fast(float& m, float& z, float m2, float z2) {
    float mn = fmaxf(m, m2);
    float a = (m == -INFINITY) ? 0.f : z * __builtin_amdgcn_exp2f(m - mn);
    float b = (m2 == -INFINITY) ? 0.f : z2 * __builtin_amdgcn_exp2f(m2 - mn);
    m = mn; z = a + b;
}

__host__ __device__ __forceinline__ int ceil_div(int a, int b) { return (a + b - 1) / b; }
__host__ __device__ __forceinline__ size_t align_up(size_t a, size_t b) { return (a + b - 1) / b * b; }

// host-side argument checks
inline bool aligned16(const void* p) { return (((uintptr_t)p) & 15u) == 0; }

// One-time set-up per device (raising a kernel's dynamic LDS limit): safe when several host threads enter
// the same entry point at once, and repeated for every device the library is used on.
struct PerDeviceOnce {
    static constexpr int MAX_DEVICES = 64;
    std::once_flag flag[MAX_DEVICES];
    bool ok[MAX_DEVICES] = {};
    template <typename Fn>
    bool run(Fn&& fn) {
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return false;
        std::call_once(flag[dev], [&] { ok[dev] = fn(); });
        return ok[dev];
    }
};
template <typename K>
inline bool raise_dynamic_lds(K kernel, int bytes) {
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess;
}

// ---- optional per-kernel timing (d3tom_profile_*): HIP events around each launch when enabled ----
namespace prof {
enum Kernel {
    IMP_STATS = 0, IMP_SCORES, IMP_FINISH, TOPK_SELECT, MERGE_NORMS, COS_ARGMAX, MERGE_ASSIGN, MERGE_SCATTER, ATTEND,
    UPDATE_DECIDERS, COS_REDUCE, LINEAR, RMSNORM, ROPE, STACK_META,
    NUM_KERNELS
};
extern bool g_enabled;
void mark_begin(int kernel, hipStream_t st);
void mark_end(int kernel, hipStream_t st);
struct Scope {
    int kernel; hipStream_t st;
    Scope(int k, hipStream_t s) : kernel(k), st(s) { if (g_enabled) mark_begin(k, s); }
    ~Scope() { if (g_enabled) mark_end(kernel, st); }
};
}  // namespace prof

#define D3TOM_LAUNCH_CHECK()                                         \
    do {                                                             \
        if (hipGetLastError() != hipSuccess) return D3TOM_ERR_DEVICE; \
    } while (0)

// launch one kernel (timed when profiling is on) and turn a rejected launch into a status
#define D3TOM_LAUNCH(KERNEL_ID, STREAM, ...)                         \
    do {                                                             \
        {                                                            \
            prof::Scope _scope(prof::KERNEL_ID, STREAM);             \
            __VA_ARGS__;                                             \
        }                                                            \
        D3TOM_LAUNCH_CHECK();                                        \
    } while (0)

}  // namespace d3tom
