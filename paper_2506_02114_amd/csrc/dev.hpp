// Device helpers shared by the library's kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.hpp"

namespace mlm {

// 2-D Morton interleave: bit b of i goes to bit 2b, bit b of j to bit 2b+1
__device__ __host__ inline uint64_t spread_bits(uint32_t v)
{
    uint64_t x = v;
    x = (x | (x << 16)) & 0x0000FFFF0000FFFFull;
    x = (x | (x << 8)) & 0x00FF00FF00FF00FFull;
    x = (x | (x << 4)) & 0x0F0F0F0F0F0F0F0Full;
    x = (x | (x << 2)) & 0x3333333333333333ull;
    x = (x | (x << 1)) & 0x5555555555555555ull;
    return x;
}

__device__ __host__ inline uint32_t compact_bits(uint64_t x)
{
    x &= 0x5555555555555555ull;
    x = (x | (x >> 1)) & 0x3333333333333333ull;
    x = (x | (x >> 2)) & 0x0F0F0F0F0F0F0F0Full;
    x = (x | (x >> 4)) & 0x00FF00FF00FF00FFull;
    x = (x | (x >> 8)) & 0x0000FFFF0000FFFFull;
    x = (x | (x >> 16)) & 0x00000000FFFFFFFFull;
    return (uint32_t)x;
}

__device__ __host__ inline uint64_t morton2(uint32_t i, uint32_t j)
{
    return spread_bits(i) | (spread_bits(j) << 1);
}

// square index of coordinate t at the finest level: floor((t + L0) * 2^KEY_BITS / (2 L0)),
// where scale = 2^KEY_BITS / (2 L0) is a power of two (exact product of the rounded sum)
__device__ inline uint32_t fine_cell(double t, double L0, double scale)
{
    double u = floor((t + L0) * scale);
    const double top = (double)((1u << KEY_BITS) - 1);
    u = u < 0.0 ? 0.0 : (u > top ? top : u);
    return (uint32_t)u;
}

// the indices in sorted a[lo, hi) of the first keys >= v and >= w (v <= w):
// both searches in step, so that their loads are in flight together
__device__ inline void two_bounds_u64(const uint64_t *a, int32_t lo, int32_t hi, uint64_t v, uint64_t w, int32_t &i,
                                      int32_t &j)
{
    int32_t l0 = lo, l1 = lo;
    for (int32_t n0 = hi - lo; n0 > 0;) {   // n0: length of either range
        const int32_t half = n0 >> 1;
        const bool up0 = a[l0 + half] < v, up1 = a[l1 + half] < w;
        // (of an even length the upper part has half - 1 keys: its range is taken
        // one longer, with a key that is known not to be less, so both keep step)
        l0 += up0 ? half + 1 : 0;
        l1 += up1 ? half + 1 : 0;
        n0 = half;
        if (n0 > 0) {
            l0 = min(l0, hi - n0);
            l1 = min(l1, hi - n0);
        }
    }
    i = l0;
    j = l1;
}

// A colleague reference: >= 0 a node of the same level, -1 nothing (outside
// the root), <= -2 the leaf -(ref + 2) of a coarser level containing the square.
// Stars of square `sc` (level shift sh) inside the reference's range.
__device__ inline void ref_stars(int32_t ref, uint64_t sc, int sh, const int32_t *__restrict__ slo,
                                 const int32_t *__restrict__ shi, const uint64_t *__restrict__ keys, int32_t &s0,
                                 int32_t &s1)
{
    s0 = s1 = 0;
    if (ref >= 0) {
        s0 = slo[ref];
        s1 = shi[ref];
    } else if (ref <= -2) {
        const int32_t L = -ref - 2, a = slo[L], b = shi[L];
        two_bounds_u64(keys, a, b, sc << sh, (sc + 1) << sh, s0, s1);
    }
}

template <class T>
__device__ inline int64_t upper_bound_i64(const T *a, int64_t n, T v)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        int64_t mid = (lo + hi) >> 1;
        if (a[mid] <= v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// complex helpers on double2 (x = real, y = imaginary)
__device__ __host__ inline double2 cmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __host__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __host__ inline double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
__device__ inline double2 cinv(double2 a)
{
    double r = 1.0 / (a.x * a.x + a.y * a.y);
    return make_double2(a.x * r, -a.y * r);
}

// the same on float2, and the complex type of a real type
__device__ __host__ inline float2 cmul(float2 a, float2 b)
{
    return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __host__ inline float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ inline float2 cinv(float2 a)
{
    float r = __builtin_amdgcn_rcpf(a.x * a.x + a.y * a.y);
    return make_float2(a.x * r, -a.y * r);
}

// wavefront-level load balancing: a wavefront owns 64 segments (cells, large
// triangles or rows) with v items each; the exclusive scan of v over the
// lanes numbers the items, and an item finds its segment by binary lifting
// over the lanes' scan values (lane shuffles, no global memory)
__device__ inline int wave_excl_scan(int v, int lane, int &total)
{
    int incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    total = __shfl(incl, 63, 64);
    return incl - v;
}

// largest lane L with excl(L) <= x (excl non-decreasing over the lanes); the
// segment of item x has at least one item since excl(L + 1) > x
__device__ inline int wave_find(int excl, int x)
{
    int lo = 0;
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1) {
        const int e = __shfl(excl, lo + step, 64);
        if (e <= x) lo += step;
    }
    return lo;
}

// the rectangle [x0, x1] x [y0, y1] that holds the rays of a request, widened
// beyond the rounding of their positions
struct RayBox {
    double x0, x1, y0, y1;
};

RayBox ray_box(const Tree &T);

// centre, half-length and its inverse of the square `code` of level lev
__device__ inline void node_geom(uint64_t code, int lev, double L0, double &cx, double &cy, double &L,
                                 double &invL)
{
    uint32_t i = compact_bits(code), j = compact_bits(code >> 1);
    L = ldexp(L0, -lev);
    invL = 1.0 / L;   // exact: L is a power of two
    cx = -L0 + (double)(2 * (int64_t)i + 1) * L;
    cy = -L0 + (double)(2 * (int64_t)j + 1) * L;
}

// whether the square meets the rays' rectangle
__device__ inline bool in_box(uint64_t code, int lev, double L0, const RayBox &b)
{
    double cx, cy, L, invL;
    node_geom(code, lev, L0, cx, cy, L, invL);
    return cx + L >= b.x0 && cx - L <= b.x1 && cy + L >= b.y0 && cy - L <= b.y1;
}

template <class R> struct Cx;
template <> struct Cx<double> {
    using c2 = double2;
    using v4 = double4;
    __device__ __host__ static c2 make(double a, double b) { return make_double2(a, b); }
    __device__ __host__ static v4 make4(double a, double b, double c) { return make_double4(a, b, c, 0.0); }
};
template <> struct Cx<float> {
    using c2 = float2;
    using v4 = float4;
    __device__ __host__ static c2 make(float a, float b) { return make_float2(a, b); }
    __device__ __host__ static v4 make4(float a, float b, float c) { return make_float4(a, b, c, 0.0f); }
};

// the smaller and the larger of two numbers (of a number and a NaN the number),
// one instruction: fmin and fmax put another before it for every operand that was
// loaded, handed over between lanes or comes from another block of the program, to
// quieten signalling NaNs, which the instruction itself does (117 of the 2638
// instructions of k_ipm_fine; where a kernel is short of registers, as
// col_term's callers are, the compiler's own spill less and are kept)
__device__ inline double lesser(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline double greater(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline float lesser(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline float greater(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// a / b: FP64 division, or a times the FP32 hardware reciprocal (1 ulp)
__device__ inline double qdiv(double a, double b) { return a / b; }

// a / b for the near-field sum: the hardware reciprocal estimate refined by
// two Newton steps y <- y + y (1 - b y) (each doubles the correct bits), then
// one product; within a few ulp of the correctly rounded quotient, and
// non-finite (as the quotient) when b is 0
__device__ inline double near_div(double a, double b)
{
    double y = __builtin_amdgcn_rcp(b);
    y = fma(fma(-b, y, 1.0), y, y);
    y = fma(fma(-b, y, 1.0), y, y);
    return a * y;
}
__device__ inline float near_div(float a, float b) { return qdiv(a, b); }
__device__ inline float qdiv(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }

// a total to the host: the value, then its sequence number behind a
// system-scope fence, so a host thread that sees the number sees the value
__device__ inline void store_host_total(int64_t *total_host, int64_t v, int64_t seq)
{
    total_host[0] = v;
    __threadfence_system();
    __hip_atomic_store(total_host + 1, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace mlm
