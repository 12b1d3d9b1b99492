// FP64 3x3 complex matrices in registers, loaded from and stored to
// site-planar fields (nine planes, element (i, j) in plane 3i + j; the
// argument V of ld / st is the plane stride, SmearGeom::P), and the lattice
// shifts the link kernels use.
#pragma once
#include <hip/hip_runtime.h>

#include "smear.h"

namespace hisq {
namespace su3 {

struct M3 {
    double2 e[9];
};

__device__ __forceinline__ M3 ld(const double2 *__restrict__ f, size_t V, long long s)
{
    M3 m;
#pragma unroll
    for (int i = 0; i < 9; i++) m.e[i] = f[i * V + s];
    return m;
}

// Stores are non-temporal: the passes write as many bytes as they read or
// more (pass 1 four times as many), and write-allocated lines would push the
// neighbour links the next sites reuse out of L2.  Every stored field is read
// again only by a later launch.
typedef double nt_double2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void st(double2 *__restrict__ f, size_t V, long long s, const M3 &m)
{
#pragma unroll
    for (int i = 0; i < 9; i++) {
        const nt_double2 v = {m.e[i].x, m.e[i].y};
        __builtin_nontemporal_store(v, reinterpret_cast<nt_double2 *>(f + i * V + s));
    }
}

// The same accesses through buffer resources, for the staple passes: a field's
// base and the plane offsets live in scalar registers and a lane supplies one
// 32-bit byte offset per site, where 64-bit per-lane addresses of 9 planes a
// matrix took a fifth of the vector instructions and, hoisted out of the site
// loops, enough registers to spill.  `f` must be the same for the whole
// wavefront.  Two resources per field, planes 0-4 and 5-8, of 2^32 - 1 bytes:
// the last plane of the first starts 64 P bytes into it and a lane adds up to
// 16 P, so P has to stay below 2^32 / 80 sites (BUF_MAX_P; the range check may
// count the scalar plane offset with the lane's, and would then drop what lies
// beyond).  The entry points that use these keep at least 51 fields (144 P
// bytes each), so memory ends first, or check P.
static_assert(5 * 16 * BUF_MAX_P <= 0xffffffffLL, "planes 0-4 of a field lie in one resource");

typedef unsigned int b128 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const double2 *f, size_t V, int half)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)(f + (half ? 5 * V : 0)), (short)0, -1, 0x00020000);
}

template <int AUX> __device__ __forceinline__ M3 ldb_aux(const double2 *f, size_t V, int s)
{
    M3 m;
    const unsigned pb = (unsigned)V * 16u;
#pragma unroll
    for (int i = 0; i < 9; i++)
        m.e[i] = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(
                                                 plane_rsrc(f, V, i >= 5), (int)((unsigned)s * 16u),
                                                 (int)((unsigned)(i >= 5 ? i - 5 : i) * pb), AUX));
    return m;
}
__device__ __forceinline__ M3 ldb(const double2 *f, size_t V, int s) { return ldb_aux<0>(f, V, s); }
__device__ __forceinline__ M3 ldb_nt(const double2 *f, size_t V, int s) { return ldb_aux<2>(f, V, s); }

__device__ __forceinline__ void stb(double2 *f, size_t V, int s, const M3 &m)
{
    const unsigned pb = (unsigned)V * 16u;
#pragma unroll
    for (int i = 0; i < 9; i++)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(b128, m.e[i]), plane_rsrc(f, V, i >= 5),
                                               (int)((unsigned)s * 16u), (int)((unsigned)(i >= 5 ? i - 5 : i) * pb), 2);
}

// The loads written before this are issued before the products after it: the
// scheduler would otherwise trade them for registers and leave two matrices in
// flight where six fit.
__device__ __forceinline__ void loads_first() { __builtin_amdgcn_sched_barrier(0); }

// c = a b
__device__ __forceinline__ M3 mul_nn(const M3 &a, const M3 &b)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const double2 x = a.e[3 * i + k], y = b.e[3 * k + j];
                re = __builtin_fma(x.x, y.x, re);
                re = __builtin_fma(-x.y, y.y, re);
                im = __builtin_fma(x.x, y.y, im);
                im = __builtin_fma(x.y, y.x, im);
            }
            c.e[3 * i + j] = make_double2(re, im);
        }
    return c;
}

// c = a b^+
__device__ __forceinline__ M3 mul_na(const M3 &a, const M3 &b)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const double2 x = a.e[3 * i + k], y = b.e[3 * j + k];
                re = __builtin_fma(x.x, y.x, re);
                re = __builtin_fma(x.y, y.y, re);
                im = __builtin_fma(x.y, y.x, im);
                im = __builtin_fma(-x.x, y.y, im);
            }
            c.e[3 * i + j] = make_double2(re, im);
        }
    return c;
}

// c = a^+ b
__device__ __forceinline__ M3 mul_an(const M3 &a, const M3 &b)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            double re = 0.0, im = 0.0;
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const double2 x = a.e[3 * k + i], y = b.e[3 * k + j];
                re = __builtin_fma(x.x, y.x, re);
                re = __builtin_fma(x.y, y.y, re);
                im = __builtin_fma(x.x, y.y, im);
                im = __builtin_fma(-x.y, y.x, im);
            }
            c.e[3 * i + j] = make_double2(re, im);
        }
    return c;
}

// acc += c m
__device__ __forceinline__ void axpy(M3 &acc, double c, const M3 &m)
{
#pragma unroll
    for (int i = 0; i < 9; i++)
        acc.e[i] = make_double2(__builtin_fma(c, m.e[i].x, acc.e[i].x), __builtin_fma(c, m.e[i].y, acc.e[i].y));
}

__device__ __forceinline__ int wrap(int v, int L)
{
    v -= v >= L ? L : 0;
    v -= v >= L ? L : 0;
    v += v < 0 ? L : 0;
    v += v < 0 ? L : 0;
    return v;
}

// site x + k * dir, for x's coordinate xd along dir (|k| <= 2 L)
template <class I> __device__ __forceinline__ I shift(I s, int xd, int S, int L, int k)
{
    return s + (I)(wrap(xd + k, L) - xd) * S;
}

__device__ __forceinline__ int pick(const int v[4], int d)
{
    return d == 0 ? v[0] : d == 1 ? v[1] : d == 2 ? v[2] : v[3];
}

// a^+
__device__ __forceinline__ M3 dag(const M3 &a)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) c.e[3 * i + j] = make_double2(a.e[3 * j + i].x, -a.e[3 * j + i].y);
    return c;
}

// a + b
__device__ __forceinline__ M3 add(const M3 &a, const M3 &b)
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 9; i++) c.e[i] = make_double2(a.e[i].x + b.e[i].x, a.e[i].y + b.e[i].y);
    return c;
}

__device__ __forceinline__ M3 zero3()
{
    M3 c;
#pragma unroll
    for (int i = 0; i < 9; i++) c.e[i] = make_double2(0.0, 0.0);
    return c;
}

}  // namespace su3
}  // namespace hisq
