// Device helpers shared by the streaming and Krylov kernels: indices, complex
// loads and stores of either precision, fixed-order block reductions.
#pragma once
#include "ppq_internal.hpp"

namespace ppq {

namespace {

constexpr int TB = 256;  // threads per block for streaming kernels
constexpr int PSTRIDE = 36;  // partial sums per block (Krylov values, adjoint parameters)
// Per-block partial sums are stored value-major, [value][block]: the one-block
// final reductions then read every value's partials as contiguous runs, one
// 1 KB line group per wavefront load, instead of one cache line per lane.
__device__ inline int64_t pidx(int64_t b, int i) { return (int64_t)i * RED_BLOCKS + b; }

__device__ inline int64_t gid() { return (int64_t)blockIdx.x * blockDim.x + threadIdx.x; }

inline unsigned nblocks(int64_t n, int tb = TB)
{
    int64_t b = (n + tb - 1) / tb;
    return (unsigned)(b < 1 ? 1 : b);
}

__device__ inline double2 ld2(const double2 *p, int64_t i) { return p[i]; }
__device__ inline double2 ld2(const float2 *p, int64_t i)
{
    float2 v = p[i];
    return make_double2((double)v.x, (double)v.y);
}
__device__ inline void st2(double2 *p, int64_t i, double2 v) { p[i] = v; }
__device__ inline void st2(float2 *p, int64_t i, double2 v) { p[i] = make_float2((float)v.x, (float)v.y); }
// Streaming forms for the Krylov basis: the sweeps and the recombination
// stream every earlier basis vector (more than the last-level cache holds),
// so their loads and the corrected vectors' stores carry the non-temporal
// hint and leave the cache to the product's tables and vectors.
typedef double nt_d2 __attribute__((ext_vector_type(2)));
typedef float nt_f2 __attribute__((ext_vector_type(2)));
__device__ inline double2 ld2nt(const double2 *p, int64_t i)
{
    const nt_d2 v = __builtin_nontemporal_load(reinterpret_cast<const nt_d2 *>(p) + i);
    return make_double2(v.x, v.y);
}
__device__ inline double2 ld2nt(const float2 *p, int64_t i)
{
    const nt_f2 v = __builtin_nontemporal_load(reinterpret_cast<const nt_f2 *>(p) + i);
    return make_double2((double)v.x, (double)v.y);
}
__device__ inline void st2nt(double2 *p, int64_t i, double2 v)
{
    const nt_d2 w = {v.x, v.y};
    __builtin_nontemporal_store(w, reinterpret_cast<nt_d2 *>(p) + i);
}
__device__ inline void st2nt(float2 *p, int64_t i, double2 v)
{
    const nt_f2 w = {(float)v.x, (float)v.y};
    __builtin_nontemporal_store(w, reinterpret_cast<nt_f2 *>(p) + i);
}
// the value a store of v into a C vector holds, without reading it back
__device__ inline double2 stored(const double2 *, double2 v) { return v; }
__device__ inline double2 stored(const float2 *, double2 v) { return make_double2((float)v.x, (float)v.y); }

// conj(a) * b accumulated
__device__ inline void cdot_acc(double2 &acc, double2 a, double2 b)
{
    acc.x = fma(a.x, b.x, fma(a.y, b.y, acc.x));
    acc.y = fma(a.x, b.y, fma(-a.y, b.x, acc.y));
}

template <int NV>
__device__ inline void block_reduce_store(double2 (&acc)[NV], double2 *partial)
{
    __shared__ double2 red[TB / 64][NV];
    int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        double2 v = acc[i];
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) {
            v.x += __shfl_xor(v.x, s, 64);
            v.y += __shfl_xor(v.y, s, 64);
        }
        if (lane == 0) red[w][i] = v;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double2 s = red[0][threadIdx.x];
        for (int ww = 1; ww < TB / 64; ++ww) {
            s.x += red[ww][threadIdx.x].x;
            s.y += red[ww][threadIdx.x].y;
        }
        partial[pidx(blockIdx.x, threadIdx.x)] = s;
    }
}

__device__ inline double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }

template <class R>
struct Cplx;
template <>
struct Cplx<double> {
    using T = double2;
    using V = double __attribute__((ext_vector_type(2)));
    __device__ static T make(double x, double y) { return make_double2(x, y); }
};
template <>
struct Cplx<float> {
    using T = float2;
    using V = float __attribute__((ext_vector_type(2)));
    __device__ static T make(float x, float y) { return make_float2(x, y); }
};

// A launch's description in device memory is read-only and its fields are wave-uniform: constant
// address space, so they come through the scalar cache.  The vectors and factors it
// names are global memory: a scalar base and a 32-bit lane offset per load.
typedef __attribute__((address_space(1))) const char gbyte;
template <class T>
__device__ inline T field(const T *p)
{
    return *(const __attribute__((address_space(4))) T *)p;
}
__device__ inline gbyte *global_base(const void *const *p)
{
    return (gbyte *)(const char *)field((const char *const *)p);
}
template <class T>
__device__ inline T at_byte(gbyte *base, uint32_t off)
{
    return *(__attribute__((address_space(1))) const T *)(base + off);
}

template <class V>
__device__ inline void cmul_acc(V &acc, V h, V v)
{
    acc.x = __builtin_elementwise_fma(h.x, v.x, __builtin_elementwise_fma(-h.y, v.y, acc.x));
    acc.y = __builtin_elementwise_fma(h.x, v.y, __builtin_elementwise_fma(h.y, v.x, acc.y));
}

// prod_{k in use} tab[k * nmax + i_k]: the diagonal factors of a product term
__device__ inline double diag_value(const GridDesc &g, gbyte *tab, int nmax, unsigned use, uint32_t key)
{
    double v = 1.0;
    for (int k = 0; k < g.D; ++k)
        if ((use >> k) & 1u)
            v *= at_byte<double>(tab + (int64_t)k * nmax * sizeof(double),
                                 ((key / g.stride[k]) % (uint32_t)g.n[k]) * (uint32_t)sizeof(double));
    return v;
}

}  // namespace

}  // namespace ppq
