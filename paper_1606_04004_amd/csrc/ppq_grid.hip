// The operator product on grid vectors: for sets that are small against the
// chip, every 1D factor of a product in one launch per factor depth.
#include <algorithm>

#include "ppq_device.hpp"

namespace ppq {

namespace {

// A grid vector holds a set's values at their keys and zeros everywhere else, so
// a fiber's members are read at base + d * stride without any table of the set,
// absent ones as zeros.  One thread per output point sums its fibers' products
// over all digits; a workgroup takes 64 consecutive points of the sorted set and
// its wavefronts share out the digits of all factors (slices), whose partial sums
// meet in LDS.  Neighbouring lanes' points are neighbours on the grid, so the loads
// of a digit are runs of it (for the last dimension: a few fibers' same entries).
// Against one launch per dimension with a lane per fiber this trades the zeros
// read (n_k digits instead of the fiber's members) for one launch instead of D,
// D times the wavefronts, no read-modify-write of y, no fiber tables, and one load
// of latency instead of three dependent ones.  Bound by the L1's 64 bytes per
// clock on large sets, by launch and load latency on small ones.  Measured inside
// steps, one product: 5.8 us on 660 functions of 48^2 (two matrix-core passes and a
// dot before: 12.5), 8.5 us on a 24^4 set (four passes: 42), 23 us on 114K functions
// of 32^4 (50), 25 us with three general terms on 12K functions of a 3D grid (76).
constexpr int GU = 8;  // digits in flight per lane

// A wavefront's slice: digits [d0, d1) of one factor.  With product terms (GENERAL)
// its sum is returned in FP64, whatever the vectors: a term's coefficient and diagonal
// factors act in FP64 and a result is rounded once, when it is stored.
template <class R, bool GENERAL>
struct Slice {
    using V = typename Cplx<R>::V;
    using S = typename Cplx<typename std::conditional<GENERAL, double, R>::type>::V;
    gbyte *x[GENERAL ? 4 : 1], *H, *H2, *diag;
    V c[GENERAL ? 4 : 1];
    double2 scale;
    uint32_t st;
    unsigned use;
    int n, nb, kind, nin, scaled, d0, d1, nmax;

    __device__ void load(const GridStage<R> *s, int w)
    {
        const GridOp<R> *op = &s->op[field(&s->slice_op[w])];
        d0 = field(&s->d0[w]);
        d1 = field(&s->d1[w]);
        x[0] = global_base((const void *const *)&op->x[0]);
        H = global_base(&op->H);
        st = field(&op->stride);
        n = field(&op->n);
        nb = field(&op->nb);
        if (GENERAL) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[i % (GENERAL ? 4 : 1)] = global_base((const void *const *)&op->x[i]);
                V ci;
                ci.x = field((const R *)&op->c[i].x);
                ci.y = field((const R *)&op->c[i].y);
                c[i % (GENERAL ? 4 : 1)] = ci;
            }
            scale = make_double2(field(&op->scale.x), field(&op->scale.y));
            H2 = global_base(&op->H2);
            diag = global_base((const void *const *)&op->diag);
            use = field(&op->use);
            kind = field(&op->kind);
            nin = field(&op->nin);
            scaled = field(&op->scaled);
            nmax = field(&s->nmax);
        }
    }

    // the slice's sum for the point (out), and the second factor's (out2)
    __device__ void sum(const GridDesc &g, uint32_t key, S &out, S &out2) const
    {
        V acc = V{0, 0}, acc2 = acc;
        if (GENERAL && kind == GRID_DIAG) {
            acc = at_byte<V>(x[0], key * (uint32_t)sizeof(V));
        } else {
            const uint32_t dp = (key / st) % (uint32_t)n;
            const uint32_t lane0 = (key - dp * st) * (uint32_t)sizeof(V);  // the fiber's first entry
            const int64_t step = (int64_t)st * sizeof(V);                  // one digit on
            if (!GENERAL || kind == GRID_REAL) {
                for (int d = d0; d < d1; d += GU) {
                    V xv[GU];
                    R t[GU];
#pragma unroll
                    for (int u = 0; u < GU; ++u) {
                        const int i = d + u < d1 ? d + u : d0;
                        xv[u] = at_byte<V>(x[0] + i * step, lane0);
                        t[u] = at_byte<R>(H + (int64_t)i * nb * sizeof(R), dp * (uint32_t)sizeof(R));
                    }
#pragma unroll
                    for (int u = 0; u < GU; ++u) {
                        // past the slice's end the entry is another digit's, which may be infinite
                        const V v = d + u < d1 ? xv[u] : V{0, 0};
                        acc.x = __builtin_elementwise_fma(t[u], v.x, acc.x);
                        acc.y = __builtin_elementwise_fma(t[u], v.y, acc.y);
                    }
                }
            } else if (GENERAL) {
                constexpr int U = GU / 2;
                const int64_t hstep = (int64_t)nb * sizeof(V);
                const uint32_t hrow = dp * (uint32_t)sizeof(V);
                for (int d = d0; d < d1; d += U) {
                    V xv[U], h[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int i = d + u < d1 ? d + u : d0;
                        xv[u] = at_byte<V>(x[0] + i * step, lane0);
                        h[u] = at_byte<V>(H + i * hstep, hrow);
                    }
                    if (nin > 1) {
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            V v = V{0, 0};
                            cmul_acc(v, c[0], xv[u]);
                            xv[u] = v;
                        }
#pragma unroll
                        for (int q = 1; q < 4; ++q) {
                            if (q >= nin) break;
                            V xq[U];
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                const int i = d + u < d1 ? d + u : d0;
                                xq[u] = at_byte<V>(x[q % (GENERAL ? 4 : 1)] + i * step, lane0);
                            }
#pragma unroll
                            for (int u = 0; u < U; ++u) cmul_acc(xv[u], c[q % (GENERAL ? 4 : 1)], xq[u]);
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (d + u < d1) cmul_acc(acc, h[u], xv[u]);
                    if (H2) {
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int i = d + u < d1 ? d + u : d0;
                            h[u] = at_byte<V>(H2 + i * hstep, hrow);
                        }
#pragma unroll
                        for (int u = 0; u < U; ++u)
                            if (d + u < d1) cmul_acc(acc2, h[u], xv[u]);
                    }
                }
            }
        }
        if (GENERAL && scaled) {
            // the term's coefficient and its diagonal factors, which commute with the
            // dense factors of the other dimensions and with the truncation
            const double w = use ? diag_value(g, diag, nmax, use, key) : 1.0;
            const double vx = acc.x, vy = acc.y;
            out.x = (scale.x * vx - scale.y * vy) * w;
            out.y = (scale.x * vy + scale.y * vx) * w;
        } else {
            out.x = acc.x;
            out.y = acc.y;
        }
        out2.x = acc2.x;
        out2.y = acc2.y;
    }
};

// DOTS 0: none; 1: <x|y> of the product's input and result (wavefront 0's points,
// one partial per workgroup); 2: <v_i|y> for the nv basis vectors at Vb.
template <class R, bool GENERAL, int DOTS>
__global__ __launch_bounds__(1024) void k_grid(const GridStage<R> *stp, GridDesc g, const uint32_t *__restrict__ keys,
                                               int64_t n, const typename Cplx<R>::T *__restrict__ xg,
                                               const R *__restrict__ V, typename Cplx<R>::T *__restrict__ y, int accumulate,
                                               const int *skip_if, int skip_j, const typename Cplx<R>::T *__restrict__ Vb,
                                               int64_t ld, int nv, double2 *__restrict__ dotp)
{
    using C = typename Cplx<R>::T;
    if (skip_if && skip_j >= *skip_if) return;
    extern __shared__ __align__(16) unsigned char smem[];
    using Vec = typename Slice<R, GENERAL>::S;
    using S = decltype(Vec{}.x);
    const int lane = threadIdx.x & 63, W = blockDim.x >> 6;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ns = field(&stp->nslice), second = GENERAL ? field(&stp->second) : 0, nout = GENERAL ? field(&stp->nout) : 0;
    const int np = second ? 2 * ns : ns;
    Slice<R, GENERAL> sl;
    if (w < ns) sl.load(stp, w);
    Vec *parts = reinterpret_cast<Vec *>(smem);                  // [slice, second results][64]
    double2 *ys = reinterpret_cast<double2 *>(parts + np * 64);  // DOTS 2: the tile's y
    constexpr int NACC = DOTS == 2 ? (MAXM + 3) / 4 : 1;  // at least four wavefronts share the vectors
    double2 acc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i) acc[i] = make_double2(0.0, 0.0);
    for (int64_t t0 = (int64_t)blockIdx.x * 64; t0 < n; t0 += (int64_t)gridDim.x * 64) {
        const int64_t p = t0 + lane;
        const bool valid = p < n;
        const uint32_t key = valid ? keys[p] : 0u;
        if (w < ns) {
            Vec a, a2;
            sl.sum(g, key, a, a2);
            parts[w * 64 + lane] = a;
            if (second) parts[(ns + w) * 64 + lane] = a2;
        }
        __syncthreads();
        for (int f = w; f <= nout; f += W) {
            Vec v = Vec{0, 0};
            // the parts of result f, lowest first
            for (uint32_t m = GENERAL ? field(&stp->parts_of[f]) : (1u << ns) - 1u; m; m &= m - 1) {
                const Vec q = parts[(__ffs(m) - 1) * 64 + lane];
                v.x += q.x;
                v.y += q.y;
            }
            if (f > 0) {
                typename Cplx<R>::T *o = (typename Cplx<R>::T *)field((char *const *)&stp->out[f - 1]);
                if (valid) o[key] = Cplx<R>::make(v.x, v.y);
                continue;
            }
            if (GENERAL && !field(&stp->writes_y)) continue;
            if (valid) {
                const C xv = xg[key];
                if (V) {
                    const S pot = V[p];
                    v.x = fma(pot, (S)xv.x, v.x);
                    v.y = fma(pot, (S)xv.y, v.y);
                }
                if (accumulate) {
                    const C o = y[p];
                    v.x += o.x;
                    v.y += o.y;
                }
                const C r = Cplx<R>::make(v.x, v.y);
                y[p] = r;
                // the dots are those of the result as it is stored
                v.x = r.x;
                v.y = r.y;
                if (DOTS == 1)
                    cdot_acc(acc[0], make_double2((double)xv.x, (double)xv.y), make_double2((double)v.x, (double)v.y));
            }
            if (DOTS == 2) ys[lane] = make_double2((double)v.x, (double)v.y);
        }
        if (DOTS == 2) {
            __syncthreads();
            if (valid) {
                const double2 yv = ys[lane];
#pragma unroll
                for (int i = 0; i < NACC; ++i) {
                    const int q = w + i * W;
                    if (q < nv) cdot_acc(acc[i], ld2(Vb, (int64_t)q * ld + p), yv);
                }
            }
        }
        __syncthreads();
    }
    if (DOTS == 1 && w == 0) {
        double2 v = acc[0];
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) {
            v.x += __shfl_xor(v.x, s, 64);
            v.y += __shfl_xor(v.y, s, 64);
        }
        if (lane == 0) dotp[blockIdx.x] = v;
    }
    if (DOTS == 2) {
#pragma unroll
        for (int i = 0; i < NACC; ++i) {
            const int q = w + i * W;
            double2 v = acc[i];
#pragma unroll
            for (int s = 32; s >= 1; s >>= 1) {
                v.x += __shfl_xor(v.x, s, 64);
                v.y += __shfl_xor(v.y, s, 64);
            }
            if (lane == 0 && q < nv) dotp[pidx(blockIdx.x, q)] = v;
        }
    }
}

template <class C>
__global__ void k_grid_put(const uint32_t *keys, const C *x, int64_t n, C *xg)
{
    const int64_t p = gid();
    if (p < n) xg[keys[p]] = x[p];
}

template <class C>
__global__ void k_grid_clear(const uint32_t *keys, int64_t n, C *xg)
{
    const int64_t p = gid();
    if (p < n) xg[keys[p]] = C{0, 0};
}

}  // namespace

template <class R>
int grid_launch(const GridStage<R> *dev, const GridStage<R> &st, const GridDesc &g, const uint32_t *keys, int64_t n,
                const typename GridStage<R>::C *xg, const R *V, typename GridStage<R>::C *y, bool accumulate,
                const int *skip_if, int skip_j, int dots, const typename GridStage<R>::C *Vb, int64_t ld, int nv,
                double2 *dotp, hipStream_t s)
{
    if (n <= 0) return 0;
    // as many tiles per workgroup for all of them, at most GRID_BLOCKS workgroups
    const int64_t tiles = (n + 63) / 64, per = (tiles + GRID_BLOCKS - 1) / GRID_BLOCKS;
    const unsigned nb = (unsigned)((tiles + per - 1) / per);
    const int W = std::max(st.nslice, 4);
    const size_t lds = (size_t)st.nslice * (st.second ? 2 : 1) * 64 *
                           (st.general ? sizeof(double2) : sizeof(typename GridStage<R>::C)) +
                       (dots == 2 ? 64 * sizeof(double2) : 0);
#define L(G, DT)                                                                                                \
    hipLaunchKernelGGL((k_grid<R, G, DT>), dim3(nb), dim3(64 * W), lds, s, dev, g, keys, n, xg, V, y, (int)accumulate, \
                       skip_if, skip_j, Vb, ld, nv, dotp)
    if (st.general) {
        if (dots == 1) L(true, 1);
        else if (dots == 2) L(true, 2);
        else L(true, 0);
    } else {
        if (dots == 1) L(false, 1);
        else if (dots == 2) L(false, 2);
        else L(false, 0);
    }
#undef L
    return (int)nb;
}

template <class C>
void grid_put(const uint32_t *keys, const C *x, int64_t n, C *xg, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_grid_put<C>, dim3(nblocks(n)), dim3(TB), 0, s, keys, x, n, xg);
}
template <class C>
void grid_clear(const uint32_t *keys, int64_t n, C *xg, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_grid_clear<C>, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, xg);
}

#define PPQ_INST(R, C)                                                                                              \
    template int grid_launch<R>(const GridStage<R> *, const GridStage<R> &, const GridDesc &, const uint32_t *,     \
                                int64_t, const C *, const R *, C *, bool, const int *, int, int, const C *, int64_t, \
                                int, double2 *, hipStream_t);                                                       \
    template void grid_put<C>(const uint32_t *, const C *, int64_t, C *, hipStream_t);                              \
    template void grid_clear<C>(const uint32_t *, int64_t, C *, hipStream_t);
PPQ_INST(double, double2)
PPQ_INST(float, float2)
#undef PPQ_INST

}  // namespace ppq
