// The operator product on fiber tables with every factor of one depth in one
// launch, on the matrix cores.
#include <algorithm>

#include "ppq_device.hpp"
#include "ppq_mfma.hpp"

namespace ppq {

namespace {

// A factor's pass as in the matrix-core form of ppq_hpsi.hip (a wavefront takes 16
// fibers, the union of their digits a window of 16 NT), with the result in a vector of
// the factor's own instead of added to y: so all factors of a depth share one launch
// and none waits for another's read-modify-write.  k_combine adds the vectors up,
// with the potential and the dots of a Krylov step.  Workgroups belong to one factor,
// hold its columns in LDS and go over their share of its fibers; NTM is the largest
// window of the launch's factors, which sets the registers.
// A pass by itself has 500-1400 wavefronts at 100K-600K functions, one or two per SIMD,
// and is bound by its chain of loads (13-33 us a pass where its products take 2-5 us).
// BATCH_NOTE
constexpr int BAB = 256;

template <class R, bool CX, int NT>
__device__ inline void batch_fibers(const BatchOp<R> *op, const GridDesc &g, int nmax, const uint32_t *keys, int np,
                                    const void *Hs, uint64_t m, uint32_t off, int ws, int lane)
{
    using V = typename Cplx<R>::V;
    using M = Mma<R>;
    constexpr int NK = 4 * NT;
    const int col = lane & 15, kr = lane >> 4;
    const int nin = field(&op->nin), add = field(&op->add);
    gbyte *x0 = global_base((const void *const *)&op->x[0]), *pi = global_base((const void *const *)&op->pi);
    __attribute__((address_space(1))) char *out =
        (__attribute__((address_space(1))) char *)field((char *const *)&op->out);
    uint32_t at[NK];  // byte offsets of the members the lane holds
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
        const int d = ws + 16 * (kb >> 2) + M::row(kr, kb & 3);
        uint32_t pos = 0;
        if ((m >> d) & 1ull) {
            pos = off + (uint32_t)__popcll(m & ((1ull << d) - 1ull));
            if (pi) pos = at_byte<uint32_t>(pi, pos * (uint32_t)sizeof(uint32_t));
        }
        at[kb] = pos;
    }
    V xin[NK];
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
        const int d = ws + 16 * (kb >> 2) + M::row(kr, kb & 3);
        xin[kb] = V{0, 0};
        if ((m >> d) & 1ull) xin[kb] = *(__attribute__((address_space(1))) const V *)(x0 + (uint64_t)at[kb] * sizeof(V));
    }
    if (CX && nin > 1) {
        auto weight = [&](int i) {
            V c;
            c.x = field((const R *)&op->c[i].x);
            c.y = field((const R *)&op->c[i].y);
            return c;
        };
        const V c0 = weight(0);
#pragma unroll
        for (int kb = 0; kb < NK; ++kb) {
            V v = V{0, 0};
            cmul_acc(v, c0, xin[kb]);
            xin[kb] = v;
        }
        for (int q = 1; q < nin; ++q) {
            gbyte *xq = global_base((const void *const *)&op->x[q]);
            const V c = weight(q);
#pragma unroll
            for (int k0 = 0; k0 < NK; k0 += 4) {
                V v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int d = ws + 16 * (k0 >> 2) + M::row(kr, u);
                    v[u] = V{0, 0};
                    if ((m >> d) & 1ull)
                        v[u] = *(__attribute__((address_space(1))) const V *)(xq + (uint64_t)at[k0 + u] * sizeof(V));
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) cmul_acc(xin[k0 + u], c, v[u]);
            }
        }
    }
    typename M::V4 accr[NT], acci[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        accr[t] = typename M::V4{0, 0, 0, 0};
        acci[t] = typename M::V4{0, 0, 0, 0};
    }
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
        const int j = ws + 16 * (kb >> 2) + M::row(kr, kb & 3);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int hi = j * np + ws + 16 * t + col;
            if (CX) {
                const V h = reinterpret_cast<const V *>(Hs)[hi];
                accr[t] = M::op(h.x, xin[kb].x, accr[t]);
                acci[t] = M::op(h.x, xin[kb].y, acci[t]);
                accr[t] = M::op(-h.y, xin[kb].y, accr[t]);
                acci[t] = M::op(h.y, xin[kb].x, acci[t]);
            } else {
                const R h = reinterpret_cast<const R *>(Hs)[hi];
                accr[t] = M::op(h, xin[kb].x, accr[t]);
                acci[t] = M::op(h, xin[kb].y, acci[t]);
            }
        }
    }
    const int scaled = CX ? field(&op->scaled) : 0;
    V cs = V{1, 0};
    unsigned use = 0;
    gbyte *diag = nullptr;
    if (scaled) {
        cs.x = field((const R *)&op->c[0].x);
        cs.y = field((const R *)&op->c[0].y);
        use = field(&op->use);
        diag = global_base((const void *const *)&op->diag);
    }
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
        const int d = ws + 16 * (kb >> 2) + M::row(kr, kb & 3);
        if (!((m >> d) & 1ull)) continue;
        V v;
        v.x = accr[kb >> 2][kb & 3];
        v.y = acci[kb >> 2][kb & 3];
        if (scaled) {
            // the term's coefficient and its diagonal factors (see ppq_grid.hip)
            const R w = use ? (R)diag_value(g, diag, nmax, use, keys[at[kb]]) : R(1);
            const V a = v;
            v.x = (cs.x * a.x - cs.y * a.y) * w;
            v.y = (cs.x * a.y + cs.y * a.x) * w;
        }
        __attribute__((address_space(1))) V *o = (__attribute__((address_space(1))) V *)(out + (uint64_t)at[kb] * sizeof(V));
        if (add) {
            const V q = *o;
            v.x += q.x;
            v.y += q.y;
        }
        *o = v;
    }
}

// The launch's description is the kernel's first argument: read from the argument
// segment itself, whose fields are wave-uniform.
template <class R, bool GENERAL, int NTM>
__global__ __launch_bounds__(BAB, NTM <= 2 ? 3 : 2) void k_batch(BatchStage<R> stage, GridDesc g, const uint32_t *__restrict__ keys,
                                                                 const int *skip_if, int skip_j)
{
    using V = typename Cplx<R>::V;
    if (skip_if && skip_j >= *skip_if) return;
    extern __shared__ __align__(16) unsigned char smem[];
    (void)stage;
    const BatchStage<R> *st = (const BatchStage<R> *)(const char *)(__attribute__((address_space(4))) const char *)
                                  __builtin_amdgcn_kernarg_segment_ptr();
    const int lane = threadIdx.x & 63, col = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int o = 0;
    const int bid = blockIdx.x;
    while (bid >= field(&st->first[o + 1])) ++o;
    const BatchOp<R> *op = &st->op[o];
    const int b = bid - field(&st->first[o]), blocks = field(&st->first[o + 1]) - field(&st->first[o]);
    const int n = field(&op->n), np = (n + 15) & ~15;
    const bool cx = GENERAL && field(&op->kind) != GRID_REAL;
    // the factor's columns, np rows each, from its 64 x 64 padded form
    gbyte *H = global_base(&op->H);
    for (int i = threadIdx.x; i < np * np; i += BAB) {
        const uint32_t at = (uint32_t)(i / np) * 64u + (uint32_t)(i % np);
        if (cx) reinterpret_cast<V *>(smem)[i] = at_byte<V>(H, at * (uint32_t)sizeof(V));
        else reinterpret_cast<R *>(smem)[i] = at_byte<R>(H, at * (uint32_t)sizeof(R));
    }
    gbyte *masks = global_base((const void *const *)&op->mask), *offs = global_base((const void *const *)&op->off);
    const uint32_t nf = (uint32_t)field(&op->nf), ngroup = (nf + 15) / 16;
    __syncthreads();
    for (uint32_t grp = b * (BAB / 64) + w; grp < ngroup; grp += blocks * (BAB / 64)) {
        const uint32_t f = grp * 16 + col;
        uint64_t m = 0;
        uint32_t off = 0;
        if (f < nf) {
            m = at_byte<uint64_t>(masks, f * (uint32_t)sizeof(uint64_t));
            off = at_byte<uint32_t>(offs, f * (uint32_t)sizeof(uint32_t));
        }
        uint64_t wm = m;
#pragma unroll
        for (int s = 8; s >= 1; s >>= 1)
            wm |= ((uint64_t)__shfl_xor((uint32_t)(wm >> 32), s, 64) << 32) | __shfl_xor((uint32_t)wm, s, 64);
        // (the builtin returns an int: digit 31 is not to spread over the upper half)
        wm = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(wm >> 32)) << 32) |
             (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)wm);
        if (wm == 0) continue;
        const int wlo = __ffsll((unsigned long long)wm) - 1, width = 64 - __clzll((long long)wm) - wlo;
#define PPQ_TILE(CX, NT)                                                                              \
    {                                                                                                 \
        const int ws = wlo < np - 16 * (NT) ? wlo : np - 16 * (NT);                                   \
        batch_fibers<R, CX, NT>(op, g, field(&st->nmax), keys, np, smem, m, off, ws, lane);           \
    }
#define PPQ_WIDTH(CX)                                       \
    if (width <= 16) PPQ_TILE(CX, 1)                         \
    else if (NTM == 2 || width <= 32) PPQ_TILE(CX, 2)        \
    else if (NTM == 3 || width <= 48) PPQ_TILE(CX, NTM < 3 ? 2 : 3) \
    else PPQ_TILE(CX, NTM)
        if constexpr (GENERAL) {
            if (cx) {
                PPQ_WIDTH(true)
            } else {
                PPQ_WIDTH(false)
            }
        } else {
            PPQ_WIDTH(false)
        }
#undef PPQ_WIDTH
#undef PPQ_TILE
    }
}

// y_p = V_p x_p + the factors' vectors at the point (+ the terms without dense
// factors).  NV >= 0: with the partial sums of <v_i|y> for i < NV and <q|y> (q the
// product's input); NV < 0: none.  Streams ny + 3 + NV vectors.
template <class R, int NV>
__global__ __launch_bounds__(TB, 2) void k_combine(BatchSum<R> ts, GridDesc g, const uint32_t *__restrict__ keys, int64_t n,
                                                   const typename Cplx<R>::T *x, const R *V, typename Cplx<R>::T *y,
                                                   const typename Cplx<R>::T *Vb, int64_t ld, double2 *partial,
                                                   const int *skip_if, int skip_j)
{
    using C = typename Cplx<R>::T;
    if (skip_if && skip_j >= *skip_if) return;
    constexpr int NA = NV >= 0 ? NV + 1 : 1;
    double2 acc[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) acc[i] = make_double2(0.0, 0.0);
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) {
        const uint32_t key = ts.ndiag ? keys[p] : 0u;
        C v[BATCH_SUMS];
#pragma unroll
        for (int i = 0; i < BATCH_SUMS; ++i)
            if (i < ts.ny) v[i] = ts.y[i][p];
        const C xv = x[p];
        C s = v[0];
#pragma unroll
        for (int i = 1; i < BATCH_SUMS; ++i) {
            if (i < ts.ny) {
                s.x += v[i].x;
                s.y += v[i].y;
            }
        }
        if (V) {
            const R pot = V[p];
            s.x = fma(pot, xv.x, s.x);
            s.y = fma(pot, xv.y, s.y);
        }
        for (int i = 0; i < ts.ndiag; ++i) {
            const R w = ts.use[i] ? (R)diag_value(g, (gbyte *)(const char *)ts.diag[i], ts.nmax, ts.use[i], key) : R(1);
            s.x += (ts.c[i].x * xv.x - ts.c[i].y * xv.y) * w;
            s.y += (ts.c[i].x * xv.y + ts.c[i].y * xv.x) * w;
        }
        y[p] = s;
        if constexpr (NV >= 0) {
            const double2 sd = make_double2((double)s.x, (double)s.y);
#pragma unroll
            for (int i = 0; i < NV; ++i) cdot_acc(acc[i], ld2(Vb, (int64_t)i * ld + p), sd);
            cdot_acc(acc[NA - 1], make_double2((double)xv.x, (double)xv.y), sd);
        }
    }
    if constexpr (NV >= 0) block_reduce_store<NA>(acc, partial);
}

}  // namespace

template <class R>
void batch_launch(BatchStage<R> &st, const GridDesc &g, const uint32_t *keys, const int *skip_if, int skip_j, hipStream_t s)
{
    if (st.nop <= 0) return;
    // BATCH_BLOCKS workgroups, shared out by the factors' fibers (at least one
    // group of 16 per wavefront)
    int nmax = 0;
    bool general = false;
    double work = 0.0;
    for (int o = 0; o < st.nop; ++o) {
        nmax = std::max(nmax, st.op[o].n);
        general = general || st.op[o].kind != GRID_REAL;
        work += (double)st.op[o].nf * (1 + st.op[o].nin);
    }
    st.first[0] = 0;
    for (int o = 0; o < st.nop; ++o) {
        const int64_t most = (st.op[o].nf + BAB / 4 - 1) / (BAB / 4);
        int64_t b = (int64_t)(BATCH_BLOCKS * ((double)st.op[o].nf * (1 + st.op[o].nin) / std::max(work, 1.0)) + 0.5);
        b = std::max<int64_t>(1, std::min(b, most));
        st.first[o + 1] = st.first[o] + (int)b;
    }
    const int np = (nmax + 15) & ~15;
    const size_t lds = (size_t)np * np * (general ? 2 : 1) * sizeof(R);
    const dim3 grid(st.first[st.nop]), block(BAB);
#define L(G, N) hipLaunchKernelGGL((k_batch<R, G, N>), grid, block, lds, s, st, g, keys, skip_if, skip_j)
    if (general) {
        if (np <= 32) L(true, 2);
        else if (np <= 48) L(true, 3);
        else L(true, 4);
    } else {
        if (np <= 32) L(false, 2);
        else if (np <= 48) L(false, 3);
        else L(false, 4);
    }
#undef L
}

template <class R>
int batch_combine(const BatchSum<R> &ts, const GridDesc &g, const uint32_t *keys, int64_t n, const typename GridOp<R>::C *x,
                 const R *V, typename GridOp<R>::C *y, int dots, const typename GridOp<R>::C *Vb, int64_t ld,
                 double2 *partial, const int *skip_if, int skip_j, hipStream_t s)
{
    if (n <= 0) return 0;
    const int nb = kry_blocks(n);
#define CALL(NV)                                                                                                      \
    hipLaunchKernelGGL((k_combine<R, NV>), dim3(nb), dim3(TB), 0, s, ts, g, keys, n, x, V, y, Vb, ld, partial, skip_if, \
                       skip_j)
    switch (dots) {
    case 0: CALL(-1); break;
    case 1: CALL(0); break;
    case 2: CALL(1); break;
    case 3: CALL(2); break;
    case 4: CALL(3); break;
    case 5: CALL(4); break;
    case 6: CALL(5); break;
    case 7: CALL(6); break;
    case 8: CALL(7); break;
    case 9: CALL(8); break;
    case 10: CALL(9); break;
    case 11: CALL(10); break;
    case 12: CALL(11); break;
    case 13: CALL(12); break;
    case 14: CALL(13); break;
    case 15: CALL(14); break;
    default: CALL(15); break;
    }
#undef CALL
    return dots ? nb : 0;
}

#define PPQ_INST(R)                                                                                                   \
    template void batch_launch<R>(BatchStage<R> &, const GridDesc &, const uint32_t *, const int *, int, hipStream_t); \
    template int batch_combine<R>(const BatchSum<R> &, const GridDesc &, const uint32_t *, int64_t,                   \
                                  const typename GridOp<R>::C *, const R *, typename GridOp<R>::C *, int,             \
                                  const typename GridOp<R>::C *, int64_t, double2 *, const int *, int, hipStream_t);
PPQ_INST(double)
PPQ_INST(float)
#undef PPQ_INST

}  // namespace ppq
