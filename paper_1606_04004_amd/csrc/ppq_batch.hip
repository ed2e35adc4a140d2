// The operator product on fiber tables with every factor of one depth in one
// launch, on the matrix cores.
#include <algorithm>

#include "ppq_device.hpp"
#include "ppq_mfma.hpp"

namespace ppq {

namespace {

// A factor's pass as in the matrix-core form of ppq_hpsi.hip (a wavefront takes 16
// fibers), but over the digits that the fibers' union holds, compressed to 16 NT, not
// over a window from its first to its last (a lattice's digits count cells and
// momenta, so its fibers have gaps: at 563K functions of 6 x 8 lattices the window
// averages 40 digits, a fiber's members 15), and with the result in a vector of the
// factor's own instead of added to y: so all factors of a depth share one launch
// and none waits for another's read-modify-write.  k_combine adds the vectors up,
// with the potential and the dots of a Krylov step.  Workgroups belong to one factor,
// hold its columns in LDS and go over their share of its fibers; 16 NTM is the longest
// of the launch's factors, which sets the registers.
// A pass by itself has 500-1400 wavefronts at 100K-600K functions, one or two per SIMD,
// and is bound by its chain of loads (13-33 us a pass where its products take 2-5 us).
// Here the chip holds as many workgroups as fit, each wavefront has the next group's
// masks on their way while it contracts the current one, and what bounds a launch is
// the gathers' latency and, with complex factors, the matrix cores.  Measured (FP64):
// a product of the 4D lattice at 563K functions 150-170 us by card (268-319 in passes; 207
// over windows of the union, without the look ahead and with 1024 workgroups at any
// register count),
// 4D at 74K 15 us (61), 6D quartic at 781K 57 us (81).
constexpr int BAB = 256;
// wavefronts per SIMD that the registers of a window allow (workgroups per CU;
// complex factors of three tiles spill a few)
constexpr int batch_waves(bool f64, int ntm)
{
    if (!f64) return ntm <= 2 ? 5 : ntm == 3 ? 4 : 3;
    return ntm <= 2 ? 4 : ntm == 3 ? 3 : 2;
}

template <class R, bool CX, int NT>
__device__ inline void batch_fibers(const BatchOp<R> *op, const GridDesc &g, int nmax, const uint32_t *keys, int np,
                                    const void *Hs, uint64_t m, uint32_t off, const uint8_t *list, int lane)
{
    using V = typename Cplx<R>::V;
    using M = Mma<R>;
    constexpr int NK = 4 * NT;
    const int col = lane & 15, kr = lane >> 4;
    const int nin = field(&op->nin), add = field(&op->add);
    gbyte *x0 = global_base((const void *const *)&op->x[0]), *pi = global_base((const void *const *)&op->pi);
    __attribute__((address_space(1))) char *out =
        (__attribute__((address_space(1))) char *)field((char *const *)&op->out);
    // list[i]: the i-th digit of the union, 64 past its end; the positions of the
    // lane's entries, and which of them are members
    uint32_t at[NK];
    unsigned member = 0;
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
        const int d = list[16 * (kb >> 2) + M::row(kr, kb & 3)];
        uint32_t pos = 0;
        if (d < 64 && ((m >> d) & 1ull)) {
            member |= 1u << kb;
            pos = off + (uint32_t)__popcll(m & ((1ull << d) - 1ull));
            if (pi) pos = at_byte<uint32_t>(pi, pos * (uint32_t)sizeof(uint32_t));
        }
        at[kb] = pos;
    }
    V xin[NK];
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
        xin[kb] = V{0, 0};
        if (member & (1u << kb)) xin[kb] = *(__attribute__((address_space(1))) const V *)(x0 + (uint64_t)at[kb] * sizeof(V));
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
            constexpr int CH = sizeof(R) == 4 ? NK : NT <= 2 ? 8 : 4;  // loads in flight that the registers allow
#pragma unroll
            for (int k0 = 0; k0 < NK; k0 += CH) {
                V v[CH];
#pragma unroll
                for (int u = 0; u < CH; ++u) {
                    const int kb = k0 + u;
                    if (kb >= NK) break;
                    v[u] = V{0, 0};
                    if (member & (1u << (kb % NK)))
                        v[u] = *(__attribute__((address_space(1))) const V *)(xq + (uint64_t)at[kb] * sizeof(V));
                }
#pragma unroll
                for (int u = 0; u < CH; ++u)
                    if (k0 + u < NK) cmul_acc(xin[k0 + u], c, v[u]);
            }
        }
    }
    typename M::V4 accr[NT], acci[NT];
    int rowd[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        rowd[t] = list[16 * t + col] & 63;
        accr[t] = typename M::V4{0, 0, 0, 0};
        acci[t] = typename M::V4{0, 0, 0, 0};
    }
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
        const int j = (list[16 * (kb >> 2) + M::row(kr, kb & 3)] & 63) * np;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int hi = j + rowd[t];
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
    double2 cs = make_double2(1.0, 0.0);
    unsigned use = 0;
    gbyte *diag = nullptr;
    if (scaled) {
        cs.x = field(&op->scale.x);
        cs.y = field(&op->scale.y);
        use = field(&op->use);
        diag = global_base((const void *const *)&op->diag);
    }
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
        if (!(member & (1u << kb))) continue;
        V v;
        v.x = accr[kb >> 2][kb & 3];
        v.y = acci[kb >> 2][kb & 3];
        __attribute__((address_space(1))) V *o = (__attribute__((address_space(1))) V *)(out + (uint64_t)at[kb] * sizeof(V));
        if (scaled) {
            // the term's coefficient and its diagonal factors (see ppq_grid.hip): in FP64,
            // rounded once, with the sum
            const double ax = v.x, ay = v.y;
            double tx = cs.x * ax - cs.y * ay, ty = cs.x * ay + cs.y * ax;
            if (use) {
                const double w = diag_value(g, diag, nmax, use, keys[at[kb]]);
                tx *= w;
                ty *= w;
            }
            if (add) {
                const V q = *o;
                tx += q.x;
                ty += q.y;
            }
            v.x = (R)tx;
            v.y = (R)ty;
        } else if (add) {
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
__global__ __launch_bounds__(BAB, batch_waves(sizeof(R) == 8, NTM)) void k_batch(BatchStage<R> stage, GridDesc g, const uint32_t *__restrict__ keys,
                                                                 const int *skip_if, int skip_j)
{
    using V = typename Cplx<R>::V;
    if (skip_if && skip_j >= *skip_if) return;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint8_t list[BAB / 64][64];
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
    // the first fibers' tables are on their way while the factor is staged, and
    // each next group's while its predecessor is contracted
    gbyte *masks = global_base((const void *const *)&op->mask), *offs = global_base((const void *const *)&op->off);
    const uint32_t nf = (uint32_t)field(&op->nf), ngroup = (nf + 15) / 16, hop = blocks * (BAB / 64);
    uint64_t mnext = 0;
    uint32_t onext = 0;
    auto fetch = [&](uint32_t grp) {
        const uint32_t f = grp * 16 + col;
        const bool in = grp < ngroup && f < nf;
        mnext = in ? at_byte<uint64_t>(masks, f * (uint32_t)sizeof(uint64_t)) : 0ull;
        onext = in ? at_byte<uint32_t>(offs, f * (uint32_t)sizeof(uint32_t)) : 0u;
    };
    fetch(b * (BAB / 64) + w);
    // the factor's columns, np rows each, from its 64 x 64 padded form
    gbyte *H = global_base(&op->H);
    for (int i = threadIdx.x; i < np * np; i += BAB) {
        const uint32_t at = (uint32_t)(i / np) * 64u + (uint32_t)(i % np);
        if (cx) reinterpret_cast<V *>(smem)[i] = at_byte<V>(H, at * (uint32_t)sizeof(V));
        else reinterpret_cast<R *>(smem)[i] = at_byte<R>(H, at * (uint32_t)sizeof(R));
    }
    __syncthreads();
    for (uint32_t grp = b * (BAB / 64) + w; grp < ngroup; grp += hop) {
        const uint64_t m = mnext;
        const uint32_t off = onext;
        fetch(grp + hop);
        uint64_t wm = m;
#pragma unroll
        for (int s = 8; s >= 1; s >>= 1)
            wm |= ((uint64_t)__shfl_xor((uint32_t)(wm >> 32), s, 64) << 32) | __shfl_xor((uint32_t)wm, s, 64);
        // (the builtin returns an int: digit 31 is not to spread over the upper half)
        wm = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(wm >> 32)) << 32) |
             (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)wm);
        if (wm == 0) continue;
        // the union's digits in order, in the wavefront's own LDS: lane d writes itself at
        // its rank among the digits present (absent: the end mark, behind them)
        const int count = __popcll(wm), below = __popcll(wm & ((1ull << lane) - 1ull));
        const bool here = (wm >> lane) & 1ull;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        list[w][here ? below : count + lane - below] = (uint8_t)(here ? lane : 64);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#define PPQ_TILE(CX, NT) batch_fibers<R, CX, NT>(op, g, field(&st->nmax), keys, np, smem, m, off, list[w], lane);
#define PPQ_COUNT(CX)                                          \
    if (count <= 16) PPQ_TILE(CX, 1)                            \
    else if (NTM == 2 || count <= 32) PPQ_TILE(CX, 2)           \
    else if (NTM == 3 || count <= 48) PPQ_TILE(CX, NTM < 3 ? 2 : 3) \
    else PPQ_TILE(CX, NTM)
        if constexpr (GENERAL) {
            if (cx) {
                PPQ_COUNT(true)
            } else {
                PPQ_COUNT(false)
            }
        } else {
            PPQ_COUNT(false)
        }
#undef PPQ_COUNT
#undef PPQ_TILE
    }
}

// y_p = V_p x_p + the factors' vectors at the point (+ the terms without dense
// factors).  NV >= 0: with the partial sums of <v_i|y> for i < NV and <q|y> (q the
// product's input); NV < 0: none.  Streams ny + 3 + NV vectors.  With terms without dense
// factors (WIDE) the sum is formed in FP64 and rounded once; for the factors' vectors alone
// that would cost 2-3% of an FP32 step (684 us and 702 on 1M functions in 4D) and spare
// a rounding each.
template <class R, int NV, bool WIDE>
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
        const double2 xd = make_double2((double)xv.x, (double)xv.y);
        C s = v[0];
        if constexpr (!WIDE) {
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
        } else {
            double2 t = make_double2((double)s.x, (double)s.y);
#pragma unroll
            for (int i = 1; i < BATCH_SUMS; ++i) {
                if (i < ts.ny) {
                    t.x += v[i].x;
                    t.y += v[i].y;
                }
            }
            if (V) {
                const double pot = V[p];
                t.x = fma(pot, xd.x, t.x);
                t.y = fma(pot, xd.y, t.y);
            }
            for (int i = 0; i < ts.ndiag; ++i) {
                const double w = ts.use[i] ? diag_value(g, (gbyte *)(const char *)ts.diag[i], ts.nmax, ts.use[i], key) : 1.0;
                t.x += (ts.c[i].x * xd.x - ts.c[i].y * xd.y) * w;
                t.y += (ts.c[i].x * xd.y + ts.c[i].y * xd.x) * w;
            }
            s = Cplx<R>::make(t.x, t.y);
        }
        y[p] = s;
        if constexpr (NV >= 0) {
            const double2 sd = make_double2((double)s.x, (double)s.y);
#pragma unroll
            for (int i = 0; i < NV; ++i) cdot_acc(acc[i], ld2(Vb, (int64_t)i * ld + p), sd);
            cdot_acc(acc[NA - 1], xd, sd);
        }
    }
    if constexpr (NV >= 0) block_reduce_store<NA>(acc, partial);
}

}  // namespace

template <class R>
void batch_launch(BatchStage<R> &st, const GridDesc &g, const uint32_t *keys, int64_t n, const int *skip_if, int skip_j,
                  hipStream_t s)
{
    if (st.nop <= 0) return;
    // as many workgroups as are resident at once (no more: the one too many would start
    // when the others end), at least one group of 16 fibers per wavefront, shared out by
    // what the factors take.  A fiber takes its own time and its digits': by fibers alone
    // a short dimension, which has many, kept the long ones short of workgroups (a product
    // in FP64, us: 64^4 x 3^2 756K 131, now 91; 64^2 x 8^3 793K 128, 70; shares rounded up
    // past the chip: 12^6 1.2M 95, 77, a 48^4 lattice 1.8M 374, 324)
    auto weight = [&](const BatchOp<R> &op) { return (6.0 * op.nf + (double)n) * (1 + op.nin); };
    int nmax = 0;
    bool general = false;
    double work = 0.0;
    for (int o = 0; o < st.nop; ++o) {
        nmax = std::max(nmax, st.op[o].n);
        general = general || st.op[o].kind != GRID_REAL;
        work += weight(st.op[o]);
    }
    const int np = (nmax + 15) & ~15;
    const size_t lds = (size_t)np * np * (general ? 2 : 1) * sizeof(R);
    const int per_cu = std::min<int>(batch_waves(sizeof(R) == 8, std::max(np / 16, 2)), (int)(LDS_BYTES / (lds + BAB)));
    const double resident = (double)BATCH_CUS * std::max(per_cu, 1);
    st.first[0] = 0;
    for (int o = 0; o < st.nop; ++o) {
        const int64_t most = (st.op[o].nf + BAB / 4 - 1) / (BAB / 4);
        int64_t b = (int64_t)(resident * (weight(st.op[o]) / std::max(work, 1.0)));
        b = std::max<int64_t>(1, std::min(b, most));
        st.first[o + 1] = st.first[o] + (int)b;
    }
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
    const bool wide = ts.ndiag > 0;
#define CALL(NV)                                                                                                       \
    if (wide)                                                                                                          \
        hipLaunchKernelGGL((k_combine<R, NV, true>), dim3(nb), dim3(TB), 0, s, ts, g, keys, n, x, V, y, Vb, ld, partial, \
                           skip_if, skip_j);                                                                           \
    else                                                                                                               \
        hipLaunchKernelGGL((k_combine<R, NV, false>), dim3(nb), dim3(TB), 0, s, ts, g, keys, n, x, V, y, Vb, ld, partial, \
                           skip_if, skip_j)
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
    template void batch_launch<R>(BatchStage<R> &, const GridDesc &, const uint32_t *, int64_t, const int *, int,     \
                                  hipStream_t);                                                                       \
    template int batch_combine<R>(const BatchSum<R> &, const GridDesc &, const uint32_t *, int64_t,                   \
                                  const typename GridOp<R>::C *, const R *, typename GridOp<R>::C *, int,             \
                                  const typename GridOp<R>::C *, int64_t, double2 *, const int *, int, hipStream_t);
PPQ_INST(double)
PPQ_INST(float)
#undef PPQ_INST

}  // namespace ppq
