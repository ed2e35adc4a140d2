// Krylov kernels: the basis sweeps of the short-iterative Lanczos and Arnoldi
// steps with the step's scalars finalised in the next kernel's prologue, the
// small exponential and the recombination.
#include <algorithm>

#include "ppq_device.hpp"

namespace ppq {

namespace {

// ---- the step's scalars -------------------------------------------------------
// A sweep and a product each leave per-block partial sums.  The kernel that
// needs the sums reduces them in its prologue, every block for itself, in one
// fixed order (so all blocks hold the same values, run after run), and block 0
// stores the results in KState for the kernels after it.  A separate one-block
// finaliser per reduction cost a launch of 5-6 us each, two per order: 19 of the
// 44 launches of a step on a 6D set and half the time of a 2D one.  The
// redundant reads (18 values x up to 512 blocks) come from the L2.
//
// No kernel reads a KState entry that its own block 0 writes: entries are
// indexed by the order, and a prologue at order j writes order j - 1's
// second-pass results and order j's first-pass ones.  (KState's order is the
// exception: it only ever drops to an order that every block of the writing kernel
// finds for itself.)
struct Scalars {
    double2 h[MAXM];   // second-pass coefficients of the provisional q_j
    double2 cc[MAXM];  // H v_j = (H q_j - sum_k cc_k v_k) / beta_{j-1}
    double2 g[MAXM];   // Arnoldi: first-pass column <v_i|H v_j>
    double alpha, ib, bm;
    int stop;
};
// Sums over groups of 16 neighbouring lanes (every lane gets its group's).
__device__ inline double2 group16_sum(double2 v)
{
#pragma unroll
    for (int s = 8; s >= 1; s >>= 1) {
        v.x += __shfl_xor(v.x, s, 64);
        v.y += __shfl_xor(v.y, s, 64);
    }
    return v;
}

// sum[value] of the partials [value][block] of nval values over nb blocks: 16
// lanes take a value, so the 256 threads sum 16 values at once with four shuffle
// steps (a wavefront a value takes six for every value in turn).
__device__ inline void sum_values(const double2 *part, int nval, int nb, double2 *sum)
{
    const int l = threadIdx.x & 15;
    for (int v = threadIdx.x >> 4; v < nval; v += TB / 16) {
        double2 s = make_double2(0.0, 0.0);
        for (int b0 = l; b0 < nb; b0 += 16 * 8) {
            double2 q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int b = b0 + 16 * u;
                q[u] = b < nb ? part[(int64_t)v * RED_BLOCKS + b] : make_double2(0.0, 0.0);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                s.x += q[u].x;
                s.y += q[u].y;
            }
        }
        s = group16_sum(s);
        if (l == 0) sum[v] = s;
    }
}

// One value over many blocks: the block's 256 threads share it (quarter sums).
__device__ inline void sum_single(const double2 *part, int nb, double2 *quarter)
{
    double2 s = make_double2(0.0, 0.0);
    for (int b0 = threadIdx.x; b0 < nb; b0 += TB * 4) {
        double2 q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] = b0 + TB * u < nb ? part[b0 + TB * u] : make_double2(0.0, 0.0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            s.x += q[u].x;
            s.y += q[u].y;
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        s.x += __shfl_xor(s.x, d, 64);
        s.y += __shfl_xor(s.y, d, 64);
    }
    if ((threadIdx.x & 63) == 0) quarter[threadIdx.x >> 6] = s;
}
__device__ inline double2 four(const double2 *q)
{
    return make_double2((q[0].x + q[1].x) + (q[2].x + q[3].x), (q[0].y + q[1].y) + (q[2].y + q[3].y));
}

// Sums NV values over the block's threads into partial[value][block]: the
// threads' values go through LDS, 16 threads then take a value each (as above).
template <int NV>
__device__ inline void block_values_store(const double2 (&acc)[NV], double2 *partial)
{
    __shared__ double2 red[NV][TB];
#pragma unroll
    for (int i = 0; i < NV; ++i) red[i][threadIdx.x] = acc[i];
    __syncthreads();
    const int l = threadIdx.x & 15;
    for (int v = threadIdx.x >> 4; v < NV; v += TB / 16) {
        double2 s = red[v][l];
#pragma unroll
        for (int u = 1; u < TB / 16; ++u) {
            s.x += red[v][l + 16 * u].x;
            s.y += red[v][l + 16 * u].y;
        }
        s = group16_sum(s);
        if (l == 0) partial[(int64_t)v * RED_BLOCKS + blockIdx.x] = s;
    }
}

// The prologue at order j (256 threads, every block).  ps: the partials of
// sweep j - 1, <v_i|q_j> (i < j) and |q_j|^2, over nbs blocks (j > 0); pd: the
// product's, <q_j|H q_j> (Arnoldi: <v_i|H q_j> for i < j, then <q_j|H q_j>),
// over nbd blocks.  First beta_{j-1} and the second-pass coefficients h of q_j;
// where the order ends before j (a breakdown, or the estimate n0 dt^j / j!
// prod beta_i within the tolerance) `stop` is set and KState's order with it.
// Then, for q_j = beta_{j-1} v_j + sum_{i<j} h_i v_i,
// Lanczos, with H v_i = beta_i v_{i+1} + alpha_i v_i + beta_{i-1} v_{i-1} (i < j),
//   g_i     = <v_i|H q_j> = beta_i <v_{i+1}|q_j> + alpha_i h_i + beta_{i-1} h_{i-1}
//   alpha_j = (<q_j|H q_j> - 2 Re sum conj(h_i) g_i + sum conj(h_i) T_ik h_k) / beta_{j-1}^2
//   cc_k    = sum_{i<j} T_ki h_i (k <= j);
// Arnoldi, with H v_i = sum_{k<=i+1} H_ki v_k (h1 + h2, and beta_i for k = i + 1),
//   cc_k    = sum_{i<j} H_ki h_i
//   g_i     = <v_i|H v_j> = (<v_i|H q_j> - cc_i) / beta_{j-1} (i < j; i = j from
//             <v_j|H q_j> = (<q_j|H q_j> - sum conj(h_i) <v_i|H q_j>) / beta_{j-1}).
template <bool ARN>
__device__ void krylov_scalars(KState *ks, int j, const double2 *ps, int nbs, const double2 *pd, int nbd, Scalars &sc)
{
    __shared__ double2 S[MAXM + 2], R[MAXM + 4];
    const int t = threadIdx.x;
    const bool store = blockIdx.x == 0;
    const int meff = ks->meff;
    // KState entries first: their latency overlaps the partials'
    const double est0 = j > 0 ? ks->est[j - 1] : 0.0, kdt = ks->kdt, ktol = ks->ktol;
    double al = 0.0, be = 0.0;
    if (t < j) al = ks->alpha[t];
    if (t < j - 1) be = ks->beta[t];
    const int ka = t >> 4, ia = t & 15;  // Arnoldi: thread (k, i) holds H_ki
    double2 a1 = make_double2(0.0, 0.0), a2 = a1;
    double bi = 0.0;
    if (ARN && t < 256 && ia < j) {
        if (ka <= ia) {
            a1 = ks->h1[ka * MAXM + ia];
            if (ia < j - 1) a2 = ks->h2[ka * MAXM + ia];
        }
        if (ia < j - 1) bi = ks->beta[ia];
    }
    sum_values(ps, j > 0 ? j + 1 : 0, nbs, S);
    if (ARN) sum_values(pd, j + 1, nbd, R);
    else sum_single(pd, nbd, R);
    __syncthreads();
    double b = 1.0;
    double2 h = make_double2(0.0, 0.0);
    if (t < 64) {
        if (t < j) h = S[t];
        const double hh = group16_sum(make_double2(h.x * h.x + h.y * h.y, 0.0)).x;  // lanes 0-15 hold the h_i
        int stop = j >= meff;
        if (j > 0 && !stop) {
            const double b2 = S[j].x - __shfl(hh, 0, 64);
            b = sqrt(b2 > 0.0 ? b2 : 0.0);
            const double est = est0 * kdt * b / (double)j;
            stop = b < 1e-13 || (ktol > 0.0 && est <= ktol);
            if (store) {
                if (t < j) ks->h2[t * MAXM + (j - 1)] = h;
                if (t == 0) {
                    ks->beta[j - 1] = b;
                    ks->est[j] = est;
                    if (stop) ks->meff = j;
                }
            }
        }
        if (t < MAXM) sc.h[t] = h;
        if (t == 0) {
            sc.stop = stop;
            sc.bm = j > 0 ? b : 0.0;
            sc.ib = j > 0 ? 1.0 / b : 1.0;
        }
        if (!ARN) {
            if (t == j - 1) be = b;
            const double2 hd = make_double2(__shfl_down(h.x, 1, 64), __shfl_down(h.y, 1, 64));
            const double2 hu = make_double2(__shfl_up(h.x, 1, 64), __shfl_up(h.y, 1, 64));
            const double bu = __shfl_up(be, 1, 64);
            const double2 hn = t + 1 < j ? hd : make_double2(b, 0.0);
            const double2 hp = t >= 1 ? hu : make_double2(0.0, 0.0);
            const double bp = t >= 1 ? bu : 0.0;
            double s1 = 0.0, s2 = 0.0;
            if (t < j) {
                const double gx = be * hn.x + al * h.x + bp * hp.x, gy = be * hn.y + al * h.y + bp * hp.y;
                s1 = h.x * gx + h.y * gy;  // Re(conj(h_i) g_i)
                s2 = al * (h.x * h.x + h.y * h.y);
                if (t + 1 < j) s2 += 2.0 * be * (h.x * hn.x + h.y * hn.y);
            }
            const double2 s = group16_sum(make_double2(s1, s2));
            double2 cc = make_double2(0.0, 0.0);
            if (t <= j) {
                cc.x = al * h.x + bp * hp.x;
                cc.y = al * h.y + bp * hp.y;
                if (t + 1 < j) {
                    cc.x += be * hd.x;
                    cc.y += be * hd.y;
                }
            }
            if (t < MAXM) sc.cc[t] = cc;
            if (t == 0) {
                const double mu = four(R).x;
                const double alpha = j > 0 ? (mu - 2.0 * s.x + s.y) / (b * b) : mu;
                sc.alpha = alpha;
                if (store && !stop) {
                    ks->alpha[j] = alpha;
                    ks->inv_b = sc.ib;
                }
            }
        }
    }
    __syncthreads();
    if (!ARN) return;
    {
        double2 term = make_double2(0.0, 0.0);
        if (ia < j) {
            const double2 hi = sc.h[ia];
            if (ka <= ia) {
                if (ia == j - 1) a2 = S[ka];
                const double2 hk = make_double2(a1.x + a2.x, a1.y + a2.y);
                term = make_double2(hk.x * hi.x - hk.y * hi.y, hk.x * hi.y + hk.y * hi.x);
            } else if (ka == ia + 1) {
                if (ia == j - 1) bi = sc.bm;
                term = make_double2(bi * hi.x, bi * hi.y);
            }
        }
        term = group16_sum(term);
        if (ia == 0) sc.cc[ka] = term;
    }
    __syncthreads();
    if (t < 64) {
        const double ib = sc.ib;
        const double2 r = t <= j ? R[t] : make_double2(0.0, 0.0);
        double2 pr = make_double2(0.0, 0.0);
        if (t < j) pr = make_double2(h.x * r.x + h.y * r.y, h.x * r.y - h.y * r.x);  // conj(h_i) r_i
        pr = group16_sum(pr);
        const double2 sum = make_double2(__shfl(pr.x, 0, 64), __shfl(pr.y, 0, 64));
        double2 g = make_double2(0.0, 0.0);
        if (t < j) g = make_double2((r.x - sc.cc[t].x) * ib, (r.y - sc.cc[t].y) * ib);
        if (t == j) {
            if (j == 0) g = r;
            else g = make_double2(((r.x - sum.x) * ib - sc.cc[t].x) * ib, ((r.y - sum.y) * ib - sc.cc[t].y) * ib);
        }
        if (t < MAXM) sc.g[t] = g;
        if (store && !sc.stop) {
            if (t <= j) ks->h1[t * MAXM + j] = g;
            if (t < MAXM) ks->h2[t * MAXM + j] = make_double2(0.0, 0.0);  // a step's last column keeps its first pass only
            if (t == j) {
                ks->alpha[j] = g.x;
                ks->inv_b = ib;
            }
        }
    }
    __syncthreads();
}

// ---- starting vector ------------------------------------------------------------
__global__ __launch_bounds__(TB) void k_norm0(const double2 *psi, int64_t n, double2 *partial)
{
    double2 acc[1] = {make_double2(0.0, 0.0)};
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) {
        double2 a = psi[p];
        acc[0].x = fma(a.x, a.x, fma(a.y, a.y, acc[0].x));
    }
    block_reduce_store<1>(acc, partial);
}

// v_0 = psi / |psi| with the norm from k_norm0's partials; block 0 starts KState
template <class C>
__global__ __launch_bounds__(TB) void k_start(const double2 *psi, int64_t n, const double2 *partial, int nb,
                                              KState *ks, int m, double dt, double tol, C *v0,
                                              const uint32_t *keys, C *xg)
{
    __shared__ double2 quarter[4];
    sum_single(partial, nb, quarter);
    __syncthreads();
    const double n0 = sqrt(four(quarter).x);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ks->n0 = n0;
        ks->meff = m;
        ks->est[0] = n0;
        ks->kdt = fabs(dt);  // the estimate is a magnitude: |dt|^k
        ks->ktol = tol;
    }
    const double s = 1.0 / n0;
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) {
        double2 a = ld2nt(psi, p);
        st2(v0, p, make_double2(a.x * s, a.y * s));
        if (xg) st2(xg, keys[p], make_double2(a.x * s, a.y * s));
    }
}

// ---- dots of a product ------------------------------------------------------------
template <class C>
__global__ __launch_bounds__(TB) void k_dot1(const C *v, const C *z, int64_t n, double2 *partial, const KState *ks,
                                             int j)
{
    if (j >= ks->meff) return;
    double2 acc[1] = {make_double2(0.0, 0.0)};
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) cdot_acc(acc[0], ld2(v, p), ld2(z, p));
    block_reduce_store<1>(acc, partial);
}

// <v_i|z> for i < NV and <q_j|z>, j = NV (slot j holds the provisional q_j, z = H q_j)
template <class C, int NV>
__global__ __launch_bounds__(TB) void k_arnoldi_dots(const C *Vb, int64_t ld, const C *z, int64_t n,
                                                     double2 *partial, const KState *ks)
{
    if (NV >= ks->meff) return;
    const C *qs = Vb + (int64_t)NV * ld;
    double2 acc[NV + 1];
#pragma unroll
    for (int i = 0; i <= NV; ++i) acc[i] = make_double2(0.0, 0.0);
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) {
        const double2 zv = ld2(z, p);
#pragma unroll
        for (int i = 0; i < NV; ++i) cdot_acc(acc[i], ld2nt(Vb, (int64_t)i * ld + p), zv);
        cdot_acc(acc[NV], ld2(qs, p), zv);
    }
    block_values_store<NV + 1>(acc, partial);
}

// a value that every lane holds, in scalar registers
__device__ inline double2 uniform(double2 v)
{
    int w[4];
    __builtin_memcpy(w, &v, 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
    double2 r;
    __builtin_memcpy(&r, w, 16);
    return r;
}

// ---- sweeps --------------------------------------------------------------------
// Step j = NV with the second Gram-Schmidt pass of each vector delayed to the
// next step's sweep.  Slot j holds the provisional q_j = beta_{j-1} v_j +
// sum_{i<j} h_i v_i (first pass only, unnormalised) and z = H q_j; with the
// scalars of the prologue one pass
//   v_j     = (q_j - sum_{i<j} h_i v_i) / beta_{j-1}           -> slot j
//   H v_j   = (z - sum_{k<j} cc_k v_k - cc_j v_j) / beta_{j-1}
//   q_{j+1} = H v_j - alpha_j v_j - beta_{j-1} v_{j-1}          -> slot j+1
// (Arnoldi: q_{j+1} = H v_j - sum_{i<=j} g_i v_i) with the partial sums of
// <v_i|q_{j+1}> (i <= j) and |q_{j+1}|^2: the next second pass's coefficients
// and beta_j.  In exact arithmetic h = 0 and this is the plain recurrence; with
// rounding it applies the same second projection as two separate sweeps would,
// one step later.
// Bound by HBM (j + 2 vectors read, 2 written) on large sets, by its launch and
// prologue on small ones: a block per 256 points up to KRY_BLOCKS, so that a
// small set's partials stay few, the first points' loads issued before the
// prologue, and reductions of 16 values at once (8.6 us to 5.7 on 660 functions,
// 11.4 to 7.5 on a 24^4 set, 83 us or 5.4 TB/s on 4M functions as before).
template <class C, int NV, bool ARN>
__global__ __launch_bounds__(TB, 2) void k_sweep(C *Vb, int64_t ld, const C *z, int64_t n, KState *ks, const double2 *ps,
                                              int nbs, const double2 *pd, int nbd, double2 *pout,
                                              const uint32_t *keys, C *xg)
{
    __shared__ Scalars sc;
    constexpr int NH = NV > 0 ? NV : 1;
    C *qs = Vb + (int64_t)NV * ld;
    C *qn = Vb + (int64_t)(NV + 1) * ld;
    // the first points' loads are on their way while the prologue sums
    double2 qv = make_double2(0.0, 0.0), hv = qv, vv[NH];
    uint32_t key = 0;
    const int64_t stride = (int64_t)gridDim.x * TB;
    auto load = [&](int64_t p) {
        if (p >= n) return;
        qv = ld2nt(qs, p);
        hv = ld2nt(z, p);
#pragma unroll
        for (int i = 0; i < NV; ++i) vv[i] = ld2nt(Vb, (int64_t)i * ld + p);
        if (xg) key = keys[p];
    };
    load(gid());
    krylov_scalars<ARN>(ks, NV, ps, nbs, pd, nbd, sc);
    if (sc.stop) return;
    double2 hq[NH], cc[NV + 1], g1[ARN ? NV + 1 : 1];
#pragma unroll
    for (int i = 0; i < NV; ++i) hq[i] = uniform(sc.h[i]);
#pragma unroll
    for (int k = 0; k <= NV; ++k) {
        cc[k] = uniform(sc.cc[k]);
        if (ARN) g1[k] = uniform(sc.g[k]);
    }
    const double ib = sc.ib, al = ARN ? 0.0 : sc.alpha, bm = sc.bm;
    double2 acc[NV + 2];
#pragma unroll
    for (int i = 0; i < NV + 2; ++i) acc[i] = make_double2(0.0, 0.0);
    for (int64_t p = gid(); p < n; p += stride) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            qv.x -= hq[i].x * vv[i].x - hq[i].y * vv[i].y;
            qv.y -= hq[i].x * vv[i].y + hq[i].y * vv[i].x;
            hv.x -= cc[i].x * vv[i].x - cc[i].y * vv[i].y;
            hv.y -= cc[i].x * vv[i].y + cc[i].y * vv[i].x;
        }
        st2nt(qs, p, make_double2(qv.x * ib, qv.y * ib));
        const double2 vj = stored(qs, make_double2(qv.x * ib, qv.y * ib));
        hv.x -= cc[NV].x * vj.x - cc[NV].y * vj.y;
        hv.y -= cc[NV].x * vj.y + cc[NV].y * vj.x;
        double2 wp = make_double2(hv.x * ib, hv.y * ib);
        if constexpr (ARN) {
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                wp.x -= g1[i].x * vv[i].x - g1[i].y * vv[i].y;
                wp.y -= g1[i].x * vv[i].y + g1[i].y * vv[i].x;
            }
            wp.x -= g1[NV].x * vj.x - g1[NV].y * vj.y;
            wp.y -= g1[NV].x * vj.y + g1[NV].y * vj.x;
        } else {
            wp = make_double2(hv.x * ib - al * vj.x, hv.y * ib - al * vj.y);
            if (NV > 0) {
                wp.x -= bm * vv[NH - 1].x;
                wp.y -= bm * vv[NH - 1].y;
            }
        }
        st2(qn, p, wp);
        if (xg) st2(xg, key, wp);
        const double2 ws = stored(qn, wp);
#pragma unroll
        for (int i = 0; i < NV; ++i) cdot_acc(acc[i], vv[i], ws);
        cdot_acc(acc[NV], vj, ws);
        acc[NV + 1].x = fma(ws.x, ws.x, fma(ws.y, ws.y, acc[NV + 1].x));
        load(p + stride);
    }
    block_values_store<NV + 2>(acc, pout);
}

// v_j = (q_j - sum_{i<j} h_i v_i) / beta_{j-1} in slot j: the last vector of a
// step that ran to its full order (no later sweep corrects it).
template <class C, int NV>
__global__ __launch_bounds__(TB) void k_fix_last(C *Vb, int64_t ld, int64_t n, const KState *ks)
{
    if (NV >= ks->meff) return;
    double2 hq[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) hq[i] = ks->h2[i * MAXM + (NV - 1)];
    const double ib = ks->inv_b;
    C *qs = Vb + (int64_t)NV * ld;
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) {
        double2 qv = ld2(qs, p);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const double2 v = ld2nt(Vb, (int64_t)i * ld + p);
            qv.x -= hq[i].x * v.x - hq[i].y * v.y;
            qv.y -= hq[i].x * v.y + hq[i].y * v.x;
        }
        st2(qs, p, make_double2(qv.x * ib, qv.y * ib));
    }
}

// ---- the small exponential ---------------------------------------------------------
// acc + sum_l P[r][l] Q[l][c] of 16 x 16 complex matrices in LDS
__device__ inline double2 mul16(const double2 (&P)[MAXM][MAXM + 1], const double2 (&Q)[MAXM][MAXM + 1], int r, int c,
                                double2 acc)
{
#pragma unroll
    for (int l = 0; l < MAXM; ++l) {
        const double2 a = P[r][l], b = Q[l][c];
        acc.x = fma(a.x, b.x, fma(-a.y, b.y, acc.x));
        acc.y = fma(a.x, b.y, fma(a.y, b.x, acc.y));
    }
    return acc;
}

// ks->y = n0 exp(-i dt Hk) e_1 for the meff x meff Krylov matrix, by scaling
// (norm at most 1/2) and squaring of the degree-16 Taylor polynomial (remainder
// below 1e-19) in powers of A^4: six products and one per squaring, where term by
// term at norm 1/8 it took 18 and two squarings more (23 us, now 12.6 us with the prologue; a
// chain of 16 x 16 products by one workgroup, bound by LDS latency).  256 threads,
// thread (r, c) owns an entry.
__device__ void small_exponential(KState *ks, int meff, double dt, bool hermitian)
{
    __shared__ double2 A[MAXM][MAXM + 1], A2[MAXM][MAXM + 1], A4[MAXM][MAXM + 1], E[2][MAXM][MAXM + 1];
    __shared__ double rown[MAXM];
    const int r = threadIdx.x / MAXM, c = threadIdx.x % MAXM;
    double2 h = make_double2(0.0, 0.0);
    if (r < meff && c < meff) {
        if (hermitian) {
            if (r == c) h = make_double2(ks->alpha[r], 0.0);
            else if (r == c + 1) h = make_double2(ks->beta[c], 0.0);
            else if (c == r + 1) h = make_double2(ks->beta[r], 0.0);
        } else {
            if (r <= c) {
                double2 a = ks->h1[r * MAXM + c], b = ks->h2[r * MAXM + c];
                h = make_double2(a.x + b.x, a.y + b.y);
            } else if (r == c + 1) {
                h = make_double2(ks->beta[c], 0.0);
            }
        }
    }
    // A = -i dt H
    double2 a = make_double2(dt * h.y, -dt * h.x);
    const double rs = group16_sum(make_double2(sqrt(a.x * a.x + a.y * a.y), 0.0)).x;  // a row is 16 lanes
    if (c == 0) rown[r] = rs;
    __syncthreads();
    double nrm = 0.0;
#pragma unroll
    for (int i = 0; i < MAXM; ++i) nrm = rown[i] > nrm ? rown[i] : nrm;
    int sq = 0;
    while (nrm > 0.5 && sq < 1100) {
        nrm *= 0.5;
        ++sq;
    }
    const double scale = ldexp(1.0, -sq);
    a = make_double2(a.x * scale, a.y * scale);
    const double one = r == c ? 1.0 : 0.0;
    const double2 zero = make_double2(0.0, 0.0);
    A[r][c] = a;
    __syncthreads();
    const double2 a2 = mul16(A, A, r, c, zero);
    A2[r][c] = a2;
    __syncthreads();
    const double2 a3 = mul16(A2, A, r, c, zero), a4 = mul16(A2, A2, r, c, zero);
    A4[r][c] = a4;
    // blocks B_i = sum_{q<4} A^q / (4 i + q)!, combined from the highest down:
    // ((((A^4 / 16! + B_3) A^4 + B_2) A^4 + B_1) A^4 + B_0
    constexpr double F[17] = {1.0,
                              1.0,
                              1.0 / 2,
                              1.0 / 6,
                              1.0 / 24,
                              1.0 / 120,
                              1.0 / 720,
                              1.0 / 5040,
                              1.0 / 40320,
                              1.0 / 362880,
                              1.0 / 3628800,
                              1.0 / 39916800,
                              1.0 / 479001600,
                              1.0 / 6227020800.0,
                              1.0 / 87178291200.0,
                              1.0 / 1307674368000.0,
                              1.0 / 20922789888000.0};
    auto block = [&](int i) {
        return make_double2(F[4 * i] * one + F[4 * i + 1] * a.x + F[4 * i + 2] * a2.x + F[4 * i + 3] * a3.x,
                            F[4 * i + 1] * a.y + F[4 * i + 2] * a2.y + F[4 * i + 3] * a3.y);
    };
    double2 e = block(3);
    e.x += F[16] * a4.x;
    e.y += F[16] * a4.y;
    int cur = 0;
    E[0][r][c] = e;
    __syncthreads();
#pragma unroll
    for (int i = 2; i >= 0; --i) {
        e = mul16(E[cur], A4, r, c, block(i));
        cur ^= 1;
        E[cur][r][c] = e;
        __syncthreads();
    }
    for (int q = 0; q < sq; ++q) {
        e = mul16(E[cur], E[cur], r, c, zero);
        cur ^= 1;
        E[cur][r][c] = e;
        __syncthreads();
    }
    if (c == 0) {
        const double n0 = ks->n0;
        ks->y[r] = (r < meff) ? make_double2(n0 * e.x, n0 * e.y) : zero;
    }
    __syncthreads();
}

// One block.  With pd: the scalars of the last order j = m - 1 (no sweep
// follows it).  With `expv`: the exponential's first column in y.  With `fold`
// (and a step that ran to its full order): its last vector is provisional,
// v_L = (q_L - sum_{i<L} h_i v_i) / beta_{L-1}, L = m - 1, so the propagated vector
// sum_k y_k v_k is sum_{k<L} (y_k - y_L h_k / beta_{L-1}) v_k + (y_L / beta_{L-1}) q_L:
// the coefficients absorb the correction.
template <bool ARN>
__global__ __launch_bounds__(TB) void k_close(KState *ks, int m, const double2 *ps, int nbs, const double2 *pd,
                                              int nbd, double dt, int expv, int fold, double *alpha0,
                                              double *order)
{
    __shared__ Scalars sc;
    __shared__ int s_meff;
    if (threadIdx.x == 0) s_meff = ks->meff;
    __syncthreads();
    int meff = s_meff;
    if (pd) {
        krylov_scalars<ARN>(ks, m - 1, ps, nbs, pd, nbd, sc);
        if (sc.stop) meff = meff < m - 1 ? meff : m - 1;
        __threadfence_block();
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (alpha0) *alpha0 = ks->alpha[0];
        if (order) {
            *order = (double)meff;
            __threadfence_system();
        }
    }
    if (!expv) return;
    small_exponential(ks, meff, dt, !ARN);
    if (!fold || meff != m || m < 2) return;
    const int L = m - 1, k = threadIdx.x;
    const double2 yl = ks->y[L];
    __syncthreads();
    const double ib = ks->inv_b;
    if (k < L) {
        const double2 h = ks->h2[k * MAXM + (L - 1)];
        double2 y = ks->y[k];
        y.x -= ib * (yl.x * h.x - yl.y * h.y);
        y.y -= ib * (yl.x * h.y + yl.y * h.x);
        ks->y[k] = y;
    }
    if (k == L) ks->y[L] = make_double2(yl.x * ib, yl.y * ib);
}

template <class C>
__global__ void k_lincomb(const C *Vb, int64_t ld, const double2 *psi_master, int64_t n, const KState *ks,
                          double2 *out)
{
    int meff = ks->meff;
    double2 y[MAXM];
#pragma unroll
    for (int i = 0; i < MAXM; ++i) y[i] = ks->y[i];
    double inv_n0 = 1.0 / ks->n0;
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * blockDim.x) {
        // j = 0 from the FP64 master copy (exact v_0 direction, its last use), j >= 1 from the basis
        double2 v = ld2nt(psi_master, p);
        v.x *= inv_n0;
        v.y *= inv_n0;
        double2 acc = make_double2(y[0].x * v.x - y[0].y * v.y, y[0].x * v.y + y[0].y * v.x);
#pragma unroll
        for (int i = 1; i < MAXM; ++i) {
            if (i < meff) {
                double2 b = ld2nt(Vb, (int64_t)i * ld + p);
                acc.x += y[i].x * b.x - y[i].y * b.y;
                acc.y += y[i].x * b.y + y[i].y * b.x;
            }
        }
        out[p] = acc;
    }
}

unsigned stream_blocks(int64_t n)
{
    const int64_t b = (n + TB - 1) / TB;
    return (unsigned)std::min<int64_t>(std::max<int64_t>(b, 1), 4 * RED_BLOCKS);
}

const double2 *sweep_partials(const double2 *partial, int j) { return partial + (int64_t)(j & 1) * KRY_SLOTS * RED_BLOCKS; }

}  // namespace

int kry_blocks(int64_t n)
{
    const int64_t b = (n + TB - 1) / TB;
    return (int)std::min<int64_t>(std::max<int64_t>(b, 1), KRY_BLOCKS);
}

template <class C>
void kry_start(const double2 *psi, int64_t n, double2 *partial, KState *ks, int m, double dt, double tol, C *v0,
               const uint32_t *keys, C *xg, hipStream_t s)
{
    const int nb = kry_blocks(n);
    hipLaunchKernelGGL(k_norm0, dim3(nb), dim3(TB), 0, s, psi, n, partial);
    hipLaunchKernelGGL(k_start<C>, dim3(nb), dim3(TB), 0, s, psi, n, partial, nb, ks, m, dt, tol, v0, keys,
                       xg);
}

#define PPQ_ORDERS(CALL)    \
    switch (j) {            \
    case 0: CALL(0); break; \
    case 1: CALL(1); break; \
    case 2: CALL(2); break; \
    case 3: CALL(3); break; \
    case 4: CALL(4); break; \
    case 5: CALL(5); break; \
    case 6: CALL(6); break; \
    case 7: CALL(7); break; \
    case 8: CALL(8); break; \
    case 9: CALL(9); break; \
    case 10: CALL(10); break; \
    case 11: CALL(11); break; \
    case 12: CALL(12); break; \
    case 13: CALL(13); break; \
    case 14: CALL(14); break; \
    case 15: CALL(15); break; \
    default: break;         \
    }

template <class C>
int kry_dots(const C *Vb, int64_t ld, const C *z, int64_t n, double2 *partial, const KState *ks, int j, bool arnoldi,
             hipStream_t s)
{
    const int nb = kry_blocks(n);
    double2 *pd = partial + KRY_DOTS;
    if (!arnoldi) {
        hipLaunchKernelGGL(k_dot1<C>, dim3(nb), dim3(TB), 0, s, Vb + (int64_t)j * ld, z, n, pd, ks, j);
        return nb;
    }
#define CALL(NV) hipLaunchKernelGGL((k_arnoldi_dots<C, NV>), dim3(nb), dim3(TB), 0, s, Vb, ld, z, n, pd, ks)
    PPQ_ORDERS(CALL)
#undef CALL
    return nb;
}

template <class C>
void kry_sweep(C *Vb, int64_t ld, const C *z, int64_t n, double2 *partial, int nbd, KState *ks, int j, bool arnoldi,
               const uint32_t *keys, C *xg, hipStream_t s)
{
    const int nb = kry_blocks(n);
    const double2 *ps = sweep_partials(partial, j + 1), *pd = partial + KRY_DOTS;
    double2 *po = const_cast<double2 *>(sweep_partials(partial, j));
    if (arnoldi) {
#define CALL(NV)                                                                                                  \
    hipLaunchKernelGGL((k_sweep<C, NV, true>), dim3(nb), dim3(TB), 0, s, Vb, ld, z, n, ks, ps, nb, pd, nbd, po, keys, xg)
        PPQ_ORDERS(CALL)
#undef CALL
    } else {
#define CALL(NV)                                                                                                   \
    hipLaunchKernelGGL((k_sweep<C, NV, false>), dim3(nb), dim3(TB), 0, s, Vb, ld, z, n, ks, ps, nb, pd, nbd, po, keys, xg)
        PPQ_ORDERS(CALL)
#undef CALL
    }
}

template <class C>
void kry_fix_last(C *Vb, int64_t ld, int64_t n, const KState *ks, int j, hipStream_t s)
{
    const unsigned nb = stream_blocks(n);
#define CALL(NV)                                                                                         \
    if constexpr (NV > 0) hipLaunchKernelGGL((k_fix_last<C, NV>), dim3(nb), dim3(TB), 0, s, Vb, ld, n, ks)
    PPQ_ORDERS(CALL)
#undef CALL
}

void kry_close(KState *ks, int m, const double2 *partial, int64_t n, int nbd, double dt, bool hermitian, bool expv,
               bool fold, hipStream_t s, double *alpha0, double *order)
{
    const int nb = kry_blocks(n);
    const double2 *ps = sweep_partials(partial, m), *pd = nbd > 0 ? partial + KRY_DOTS : nullptr;
    if (hermitian)
        hipLaunchKernelGGL(k_close<false>, dim3(1), dim3(TB), 0, s, ks, m, ps, nb, pd, nbd, dt, (int)expv, (int)fold,
                           alpha0, order);
    else
        hipLaunchKernelGGL(k_close<true>, dim3(1), dim3(TB), 0, s, ks, m, ps, nb, pd, nbd, dt, (int)expv, (int)fold,
                           alpha0, order);
}

template <class C>
void lincomb(const C *Vb, int64_t ld, const double2 *psi_master, int64_t n, const KState *ks, double2 *psi_out,
             hipStream_t s)
{
    hipLaunchKernelGGL(k_lincomb<C>, dim3(stream_blocks(n)), dim3(TB), 0, s, Vb, ld, psi_master, n, ks, psi_out);
}

#define PPQ_INST(C)                                                                                                \
    template void kry_start<C>(const double2 *, int64_t, double2 *, KState *, int, double, double, C *,            \
                               const uint32_t *, C *, hipStream_t);                                                \
    template int kry_dots<C>(const C *, int64_t, const C *, int64_t, double2 *, const KState *, int, bool,         \
                             hipStream_t);                                                                         \
    template void kry_sweep<C>(C *, int64_t, const C *, int64_t, double2 *, int, KState *, int, bool,         \
                               const uint32_t *, C *, hipStream_t);                                                \
    template void kry_fix_last<C>(C *, int64_t, int64_t, const KState *, int, hipStream_t);                        \
    template void lincomb<C>(const C *, int64_t, const double2 *, int64_t, const KState *, double2 *, hipStream_t);
PPQ_INST(double2)
PPQ_INST(float2)
#undef PPQ_INST

}  // namespace ppq
