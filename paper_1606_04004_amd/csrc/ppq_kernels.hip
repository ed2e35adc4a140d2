// gfx950 kernels: scans, adaption (flag / dilate / compact / remap), fiber
// tables, potential cache, Krylov vector work, small exponential, observables.
// The fiber contraction kernels live in ppq_hpsi.hip.
#include <algorithm>
#include <limits>

#include "ppq_device.hpp"

namespace ppq {

namespace {

// complex product without contraction: (ac - bd) + i(ad + bc)
__device__ inline double2 cmul_rn(double2 a, double2 b)
{
    return make_double2(__dsub_rn(__dmul_rn(a.x, b.x), __dmul_rn(a.y, b.y)),
                        __dadd_rn(__dmul_rn(a.x, b.y), __dmul_rn(a.y, b.x)));
}

__device__ inline bool above_eps(double2 c, double eps2)
{
    return __dadd_rn(__dmul_rn(c.x, c.x), __dmul_rn(c.y, c.y)) >= eps2;
}

__device__ inline void set_bit(uint64_t *bm, uint32_t key)
{
    atomicOr((unsigned long long *)&bm[key >> 6], 1ull << (key & 63));
}

// Sets bit `key` for every lane with `valid`; all 64 lanes of the wavefront
// must call it together.  Lanes that target the same word are merged by a
// segmented OR across neighbouring lanes, so one atomic per run of lanes
// hitting one word is issued (sorted keys put most of a wavefront's targets
// in a few words).
__device__ inline void set_bit_wave(uint64_t *bm, uint32_t key, bool valid)
{
    const int lane = threadIdx.x & 63;
    uint32_t w = valid ? (key >> 6) : 0xffffffffu;
    uint64_t bits = valid ? (1ull << (key & 63)) : 0ull;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t ow = __shfl_up(w, d, 64);
        uint32_t olo = __shfl_up((uint32_t)bits, d, 64);
        uint32_t ohi = __shfl_up((uint32_t)(bits >> 32), d, 64);
        if (lane >= d && ow == w) bits |= ((uint64_t)ohi << 32) | olo;
    }
    uint32_t nw = __shfl_down(w, 1, 64);
    bool last = (lane == 63) || (nw != w);
    if (valid && last) atomicOr((unsigned long long *)&bm[w], (unsigned long long)bits);
}

// Phase-space axis `part` of dimension k for `key`: the grid index of a DVR
// dimension (part 0), or the cell (part 0) and level (part 1) index of a
// lattice dimension; its index, extent and key stride.
__device__ inline void phase_axis(const GridDesc &g, uint32_t key, int k, int part, int &idx, int &ext, int64_t &str)
{
    const int d = (int)((key / g.stride[k]) % (uint32_t)g.n[k]);
    if (g.lat_s[k] == 0) {
        idx = d;
        ext = g.n[k];
        str = g.stride[k];
    } else if (part == 0) {
        idx = d / g.lat_l[k];
        ext = g.lat_s[k];
        str = (int64_t)g.lat_l[k] * g.stride[k];
    } else {
        idx = d % g.lat_l[k];
        ext = g.lat_l[k];
        str = g.stride[k];
    }
}

// Marks `key` and its neighbours of the selected stencil for lanes with `keep`
// (wave-collective: every lane runs the same loop bounds, which depend on the
// grid alone).  The wider balls of Sec. III.A count index changes over the
// phase-space axes: one per DVR dimension, two (cell, level) per lattice one.
__device__ inline void set_with_neighbours(const GridDesc &g, uint64_t *bm, uint32_t key, bool keep)
{
    if (g.pairs == 2) {
        // ball radius 2: every combination of -1/0/+1 changes over the axes,
        // the key itself included; the combinations are counted in base 3,
        // one digit per axis.  A wavefront with nothing to keep skips them
        // (the test is uniform across its lanes, so the collective calls
        // stay in step).
        if (__ballot(keep) == 0) return;
        int naxes = 0;
        for (int k = 0; k < g.D; ++k) naxes += g.lat_s[k] ? 2 : 1;
        int ncomb = 1;
        for (int a = 0; a < naxes; ++a) ncomb *= 3;
        for (int cmb = 0; cmb < ncomb; ++cmb) {
            int rest = cmb;
            bool inside = keep;
            int64_t shift = 0;
            for (int k = 0; k < g.D; ++k) {
                for (int part = 0; part < (g.lat_s[k] ? 2 : 1); ++part) {
                    int idx, ext;
                    int64_t str;
                    phase_axis(g, key, k, part, idx, ext, str);
                    const int a = rest % 3 - 1;
                    rest /= 3;
                    inside = inside && idx + a >= 0 && idx + a < ext;
                    shift += a * str;
                }
            }
            set_bit_wave(bm, (uint32_t)((int64_t)key + shift), inside);
        }
        return;
    }
    set_bit_wave(bm, key, keep);
    for (int k = 0; k < g.D; ++k) {
        uint32_t sk = g.stride[k];
        int d = (int)((key / sk) % (uint32_t)g.n[k]);
        if (g.lat_s[k] == 0) {
            set_bit_wave(bm, key - sk, keep && d > 0);
            set_bit_wave(bm, key + sk, keep && d + 1 < g.n[k]);
        } else {
            int nl = g.lat_l[k];
            int si = d / nl, l = d % nl;
            set_bit_wave(bm, key - (uint32_t)nl * sk, keep && si > 0);
            set_bit_wave(bm, key + (uint32_t)nl * sk, keep && si + 1 < g.lat_s[k]);
            set_bit_wave(bm, key - sk, keep && l > 0);
            set_bit_wave(bm, key + sk, keep && l + 1 < nl);
        }
    }
    // ball radius sqrt(2): also every change of +-1 on two axes at once
    if (g.pairs == 1) {
        for (int k = 0; k < g.D; ++k) {
            for (int pk = 0; pk < (g.lat_s[k] ? 2 : 1); ++pk) {
                int ia, ea;
                int64_t sa;
                phase_axis(g, key, k, pk, ia, ea, sa);
                for (int l = k; l < g.D; ++l) {
                    for (int pl = (l == k ? pk + 1 : 0); pl < (g.lat_s[l] ? 2 : 1); ++pl) {
                        int ib, eb;
                        int64_t sb;
                        phase_axis(g, key, l, pl, ib, eb, sb);
                        const bool ad = ia > 0, au = ia + 1 < ea, bd = ib > 0, bu = ib + 1 < eb;
                        set_bit_wave(bm, (uint32_t)((int64_t)key - sa - sb), keep && ad && bd);
                        set_bit_wave(bm, (uint32_t)((int64_t)key - sa + sb), keep && ad && bu);
                        set_bit_wave(bm, (uint32_t)((int64_t)key + sa - sb), keep && au && bd);
                        set_bit_wave(bm, (uint32_t)((int64_t)key + sa + sb), keep && au && bu);
                    }
                }
            }
        }
    }
}

// Counts `pred` over the block and adds the block's total with one atomic
// (integer, so the sum is order-independent).  Block-collective.
__device__ inline void count_ballot(bool pred, unsigned long long *counter)
{
    __shared__ unsigned s_cnt;
    if (threadIdx.x == 0) s_cnt = 0u;
    __syncthreads();
    uint64_t b = __ballot(pred);
    if ((threadIdx.x & 63) == 0 && b) atomicAdd(&s_cnt, (unsigned)__popcll(b));
    __syncthreads();
    if (threadIdx.x == 0 && s_cnt) atomicAdd(counter, (unsigned long long)s_cnt);
}

// Counts `pred` over the block into block_counts[blockIdx.x] (a plain store:
// thousands of blocks adding to one address serialise).  Block-collective.
__device__ inline void count_block(bool pred, unsigned *block_counts)
{
    __shared__ unsigned s_cnt;
    if (threadIdx.x == 0) s_cnt = 0u;
    __syncthreads();
    uint64_t b = __ballot(pred);
    if ((threadIdx.x & 63) == 0 && b) atomicAdd(&s_cnt, (unsigned)__popcll(b));
    __syncthreads();
    if (threadIdx.x == 0) block_counts[blockIdx.x] = s_cnt;
}

// *out = sum of nb block counts (one block, fixed order)
__global__ __launch_bounds__(1024) void k_sum_counts(const unsigned *bc, int64_t nb, unsigned long long *out)
{
    __shared__ unsigned long long s_part[16];
    unsigned long long c = 0;
    for (int64_t i = threadIdx.x; i < nb; i += 1024) c += bc[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int i = 0; i < 16; ++i) t += s_part[i];
        *out = t;
    }
}

// ---- scan ------------------------------------------------------------------
constexpr int SB = 256;
// Elements a thread takes: eight, or one while that makes at most as many tiles as the
// top scan has threads (fewer blocks than CUs would each be a chain of eight: a 4D
// bitmap of 16K words dilated, scanned and compacted in 8 blocks 29 + 21 us, 8 + 6 in 64).
constexpr int SI = 8;
constexpr int64_t SCAN_ONE = (int64_t)SB * 1024;
static int scan_items(int64_t n) { return n <= SCAN_ONE ? 1 : SI; }
static int64_t scan_tiles(int64_t n)
{
    const int64_t t = (int64_t)SB * scan_items(n);
    return std::max<int64_t>((n + t - 1) / t, 1);
}

__device__ inline uint32_t wave_incl_scan(uint32_t v)
{
    int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t t = __shfl_up(v, d, 64);
        if (lane >= d) v += t;
    }
    return v;
}

template <int NT>
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t *total)
{
    __shared__ uint32_t wsum[NT / 64];
    uint32_t inc = wave_incl_scan(v);
    int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        uint32_t s = wsum[i];
        if (i < w) off += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

struct PopLoad {
    const uint64_t *w;
    __device__ uint32_t operator()(int64_t i) const { return (uint32_t)__popcll(w[i]); }
};
struct U32Load {
    const uint32_t *a;
    __device__ uint32_t operator()(int64_t i) const { return a[i]; }
};

template <class L, int I>
__global__ __launch_bounds__(SB) void k_scan_reduce(L ld, int64_t n, uint32_t *tile_sums)
{
    int64_t base = (int64_t)blockIdx.x * (SB * I);
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < I; ++i) {
        int64_t idx = base + (int64_t)i * SB + threadIdx.x;
        if (idx < n) s += ld(idx);
    }
    uint32_t tot;
    block_excl_scan<SB>(s, &tot);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
}

// (host_total, host_count: pinned mirrors of the total and of a device counter
// for a caller that waits for them, without copies of their own)
__global__ __launch_bounds__(1024) void k_scan_top(uint32_t *tile, int64_t ntiles, uint32_t *total,
                                                   uint32_t *host_total, const unsigned long long *count,
                                                   unsigned long long *host_count)
{
    int64_t per = (ntiles + 1023) / 1024;
    int64_t lo = threadIdx.x * per, hi = lo + per < ntiles ? lo + per : ntiles;
    uint32_t s = 0;
    for (int64_t i = lo; i < hi; ++i) s += tile[i];
    uint32_t tot;
    uint32_t off = block_excl_scan<1024>(s, &tot);
    for (int64_t i = lo; i < hi; ++i) {
        uint32_t v = tile[i];
        tile[i] = off;
        off += v;
    }
    if (threadIdx.x == 0) {
        *total = tot;
        if (host_total) *host_total = tot;
        if (host_count) *host_count = *count;
        if (host_total || host_count) __threadfence_system();
    }
}

// The tile's I rows of SB consecutive elements, each row read and written by
// the whole block (coalesced): a wavefront scan per row and wave, then every
// thread adds the totals of the (row, wave) pieces before its own.
template <class L, int I>
__global__ __launch_bounds__(SB) void k_scan_apply(L ld, int64_t n, const uint32_t *tile_off, uint32_t *out)
{
    constexpr int NW = SB / 64;
    __shared__ uint32_t wsum[I * NW];
    const int64_t base = (int64_t)blockIdx.x * (SB * I) + threadIdx.x;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t v[I], inc[I];
#pragma unroll
    for (int i = 0; i < I; ++i) v[i] = (base + (int64_t)i * SB < n) ? ld(base + (int64_t)i * SB) : 0u;
#pragma unroll
    for (int i = 0; i < I; ++i) {
        inc[i] = wave_incl_scan(v[i]);
        if (lane == 63) wsum[i * NW + w] = inc[i];
    }
    __syncthreads();
    uint32_t off = tile_off[blockIdx.x];
#pragma unroll
    for (int i = 0; i < I; ++i) {
        uint32_t before = 0, row = 0;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            const uint32_t t = wsum[i * NW + ww];
            before += ww < w ? t : 0u;
            row += t;
        }
        const int64_t idx = base + (int64_t)i * SB;
        if (idx < n) out[idx] = off + before + inc[i] - v[i];
        off += row;
    }
}

template <class L, int I>
void scan_launch(L ld, int64_t n, uint32_t *out, uint32_t *total, uint32_t *tmp, hipStream_t s)
{
    const unsigned tiles = (unsigned)scan_tiles(n);
    hipLaunchKernelGGL((k_scan_reduce<L, I>), dim3(tiles), dim3(SB), 0, s, ld, n, tmp);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, tmp, (int64_t)tiles, total, nullptr, nullptr, nullptr);
    hipLaunchKernelGGL((k_scan_apply<L, I>), dim3(tiles), dim3(SB), 0, s, ld, n, tmp, out);
}
template <class L>
void scan_impl(L ld, int64_t n, uint32_t *out, uint32_t *total, uint32_t *tmp, hipStream_t s)
{
    if (scan_items(n) == 1) scan_launch<L, 1>(ld, n, out, total, tmp, s);
    else scan_launch<L, SI>(ld, n, out, total, tmp, s);
}

// ---- fills -----------------------------------------------------------------
template <class T>
__global__ void k_fill(T *p, int64_t n, T v)
{
    for (int64_t i = gid(); i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// ---- adaption ----------------------------------------------------------------
// One thread per grid function; a wavefront that keeps none (most of a large
// grid) does not enter the stencil.
__global__ void k_init_flag(GridDesc g, const double2 *tabs, int nmax, double eps2, uint64_t *bm)
{
    // wave-uniform trip count: every lane runs every iteration
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < (int64_t)g.total;
         base += (int64_t)gridDim.x * blockDim.x) {
        int64_t i = base + threadIdx.x;
        bool inside = i < (int64_t)g.total;
        uint32_t key = inside ? (uint32_t)i : 0u;
        double2 v = make_double2(1.0, 0.0);
        for (int k = 0; k < g.D; ++k) {
            int d = (int)((key / g.stride[k]) % (uint32_t)g.n[k]);
            v = cmul_rn(v, tabs[k * nmax + d]);
        }
        bool keep = inside && above_eps(v, eps2);
        if (__ballot(keep) == 0) continue;
        set_with_neighbours(g, bm, key, keep);
    }
}

__global__ void k_product_values(const uint32_t *keys, int64_t n, GridDesc g, const double2 *tabs, int nmax,
                                 double2 *out)
{
    int64_t p = gid();
    if (p >= n) return;
    uint32_t key = keys[p];
    double2 v = make_double2(1.0, 0.0);
    for (int k = 0; k < g.D; ++k) {
        int d = (int)((key / g.stride[k]) % (uint32_t)g.n[k]);
        v = cmul_rn(v, tabs[k * nmax + d]);
    }
    out[p] = v;
}

__global__ void k_dilate(const uint32_t *keys, const double2 *psi, int64_t n, GridDesc g, double eps2,
                         uint64_t *bm, unsigned *block_counts)
{
    int64_t p = gid();
    bool keep = false;
    uint32_t key = 0;
    if (p < n) {
        key = keys[p];
        keep = above_eps(psi[p], eps2);
    }
    set_with_neighbours(g, bm, key, keep);
    count_block(keep, block_counts);
}

// ---- word-parallel dilation (the +-1 stencil on DVR axes) ---------------------
__device__ inline int64_t i64min(int64_t a, int64_t b) { return a < b ? a : b; }
__device__ inline int64_t i64max(int64_t a, int64_t b) { return a > b ? a : b; }

// bits [lo, hi) of a word (0 <= lo, hi <= 64)
__device__ inline uint64_t bit_range(int lo, int hi)
{
    if (hi <= lo) return 0ull;
    const uint64_t up = hi >= 64 ? ~0ull : ((1ull << hi) - 1ull);
    return up & ~((1ull << lo) - 1ull);
}

// the 64 bits of K from bit b on (bits outside the nwords words read 0)
__device__ inline uint64_t bit_window(const uint64_t *K, int64_t nwords, int64_t b)
{
    const int64_t q = b >> 6;  // rounds down for negative b
    const int r = (int)(b & 63);
    const uint64_t lo = (q >= 0 && q < nwords) ? K[q] : 0ull;
    if (r == 0) return lo;
    const uint64_t hi = (q + 1 >= 0 && q + 1 < nwords) ? K[q + 1] : 0ull;
    return (lo >> r) | (hi << (64 - r));
}

// K: one bit per function above the threshold (and the block counts of them)
__global__ void k_mark_kept(const uint32_t *keys, const double2 *psi, int64_t n, double eps2, uint64_t *K,
                            unsigned *block_counts)
{
    int64_t p = gid();
    bool keep = false;
    uint32_t key = 0;
    if (p < n) {
        key = keys[p];
        keep = above_eps(psi[p], eps2);
    }
    set_bit_wave(K, key, keep);
    count_block(keep, block_counts);
}

// bm = K with every +-1 neighbour on one axis: the neighbours one stride s_k
// below are K read s_k bits earlier, kept where the key's digit k is not 0
// (one stride above: not n_k - 1).  With P = s_k n_k, digit k is 0 on the
// runs [m P, m P + s_k) and n_k - 1 on [(m + 1) P - s_k, (m + 1) P).  A
// wavefront takes I rows of 64 consecutive words; each lane keeps, per
// dimension, the position of its word's first bit within the period and
// advances it by 64 words' worth per row (no division per word).  Every word
// is written, the grid's tail bits cleared.
// A block's words are one tile of the popcount scan that follows: it leaves the
// tile's sum, so the scan reads the new bitmap once less; the last block adds
// up the block counts of the functions kept.
static_assert(TB == SB, "a block dilates one scan tile");
template <int I>
__global__ __launch_bounds__(TB) void k_dilate_words(const uint64_t *K, int64_t nwords, GridDesc g, uint64_t *bm,
                                                     uint32_t *tile_sums, const unsigned *block_counts, int64_t ncounts,
                                                     unsigned long long *nabove)
{
    __shared__ unsigned long long s_sum[TB / 64];
    const int lane = threadIdx.x & 63;
    const int64_t w0 = (gid() >> 6) * 64 * I + lane;
    int64_t pos[MAXD], inc[MAXD];
#pragma unroll
    for (int k = 0; k < MAXD; ++k) {
        pos[k] = 0;
        inc[k] = 0;
        if (k < g.D) {
            // (keys are below 2^32; lanes past the end are not used)
            const uint32_t P = g.stride[k] * (uint32_t)g.n[k];
            pos[k] = w0 < nwords ? (int64_t)((uint32_t)(w0 * 64) % P) : 0;
            inc[k] = I > 1 ? (int64_t)((uint32_t)(64 * 64) % P) : 0;
        }
    }
    uint32_t bits = 0;
    for (int it = 0; it < I; ++it) {
        const int64_t w = w0 + (int64_t)it * 64;
        if (w >= nwords) break;
        const int64_t a = w * 64;
        uint64_t acc = K[w];
#pragma unroll
        for (int k = 0; k < MAXD; ++k) {
            if (k < g.D) {
                const int64_t st = g.stride[k], P = st * g.n[k];
                const uint64_t below = bit_window(K, nwords, a - st), above = bit_window(K, nwords, a + st);
                if (below | above) {  // (most of a large grid is empty)
                    uint64_t zm = 0ull, tm = 0ull;
                    for (int64_t r0 = -pos[k]; r0 < 64; r0 += P) {
                        if (r0 + st > 0) zm |= bit_range((int)i64max(r0, 0), (int)i64min(r0 + st, 64));
                        const int64_t ts = r0 + P - st;
                        if (r0 + P > 0 && ts < 64) tm |= bit_range((int)i64max(ts, 0), (int)i64min(r0 + P, 64));
                    }
                    acc |= (below & ~zm) | (above & ~tm);
                }
                pos[k] += inc[k];
                if (pos[k] >= P) pos[k] -= P;
            }
        }
        const int64_t tail = (int64_t)g.total - a;
        if (tail < 64) acc &= tail > 0 ? ((1ull << tail) - 1ull) : 0ull;
        bm[w] = acc;
        if (w == nwords - 1) bm[nwords] = bm[nwords + 1] = 0ull;
        bits += (uint32_t)__popcll(acc);
    }
    uint32_t tot;
    block_excl_scan<TB>(bits, &tot);
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = tot;
    if (blockIdx.x != gridDim.x - 1) return;
    unsigned long long c = 0;
    for (int64_t i = threadIdx.x; i < ncounts; i += TB) c += block_counts[i];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
    if (lane == 0) s_sum[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int i = 0; i < TB / 64; ++i) t += s_sum[i];
        *nabove = t;
    }
}

// Relative exclusion (Sec. II.E): counts the current functions whose bit the
// dilated set leaves clear, i.e. those adaption would drop (block counts).
__global__ void k_count_dropped(const uint32_t *keys, int64_t n, const uint64_t *bm, unsigned *block_counts)
{
    int64_t p = gid();
    bool drop = false;
    if (p < n) {
        uint32_t key = keys[p];
        drop = ((bm[key >> 6] >> (key & 63)) & 1ull) == 0ull;
    }
    count_block(drop, block_counts);
}

// Keeps every current function when no more than rel * n of them would be
// dropped: functions go only if more than that fraction goes.  The test reads
// one device value, so it is uniform over the grid.
__global__ void k_keep_all_if(const uint32_t *keys, int64_t n, uint64_t *bm, const unsigned long long *dropped,
                              double rel)
{
    if ((double)*dropped > rel * (double)n) return;
    int64_t p = gid();
    set_bit_wave(bm, p < n ? keys[p] : 0u, p < n);
}

__global__ void k_mark(const uint32_t *keys, int64_t n, uint64_t *bm)
{
    int64_t p = gid();
    if (p < n) set_bit(bm, keys[p]);
}

// The scan's last pass and the compaction in one: every word's prefix (as
// k_scan_apply) and the keys of its bits; K, with K, is cleared for the next adaption.
template <int I>
__global__ __launch_bounds__(SB) void k_apply_compact(const uint64_t *bm, int64_t nwords, const uint32_t *tile_off,
                                                      uint32_t *prefix, uint32_t *keys_out, uint64_t *K)
{
    constexpr int NW = SB / 64;
    __shared__ uint32_t wsum[I * NW];
    const int64_t base = (int64_t)blockIdx.x * (SB * I) + threadIdx.x;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint64_t word[I];
    uint32_t inc[I];
#pragma unroll
    for (int i = 0; i < I; ++i) word[i] = (base + (int64_t)i * SB < nwords) ? bm[base + (int64_t)i * SB] : 0ull;
#pragma unroll
    for (int i = 0; i < I; ++i) {
        inc[i] = wave_incl_scan((uint32_t)__popcll(word[i]));
        if (lane == 63) wsum[i * NW + w] = inc[i];
    }
    __syncthreads();
    uint32_t off = tile_off[blockIdx.x];
#pragma unroll
    for (int i = 0; i < I; ++i) {
        uint32_t before = 0, row = 0;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            const uint32_t t = wsum[i * NW + ww];
            before += ww < w ? t : 0u;
            row += t;
        }
        const int64_t idx = base + (int64_t)i * SB;
        if (idx < nwords) {
            uint32_t q = off + before + inc[i] - (uint32_t)__popcll(word[i]);
            prefix[idx] = q;
            if (K) K[idx] = 0ull;
            for (uint64_t b = word[i]; b; b &= b - 1)
                keys_out[q++] = (uint32_t)(idx * 64 + (__ffsll((unsigned long long)b) - 1));
        }
        off += row;
    }
}

__global__ void k_remap(const uint32_t *okeys, const double2 *opsi, int64_t n_old, const uint64_t *bm,
                        const uint32_t *prefix, double2 *npsi)
{
    int64_t p = gid();
    if (p >= n_old) return;
    uint32_t key = okeys[p];
    uint64_t word = bm[key >> 6];
    uint32_t b = key & 63;
    if ((word >> b) & 1ull) {
        uint32_t q = prefix[key >> 6] + (uint32_t)__popcll(word & ((1ull << b) - 1ull));
        npsi[q] = opsi[p];
    }
}

// The carried-over values of an adaption in two launches: zeros (psi) and NaN
// (V, optional) for every new function, then every old function's values at
// its rank in the new set.
template <class T>
__global__ void k_fill_new(double2 *psi, T *V, int64_t n, T nan)
{
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * blockDim.x) {
        psi[p] = make_double2(0.0, 0.0);
        if (V) V[p] = nan;
    }
}

template <class T>
__global__ void k_remap_all(const uint32_t *okeys, const double2 *opsi, const T *oV, int64_t n_old, const uint64_t *bm,
                            const uint32_t *prefix, double2 *npsi, T *nV)
{
    const int64_t p = gid();
    if (p >= n_old) return;
    const uint32_t key = okeys[p];
    const uint64_t word = bm[key >> 6];
    const uint32_t first = prefix[key >> 6], b = key & 63;
    const double2 c = opsi[p];
    const T v = nV ? oV[p] : T(0);
    if ((word >> b) & 1ull) {
        const uint32_t q = first + (uint32_t)__popcll(word & ((1ull << b) - 1ull));
        npsi[q] = c;
        if (nV) nV[q] = v;
    }
}

// ---- fiber tables ------------------------------------------------------------
__global__ void k_last_flags(const uint32_t *keys, int64_t n, int nl, uint32_t *flags)
{
    int64_t p = gid();
    if (p >= n) return;
    flags[p] = (p == 0 || keys[p] / (uint32_t)nl != keys[p - 1] / (uint32_t)nl) ? 1u : 0u;
}

// info[p] = the digit, with the fiber-start flag in bit 7 (dimensions of at
// most 64 points); a longer dimension (up to 256 points) keeps the digit alone
__global__ void k_last_info(const uint32_t *keys, int64_t n, int nl, uint8_t *info)
{
    int64_t p = gid();
    if (p >= n) return;
    bool start = (p == 0 || keys[p] / (uint32_t)nl != keys[p - 1] / (uint32_t)nl);
    const uint32_t flag = (start && nl <= NMAX_MASK) ? 0x80u : 0u;
    info[p] = (uint8_t)((keys[p] % (uint32_t)nl) | flag);
}

// mask[0, *nf) = 0 (the fiber count is on the device)
__global__ void k_zero_masks(uint64_t *mask, const uint32_t *nf)
{
    const int64_t m = *nf;
    for (int64_t i = gid(); i < m; i += (int64_t)gridDim.x * blockDim.x) mask[i] = 0ull;
}

// One thread per point: the fiber start writes off; every point's digit bit
// is ORed over the wavefront's consecutive lanes of its fiber and the
// segment's last lane adds it to the (zeroed) mask, so a fiber costs one or
// two atomics however its points fall over the wavefronts.  A dimension
// longer than a mask word keeps no mask.
__global__ void k_last_fill(const uint32_t *keys, int64_t n, int nl, const uint32_t *flags, const uint32_t *fidx,
                            const uint32_t *nf, uint32_t *off, uint64_t *mask)
{
    const int64_t p = gid();
    const int lane = threadIdx.x & 63;
    if (p == 0) off[*nf] = (uint32_t)n;
    const bool valid = p < n;
    uint32_t f = 0xffffffffu;
    uint64_t bits = 0ull;
    if (valid) {
        const uint32_t st = flags[p];
        f = fidx[p] - (st ? 0u : 1u);  // fidx counts the starts before p
        if (st) off[f] = (uint32_t)p;
        if (nl <= NMAX_MASK) bits = 1ull << (keys[p] % (uint32_t)nl);
    }
    if (nl > NMAX_MASK) return;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t of = __shfl_up(f, d, 64);
        const uint32_t lo = __shfl_up((uint32_t)bits, d, 64), hi = __shfl_up((uint32_t)(bits >> 32), d, 64);
        if (lane >= d && of == f) bits |= ((uint64_t)hi << 32) | lo;
    }
    const uint32_t nxt = __shfl_down(f, 1, 64);
    if (valid && (lane == 63 || nxt != f)) atomicOr((unsigned long long *)&mask[f], (unsigned long long)bits);
}

__device__ inline uint32_t rotate_key(uint32_t key, uint32_t sk, uint32_t nk, uint32_t *dig)
{
    uint32_t hi = key / (sk * nk);
    uint32_t rem = key - hi * sk * nk;
    uint32_t d = rem / sk, lo = rem - d * sk;
    *dig = d;
    return (hi * sk + lo) * nk + d;
}

// bits [base, base+len) of the bitmap, len <= 64
__device__ inline uint64_t extract_bits(const uint64_t *bm, uint32_t base, int len)
{
    uint32_t w0 = base >> 6, sh = base & 63;
    uint64_t v = bm[w0] >> sh;
    if (sh != 0 && sh + (uint32_t)len > 64) v |= bm[w0 + 1] << (64 - sh);
    return len == 64 ? v : (v & ((1ull << len) - 1ull));
}

// Key of a point in the frame whose digit order is (inner digits, outer
// digits): with S_in the product of the inner sizes and N_out = total / S_in,
// the frame key is (key mod S_in) * N_out + key / S_in.  rin == 0 keeps the
// row-major frame.
__device__ inline uint32_t frame_key(uint32_t key, uint32_t rin, uint32_t rout)
{
    return rin ? (key % rin) * rout + key / rin : key;
}

__global__ void k_rot_set(const uint32_t *keys, int64_t n, uint32_t sk, uint32_t nk, uint32_t rin, uint32_t rout,
                          uint64_t *bm)
{
    int64_t p = gid();
    uint32_t d, rk = 0;
    if (p < n) rk = rotate_key(frame_key(keys[p], rin, rout), sk, nk, &d);
    set_bit_wave(bm, rk, p < n);
}

// q = rank of the point in the rotated order.  pi[q] receives map[p] (p when
// map is null); inv[p] = q when inv is given.  flags/tmpmask/info describe the
// fibers along the rotated (last) digit (info may be null).
__global__ void k_rot_rank(const uint32_t *keys, int64_t n, uint32_t sk, uint32_t nk, uint32_t rin, uint32_t rout,
                           const uint64_t *bm, const uint32_t *prefix, const uint32_t *map, uint32_t *pi,
                           uint32_t *inv, uint32_t *flags, uint64_t *tmpmask, uint8_t *info)
{
    int64_t p = gid();
    if (p >= n) return;
    uint32_t d;
    uint32_t rk = rotate_key(frame_key(keys[p], rin, rout), sk, nk, &d);
    uint64_t word = bm[rk >> 6];
    uint32_t q = prefix[rk >> 6] + (uint32_t)__popcll(word & ((1ull << (rk & 63)) - 1ull));
    pi[q] = map ? map[p] : (uint32_t)p;
    if (inv) inv[p] = q;
    if (nk > (uint32_t)NMAX_MASK) {
        // a dimension longer than a mask word: the entry starts a fiber when no
        // bit of its fiber lies below it; info keeps the digit alone
        bool start = true;
        for (uint32_t b = rk - d; b < rk && start; b = (b | 63u) + 1u) {
            const uint32_t e = (b | 63u) + 1u < rk ? (b | 63u) + 1u : rk;
            const uint64_t w = bm[b >> 6] >> (b & 63u);
            const uint32_t len = e - b;
            start = (len >= 64 ? w : (w & ((1ull << len) - 1ull))) == 0;
        }
        flags[q] = start ? 1u : 0u;
        if (info) info[q] = (uint8_t)d;
        return;
    }
    uint64_t m = extract_bits(bm, rk - d, (int)nk);
    bool start = (m & ((1ull << d) - 1ull)) == 0;
    flags[q] = start ? 1u : 0u;
    if (start) tmpmask[q] = m;
    if (info) info[q] = (uint8_t)(d | (start ? 0x80u : 0u));
}

// ---- fiber tables of every dimension in one set of launches --------------------
// From the set's row-major bitmap and its prefix, tile by tile.
// A tile of dimension k: the fibers of up to 64 consecutive keys below digit k, so
// digit d of all of them is a run of bits, and n_k runs hold the tile.  No rotated
// bitmap is formed: a first pass counts each tile's points and fibers (a thread per
// tile, neighbours read neighbouring words), one scan numbers them, and a second
// pass writes the tiles that hold points.  There a lane is a fiber: the runs, loaded
// a digit per lane, are read from lane to lane, a point's position is its run's rank
// plus the run's bits below the lane, and the permutation leaves through LDS in
// contiguous stores.  Bound by the instructions of the second pass.  Measured, 4M
// functions of a 24^6 grid (950K tiles): 15 us for the bitmap, 58 for the counts, 124
// for the tiles (rotated bitmaps, a walk over them in rank order and four passes over
// the points for the last dimension, before: 173, 236 and 50); 108K of 48^4 6 and 11
// (38 the walk); 33K of 24^3 x 8, a build
// with its waits 134 (173).
// Of the last dimension `base` is the first fiber's first key, `len` the fibers.
__device__ inline void tile_of(const TileAll &r, uint32_t tile, int &k, uint32_t &base, int &len)
{
    k = 0;
    while (tile >= r.first[k + 1]) ++k;
    const uint32_t i = tile - r.first[k], hi = i / r.per[k], lo = (i - hi * r.per[k]) * 64u;
    const uint32_t row = k + 1 < r.nd ? r.sk[k] : r.fibers;
    base = k + 1 < r.nd ? hi * r.nk[k] * r.sk[k] + lo : lo * r.nk[k];
    len = (int)(row - lo < 64u ? row - lo : 64u);
}

// S lanes share a tile's digits: one while there are tiles enough for every SIMD.
// The blocks from `wide` on take the last dimension, a wavefront LAST_TILES of its
// tiles, a lane per fiber (only the fibers are counted: its points are in key order).
constexpr int LAST_TILES = 4;
template <int S>
__global__ __launch_bounds__(TB) void k_tile_count(TileAll r, unsigned wide, const uint64_t *bm, uint32_t *cnt)
{
    const uint32_t nt = r.first[r.nd], end = r.first[r.nd - 1];
    int k, len;
    uint32_t base;
    if (blockIdx.x >= wide) {
        const int lane = threadIdx.x & 63;
        const uint32_t wave = (blockIdx.x - wide) * (TB / 64) + (threadIdx.x >> 6);
#pragma unroll
        for (int u = 0; u < LAST_TILES; ++u) {
            const uint32_t tile = end + wave * LAST_TILES + u;
            if (tile >= nt) break;
            tile_of(r, tile, k, base, len);
            const uint64_t v = lane < len ? extract_bits(bm, base + (uint32_t)lane * r.nk[k], (int)r.nk[k]) : 0ull;
            const uint32_t c = (uint32_t)__popcll(__ballot(v != 0));
            if (lane == 0) cnt[tile] = cnt[nt + tile] = c;
        }
        return;
    }
    const uint32_t tile = (uint32_t)(gid() / S), sub = (uint32_t)(gid() % S);
    if (tile >= end) return;
    tile_of(r, tile, k, base, len);
    uint64_t any = 0;
    uint32_t points = 0;
    const uint32_t nk = r.nk[k], sk = r.sk[k];
#pragma unroll 16
    for (uint32_t d = sub; d < nk; d += S) {
        const uint64_t v = extract_bits(bm, base + d * sk, len);
        any |= v;
        points += (uint32_t)__popcll(v);
    }
#pragma unroll
    for (int x = 1; x < S; x <<= 1) {
        points += __shfl_xor(points, x, 64);
        any |= ((uint64_t)__shfl_xor((uint32_t)(any >> 32), x, 64) << 32) | __shfl_xor((uint32_t)any, x, 64);
    }
    if (sub == 0) {
        cnt[tile] = points;
        cnt[nt + tile] = (uint32_t)__popcll(any);
    }
}

__device__ inline uint64_t readlane64(uint64_t v, int l)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
}
__device__ inline uint32_t bits_below_lane(uint64_t v)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(v >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)v, 0u));
}

// smem: 64 max(n_k) positions per wavefront
__global__ __launch_bounds__(TB) void k_tile_fill(TileAll r, uint32_t n, int nmax, int group, const uint64_t *bm, const uint32_t *prefix,
                                                  const uint32_t *cnt, const uint32_t *offs, const uint32_t *total,
                                                  TabPtrs t, uint32_t *nf)
{
    extern __shared__ uint32_t s_pos[];
    const uint32_t nt = r.first[r.nd];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t *sl = s_pos + wave * 64 * nmax;
    if (blockIdx.x == 0 && (int)threadIdx.x < r.nd) {
        // the dimension's fibers and the end of its last one
        const int k = threadIdx.x;
        const uint32_t end = k + 1 < r.nd ? offs[nt + r.first[k + 1]] : *total;
        nf[k] = end - offs[nt + r.first[k]];
        t.off[k][nf[k]] = n;
    }
    const uint32_t t0 = ((uint32_t)blockIdx.x * (TB / 64) + (uint32_t)wave) * (uint32_t)group;
    uint64_t todo = __ballot(lane < group && t0 + lane < nt && cnt[t0 + lane] != 0);
    for (; todo; todo &= todo - 1) {
        const uint32_t tile = t0 + (uint32_t)(__ffsll((unsigned long long)todo) - 1);
        int k, len;
        uint32_t base;
        tile_of(r, tile, k, base, len);
        const uint32_t nk = r.nk[k], sk = r.sk[k];
        // (the counts before the tile's dimension: n points each)
        const uint32_t q0 = offs[tile] - (uint32_t)k * n, f0 = offs[nt + tile] - offs[nt + r.first[k]];
        if (k + 1 == r.nd) {
            // the fibers' windows lie one after the other, their points in key order
            uint64_t m = 0;
            uint32_t q = 0;
            if (lane < len) {
                const uint32_t at = base + (uint32_t)lane * nk;
                m = extract_bits(bm, at, (int)nk);
                q = prefix[at >> 6] + (uint32_t)__popcll(bm[at >> 6] & ((1ull << (at & 63)) - 1ull));
            }
            const uint64_t fibers = __ballot(m != 0);
            if (m) {
                const uint32_t f = f0 + bits_below_lane(fibers);
                t.off[k][f] = q;
                t.mask[k][f] = m;
            }
            uint8_t *si = reinterpret_cast<uint8_t *>(sl);
            const int first = __ffsll((unsigned long long)fibers) - 1, last = 63 - __clzll((long long)fibers);
            const uint32_t p0 = __shfl(q, first, 64), points = __shfl(q + (uint32_t)__popcll(m), last, 64) - p0;
            uint32_t at = q - p0, start = 0x80u;
            for (uint64_t x = m; x; x &= x - 1) {
                si[at++] = (uint8_t)((uint32_t)(__ffsll((unsigned long long)x) - 1) | start);
                start = 0;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (uint32_t i = (uint32_t)lane; i < points; i += 64) t.info[p0 + i] = si[i];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            continue;
        }
        uint64_t run = 0;
        uint32_t rank = 0;
        if ((uint32_t)lane < nk) {
            const uint32_t at = base + (uint32_t)lane * sk, w = at >> 6, sh = at & 63;
            const uint64_t lo = bm[w], hi = bm[w + 1];
            run = sh ? (lo >> sh) | (hi << (64 - sh)) : lo;
            if (len < 64) run &= (1ull << len) - 1ull;
            rank = prefix[w] + (uint32_t)__popcll(lo & ((1ull << sh) - 1ull));
        }
        const uint64_t digits = __ballot(run != 0);
        uint64_t m = 0;
        for (uint64_t x = digits; x; x &= x - 1) {
            const int d = __ffsll((unsigned long long)x) - 1;
            if (__builtin_amdgcn_inverse_ballot_w64(readlane64(run, d))) m |= 1ull << d;
        }
        const uint32_t c = (uint32_t)__popcll(m), incl = wave_incl_scan(c), points = __shfl(incl, 63, 64);
        const uint64_t fibers = __ballot(m != 0);
        if (m) {
            const uint32_t f = f0 + bits_below_lane(fibers);
            t.off[k][f] = q0 + incl - c;
            t.mask[k][f] = m;
        }
        uint32_t at = incl - c;
        for (uint64_t x = digits; x; x &= x - 1) {
            const int d = __ffsll((unsigned long long)x) - 1;
            const uint64_t v = readlane64(run, d);
            const uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)rank, d) + bits_below_lane(v);
            if (__builtin_amdgcn_inverse_ballot_w64(v)) sl[at++] = pos;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (uint32_t i = (uint32_t)lane; i < points; i += 64) t.pi[k][q0 + i] = sl[i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// ---- the same tables from rotated bitmaps --------------------------------------
// Where the last dimensions are short a tile holds few lanes (s_k of 64), and there
// are more tiles than words in the bitmap.  Then every dimension but the last has a
// bitmap of its own with digit k moved last, one after the other, and the row-major
// bitmap of the set after them, each nwords long.  Every bitmap holds exactly n bits
// (rotation permutes the keys), so one prefix over all of them gives bitmap k's ranks
// offset by k n.  Bound by the passes over the bitmaps: 64^4 x 5^2 (17.3M tiles, 6.6M
// words) with 12K functions 0.4 ms instead of 1.2, 64^4 x 4^3 (85M tiles, 16.8M words)
// with 750K 1.4 instead of 5.8.
__global__ void k_rot_set_all(const uint32_t *keys, int64_t n, RotAll r, uint64_t *bm, uint64_t *occ)
{
    int64_t p = gid();
    const bool valid = p < n;
    const uint32_t key = valid ? keys[p] : 0u;
    for (int k = 0; k < r.nd; ++k) {
        uint32_t d, rk = 0;
        if (valid) rk = rotate_key(key, r.sk[k], r.nk[k], &d);
        set_bit_wave(bm + (int64_t)k * r.nwords, rk, valid);
        // the point's fiber slot (the rotated key without its last digit)
        set_bit_wave(occ + r.owoff[k], rk / r.nk[k], valid);
    }
    // segment nd: the row-major bitmap of the set itself (point positions)
    set_bit_wave(bm + (int64_t)r.nd * r.nwords, key, valid);
}

// The r-th (0-based) set bit of v (r < popcount(v)): six halving steps.
__device__ inline int select_bit(uint64_t v, int r)
{
    int pos = 0;
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) {
        const int c = __popcll(v & ((1ull << sh) - 1ull));
        if (r >= c) {
            r -= c;
            v >>= sh;
            pos += sh;
        }
    }
    return pos;
}

// Rank order gather: the rotated bitmaps are walked word by word, so the
// points of dimension k come out in rank order q and every table write is
// contiguous.  A wavefront takes 64 consecutive words of the concatenated
// rotated segments; their set bits are dealt out to the lanes 64 at a time
// (a dense word's bits spread over the wavefront instead of one lane).  For
// the bit of rotated key rk: q from the segment's prefix, the point's
// position p from the row-major segment (rank of the un-rotated key), the
// fiber start and mask from the n_k-bit window holding rk, and the fiber's
// number from the rank of its slot among the occupied ones.
__global__ __launch_bounds__(TB) void k_rank_gather(int64_t n, RotAll r, const uint64_t *bm, const uint32_t *prefix,
                                                    const uint64_t *occ, const uint32_t *oprefix, TabPtrs t)
{
    __shared__ uint64_t s_word[TB];
    __shared__ uint32_t s_off[TB];
    __shared__ uint32_t s_q0[TB];
    __shared__ uint32_t s_w[TB];
    const int lane = threadIdx.x & 63, wbase = threadIdx.x & ~63;
    const int64_t nw = (int64_t)r.nd * r.nwords;
    const int64_t w = (int64_t)blockIdx.x * TB + threadIdx.x;
    uint64_t word = 0;
    uint32_t q0 = 0;
    if (w < nw) {
        word = bm[w];
        const int k = (int)(w / r.nwords);
        q0 = prefix[w] - (uint32_t)((int64_t)k * n);
    }
    const uint32_t cnt = (uint32_t)__popcll(word);
    // exclusive prefix of the counts over the wavefront
    uint32_t incl = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
    }
    const uint32_t total = __shfl(incl, 63, 64);
    s_word[threadIdx.x] = word;
    s_off[threadIdx.x] = incl - cnt;
    s_q0[threadIdx.x] = q0;
    s_w[threadIdx.x] = (uint32_t)(w < nw ? w % r.nwords : 0);
    __syncthreads();
    const uint64_t *rowm = bm + nw;            // row-major segment
    const uint32_t *rowp = prefix + nw;
    const uint32_t rbase = (uint32_t)((int64_t)r.nd * n);
    for (uint32_t b0 = 0; b0 < total; b0 += 64) {
        const uint32_t b = b0 + lane;
        if (b >= total) break;
        // source lane: the last lane whose offset is <= b (offsets ascend)
        int lo = 0, hi = 63;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (s_off[wbase + mid] <= b) lo = mid;
            else hi = mid - 1;
        }
        const int src = wbase + lo;
        const int rr = (int)(b - s_off[src]);
        const uint64_t sw = s_word[src];
        const int pos = select_bit(sw, rr);
        const int64_t wg = (int64_t)blockIdx.x * TB + src;  // global word index
        const int k = (int)(wg / r.nwords);
        const uint32_t rk = s_w[src] * 64u + (uint32_t)pos;
        const uint32_t q = s_q0[src] + (uint32_t)rr;
        // un-rotate: rk = (hi * sk + lo) * nk + d  ->  key = (hi * nk + d) * sk + lo
        const uint32_t nk = r.nk[k], sk = r.sk[k];
        const uint32_t d = rk % nk, tq = rk / nk;
        const uint32_t khi = tq / sk, klo = tq - khi * sk;
        const uint32_t key = (khi * nk + d) * sk + klo;
        const uint32_t p = rowp[key >> 6] - rbase +
                           (uint32_t)__popcll(rowm[key >> 6] & ((1ull << (key & 63)) - 1ull));
        t.pi[k][q] = p;
        const uint64_t *seg = bm + (int64_t)k * r.nwords;
        const uint64_t m = extract_bits(seg, rk - d, (int)nk);
        if ((m & ((1ull << d) - 1ull)) == 0) {
            // the fiber's first point: its slot tq's rank among the occupied slots
            const int64_t o0 = r.owoff[k], ow = o0 + (tq >> 6);
            const uint32_t f = oprefix[ow] - oprefix[o0] + (uint32_t)__popcll(occ[ow] & ((1ull << (tq & 63)) - 1ull));
            t.off[k][f] = q;
            t.mask[k][f] = m;
        }
    }
}

// Per dimension: the fiber count (occupied slots) and the end sentinel
// off_k[nf_k] = n.  `total` is the occupancy scan's total over all dimensions.
__global__ void k_occ_counts(const uint32_t *oprefix, int64_t n, RotAll r, const uint32_t *total, TabPtrs t,
                             uint32_t *nf)
{
    const int k = threadIdx.x;
    if (k >= r.nd) return;
    const uint32_t b0 = oprefix[r.owoff[k]];
    const uint32_t b1 = (k + 1 < r.nd) ? oprefix[r.owoff[k + 1]] : *total;
    nf[k] = b1 - b0;
    t.off[k][b1 - b0] = (uint32_t)n;
}

// Chunks of whole blocks for the block-fused H*psi.  A block is a maximal run
// of frame positions with the same block id (key / S_in in the row-major frame,
// key mod S_in in the inner-first frame, both non-decreasing along the frame).
// Chunk t starts at the first block start at or after t * S, so every chunk
// holds whole blocks; chunk[nch] = n.  counters[0] counts the chunks longer
// than cap (their indices go to big), counters[1] is the longest chunk.
__device__ inline uint32_t block_id(const uint32_t *keys, const uint32_t *P, uint32_t r, uint32_t sin, int inner)
{
    uint32_t k = keys[P ? P[r] : r];
    return inner ? k % sin : k / sin;
}

__device__ uint32_t chunk_start(const uint32_t *keys, const uint32_t *P, uint32_t n, uint32_t sin, int inner,
                                uint64_t st)
{
    if (st >= n) return n;
    uint32_t r = (uint32_t)st;
    uint32_t id = block_id(keys, P, r, sin, inner);
    if (r == 0 || block_id(keys, P, r - 1, sin, inner) != id) return r;
    uint32_t lo = r + 1, hi = n;
    while (lo < hi) {
        uint32_t mid = lo + (hi - lo) / 2;
        if (block_id(keys, P, mid, sin, inner) == id) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__global__ void k_chunks(const uint32_t *keys, const uint32_t *P, uint32_t n, uint32_t sin, int inner, uint32_t S,
                         uint32_t nch, uint32_t cap, uint32_t *chunk, uint32_t *big, uint32_t *counters)
{
    int64_t t = gid();
    if (t > nch) return;
    uint32_t a = chunk_start(keys, P, n, sin, inner, (uint64_t)t * S);
    chunk[t] = a;
    if (t == nch) return;
    uint32_t b = chunk_start(keys, P, n, sin, inner, (uint64_t)(t + 1) * S);
    uint32_t len = b - a;
    if (len > 0) atomicMax(&counters[1], len);
    if (len > cap) big[atomicAdd(&counters[0], 1u)] = (uint32_t)t;
}

// ---- plane tables (two adjacent dimensions merged into one digit) ------------
// q = the point's rank in the pair's frame (its own position in the identity
// frame, bm == nullptr); P[q] = p, the pair's two digits and the plane key
// (the frame key without the merged digit).
__global__ void k_plane_rank(const uint32_t *keys, int64_t n, uint32_t sk, uint32_t na, uint32_t nb,
                             const uint64_t *bm, const uint32_t *prefix, uint32_t *P, uint16_t *dig, uint32_t *pkey)
{
    int64_t p = gid();
    if (p >= n) return;
    const uint32_t nk = na * nb;
    uint32_t d;
    const uint32_t rk = rotate_key(keys[p], sk, nk, &d);
    uint32_t q = (uint32_t)p;
    if (bm) {
        q = prefix[rk >> 6] + (uint32_t)__popcll(bm[rk >> 6] & ((1ull << (rk & 63)) - 1ull));
        P[q] = (uint32_t)p;
    }
    dig[q] = (uint16_t)(((d / nb) << 8) | (d % nb));
    pkey[q] = rk / nk;
}

// Marks the last member of every plane (bit 15 of its digits).
__global__ void k_plane_flags(const uint32_t *pkey, int64_t n, uint32_t *flags, uint16_t *dig)
{
    int64_t q = gid();
    if (q >= n) return;
    const uint32_t k = pkey[q];
    flags[q] = (q == 0 || k != pkey[q - 1]) ? 1u : 0u;
    if (q == n - 1 || k != pkey[q + 1]) dig[q] = (uint16_t)(dig[q] | 0x8000u);
}

__global__ void k_plane_fill(const uint32_t *flags, const uint32_t *pidx, int64_t n, const uint32_t *np,
                             uint32_t *poff)
{
    int64_t q = gid();
    if (q == 0) poff[*np] = (uint32_t)n;
    if (q < n && flags[q]) poff[pidx[q]] = (uint32_t)q;
}

// Task t starts at the first plane start at or after t S (n for none):
// plane pl starts the tasks t with poff[pl - 1] < t S <= poff[pl].
__global__ void k_plane_tasks(const uint32_t *poff, const uint32_t *np, int64_t n, uint32_t S, uint32_t ntask,
                              uint32_t *tstart)
{
    int64_t pl = gid();
    const uint32_t npl = *np;
    if (pl > (int64_t)npl) return;
    const uint32_t lo = pl == 0 ? 0u : poff[pl - 1] / S + 1u;
    const uint32_t hi = pl == (int64_t)npl ? ntask : poff[pl] / S;
    const uint32_t st = pl == (int64_t)npl ? (uint32_t)n : poff[pl];
    for (uint32_t t = lo; t <= hi && t <= ntask; ++t) tstart[t] = st;
}

// Pair-pass tasks: task t starts at the first plane start at or after t W (n
// if none).  The plane holding position t W ends within nab positions, so one
// wavefront per task looks at positions [t W, t W + nab] only.
__global__ void k_pair_tasks(const uint32_t *keys, int64_t n, uint32_t nab, uint32_t W, uint32_t ntask,
                             uint32_t *tstart)
{
    const int64_t t = gid() >> 6;
    const int lane = threadIdx.x & 63;
    if (t > (int64_t)ntask) return;
    uint32_t st = (uint32_t)n;
    if (t < (int64_t)ntask) {
        const int64_t q0 = t * W, qe = q0 + (int64_t)nab < n - 1 ? q0 + (int64_t)nab : n - 1;
        for (int64_t b = q0; b <= qe; b += 64) {
            const int64_t q = b + lane;
            const bool start = q <= qe && (q == 0 || keys[q] / nab != keys[q - 1] / nab);
            const uint64_t m = __ballot(start);
            if (m) {
                st = (uint32_t)(b + __ffsll((unsigned long long)m) - 1);
                break;
            }
        }
    }
    if (lane == 0) tstart[t] = st;
}

__global__ void k_fib_fill(const uint32_t *flags, const uint32_t *fidx, const uint64_t *tmpmask, int64_t n,
                           const uint32_t *nf, uint32_t *off, uint64_t *mask)
{
    int64_t q = gid();
    if (q == 0) off[*nf] = (uint32_t)n;
    if (q >= n || !flags[q]) return;
    uint32_t f = fidx[q];
    off[f] = (uint32_t)q;
    if (mask) mask[f] = tmpmask[q];
}

// ---- potential cache -----------------------------------------------------------
// Potential cache: V_I = sum_t coef_t prod_f tab_{t,f}[digit_{dim_{t,f}}(I)].
// Term descriptors and the (deduplicated) 1D tables are staged in LDS.
constexpr int POT_MAX_TERMS = 256;
constexpr int POT_MAX_TAB = 2048;
constexpr int POT_MAX_FAC = 4;

// A key's digits, digit k in byte k (a dimension has at most 256 points).
__device__ inline uint64_t packed_digits(uint32_t key, const GridDesc &g)
{
    uint64_t digits = 0;
#pragma unroll
    for (int k = MAXD - 1; k >= 0; --k) {
        if (k < g.D) {
            const uint32_t q = key / (uint32_t)g.n[k];
            digits |= (uint64_t)(key - q * (uint32_t)g.n[k]) << (8 * k);
            key = q;
        }
    }
    return digits;
}

// Grid-stride over the points (or over a list of them, or over those whose value
// is missing): the term descriptors and tables are staged in LDS once per block.
// Bound by the instructions per factor, so a thread takes P points through each
// descriptor, which is read for the whole wavefront, and a point's digits are the
// bytes of one word, shifted by a wave-uniform amount (picking the digit out of an
// array by compares took 366 us over 4M functions with the 41 terms of the
// six-dimensional quartic, this 92).
template <int P>
__global__ __launch_bounds__(TB) void k_potential(const uint32_t *keys, int64_t n, GridDesc g, PotDesc pd, double *V,
                                                  float *Vf, const uint32_t *list, const unsigned *count, int missing)
{
    __shared__ double s_coef[POT_MAX_TERMS];
    __shared__ int s_nf[POT_MAX_TERMS];
    __shared__ int s_fac[POT_MAX_TERMS][POT_MAX_FAC];  // (first entry of the table << 6) | bit of the digit
    __shared__ double s_tab[POT_MAX_TAB];
    for (int t = threadIdx.x; t < pd.nterm; t += TB) {
        int ti[MAXD];
#pragma unroll
        for (int k = 0; k < MAXD; ++k) ti[k] = k < g.D ? pd.tab[t * pd.D + k] : -1;
        s_coef[t] = pd.coef[t];
        int nf = 0;
#pragma unroll
        for (int k = 0; k < MAXD; ++k)
            if (ti[k] >= 0 && nf < POT_MAX_FAC) s_fac[t][nf++] = ((ti[k] * pd.nmax) << 6) | (8 * k);
        s_nf[t] = nf;
    }
    for (int i = threadIdx.x; i < pd.ntab * pd.nmax; i += TB) s_tab[i] = pd.tabs[i];
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * TB;
    const int64_t m = list ? (int64_t)*count : n;
    for (int64_t i = gid(); i < m; i += P * stride) {
        int64_t p[P];
        uint64_t digits[P];
        double v[P];
        bool any = false;
#pragma unroll
        for (int u = 0; u < P; ++u) {
            const int64_t j = i + u * stride;
            p[u] = j < m ? (list ? (int64_t)list[j] : j) : -1;
            if (missing && p[u] >= 0 && (V ? V[p[u]] == V[p[u]] : Vf[p[u]] == Vf[p[u]])) p[u] = -1;
            any = any || p[u] >= 0;
        }
        if (!any) continue;
#pragma unroll
        for (int u = 0; u < P; ++u) {
            digits[u] = packed_digits(p[u] >= 0 ? keys[p[u]] : 0u, g);
            v[u] = 0.0;
        }
        for (int t = 0; t < pd.nterm; ++t) {
            const double c = s_coef[t];
            double f[P];
#pragma unroll
            for (int u = 0; u < P; ++u) f[u] = c;
            const int nf = __builtin_amdgcn_readfirstlane(s_nf[t]);
#pragma unroll
            for (int j = 0; j < POT_MAX_FAC; ++j) {
                if (j < nf) {
                    const int e = __builtin_amdgcn_readfirstlane(s_fac[t][j]);
                    const double *tab = s_tab + (e >> 6);
#pragma unroll
                    for (int u = 0; u < P; ++u) f[u] *= tab[(uint32_t)(digits[u] >> (e & 63)) & 255u];
                }
            }
#pragma unroll
            for (int u = 0; u < P; ++u) v[u] += f[u];
        }
#pragma unroll
        for (int u = 0; u < P; ++u) {
            if (p[u] < 0) continue;
            if (V) V[p[u]] = v[u];
            if (Vf) Vf[p[u]] = (float)v[u];
        }
    }
}

// Positions whose potential is missing (NaN) into list.  Each block takes a
// contiguous range: it counts, reserves its segment with one atomic (block
// segments in any order), then writes its positions in order.
template <class T>
__global__ __launch_bounds__(TB) void k_missing(const T *V, int64_t n, uint32_t *list, unsigned *count)
{
    __shared__ unsigned s_w[TB / 64];
    __shared__ unsigned s_base, s_run;
    const int64_t per = (n + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * per;
    const int64_t hi = lo + per < n ? lo + per : n;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    unsigned c = 0;
    for (int64_t p = lo + threadIdx.x; p < hi; p += TB) c += (V[p] == V[p]) ? 0u : 1u;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
    if (lane == 0) s_w[w] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned tot = 0;
        for (int i = 0; i < TB / 64; ++i) tot += s_w[i];
        s_base = tot ? atomicAdd(count, tot) : 0u;
        s_run = 0u;
    }
    __syncthreads();
    for (int64_t p0 = lo; p0 < hi; p0 += TB) {
        const int64_t p = p0 + threadIdx.x;
        const bool miss = p < hi && !(V[p] == V[p]);
        const uint64_t b = __ballot(miss);
        if (lane == 0) s_w[w] = (unsigned)__popcll(b);
        __syncthreads();
        unsigned off = s_base + s_run;
        for (int i = 0; i < w; ++i) off += s_w[i];
        if (miss) list[off + (unsigned)__popcll(b & ((1ull << lane) - 1ull))] = (uint32_t)p;
        __syncthreads();
        if (threadIdx.x == 0)
            for (int i = 0; i < TB / 64; ++i) s_run += s_w[i];
        __syncthreads();
    }
}

// ---- Krylov vectors ---------------------------------------------------------------
__global__ __launch_bounds__(TB) void k_dot_partial(const double2 *a, const double2 *b, int64_t n,
                                                    double2 *partial)
{
    double2 acc[1] = {make_double2(0.0, 0.0)};
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) cdot_acc(acc[0], a[p], b[p]);
    block_reduce_store<1>(acc, partial);
}

// ---- autocorrelation at twice the time --------------------------------------------
// sum_I c_I^2 (no conjugate): C(2t) = <psi(t)*|psi(t)> when the initial packet
// is real and the operator real symmetric (Eq. acorr and the text after it).
__global__ __launch_bounds__(TB) void k_sq_partial(const double2 *psi, int64_t n, double2 *partial)
{
    double2 acc[1] = {make_double2(0.0, 0.0)};
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) {
        const double2 c = psi[p];
        acc[0].x = fma(c.x, c.x, fma(-c.y, c.y, acc[0].x));
        acc[0].y = fma(2.0 * c.x, c.y, acc[0].y);
    }
    block_reduce_store<1>(acc, partial);
}

// fixed-order sum of the first partial of nb blocks into *out
__global__ __launch_bounds__(TB) void k_sum_partial1(const double2 *partial, int nb, double2 *out)
{
    __shared__ double2 red[TB];
    double2 s = make_double2(0.0, 0.0);
    for (int b = threadIdx.x; b < nb; b += TB) {
        s.x += partial[pidx(b, 0)].x;
        s.y += partial[pidx(b, 0)].y;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = TB / 2; st >= 1; st >>= 1) {
        if ((int)threadIdx.x < st) {
            red[threadIdx.x].x += red[threadIdx.x + st].x;
            red[threadIdx.x].y += red[threadIdx.x + st].y;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// ---- observables ------------------------------------------------------------------
__global__ __launch_bounds__(TB) void k_obs_partial(const uint32_t *keys, const double2 *psi, int64_t n, GridDesc g,
                                                    const double2 *bra, int nmax, double eps2, double2 *partial)
{
    // the 1D tables of the reference packet (at most MAXD x 64 entries) in LDS
    __shared__ double2 sbra[MAXD * NMAX_FIBER];
    for (int i = threadIdx.x; i < g.D * nmax; i += TB) sbra[i] = bra[i];
    __syncthreads();
    double2 acc[3] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
    // OBS_U points per thread and pass, every load issued before the first
    // use (one memory latency per pass instead of one per point)
    constexpr int OBS_U = 4;
    const int64_t stride = (int64_t)gridDim.x * TB;
    for (int64_t p0 = gid(); p0 < n; p0 += stride * OBS_U) {
        double2 c[OBS_U];
        uint32_t key[OBS_U];
#pragma unroll
        for (int u = 0; u < OBS_U; ++u) {
            const int64_t p = p0 + u * stride;
            c[u] = p < n ? psi[p] : make_double2(0.0, 0.0);
            key[u] = p < n ? keys[p] : 0u;
        }
        double2 v[OBS_U];
#pragma unroll
        for (int u = 0; u < OBS_U; ++u) v[u] = make_double2(1.0, 0.0);
        for (int k = 0; k < g.D; ++k) {
#pragma unroll
            for (int u = 0; u < OBS_U; ++u) {
                const int d = (int)((key[u] / g.stride[k]) % (uint32_t)g.n[k]);
                v[u] = cmul(v[u], sbra[k * nmax + d]);
            }
        }
#pragma unroll
        for (int u = 0; u < OBS_U; ++u) {
            if (p0 + u * stride >= n) continue;
            acc[0].x = fma(c[u].x, c[u].x, fma(c[u].y, c[u].y, acc[0].x));
            cdot_acc(acc[1], v[u], c[u]);
            if (above_eps(c[u], eps2)) acc[2].x += 1.0;
        }
    }
    block_reduce_store<3>(acc, partial);
}

// The record's sums, with the fields that the host knows (and the order from
// KState where only the device knows it).
__global__ __launch_bounds__(TB) void k_obs_final(const double2 *partial, int nb, double *rec, ObsFields f, const KState *ks)
{
    __shared__ double2 red[TB / 64][3];
    double2 v[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) v[i] = make_double2(0.0, 0.0);
    for (int b = threadIdx.x; b < nb; b += TB) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const double2 q = partial[pidx(b, i)];
            v[i].x += q.x;
            v[i].y += q.y;
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            v[i].x += __shfl_xor(v[i].x, d, 64);
            v[i].y += __shfl_xor(v[i].y, d, 64);
        }
    }
    if ((threadIdx.x & 63) == 0)
        for (int i = 0; i < 3; ++i) red[threadIdx.x >> 6][i] = v[i];
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int i = 0; i < 3; ++i)
        for (int w = 1; w < TB / 64; ++w) {
            red[0][i].x += red[w][i].x;
            red[0][i].y += red[w][i].y;
        }
    rec[PPQ_OBS_NORM2] = red[0][0].x;
    rec[PPQ_OBS_ACF_RE] = red[0][1].x;
    rec[PPQ_OBS_ACF_IM] = red[0][1].y;
    rec[PPQ_OBS_NABOVE] = red[0][2].x;
    rec[PPQ_OBS_T] = f.t;
    rec[PPQ_OBS_NACTIVE] = f.nact;
    rec[PPQ_OBS_KRYLOV] = ks ? (double)ks->meff : f.krylov;
    rec[PPQ_OBS_SUBSTEPS] = f.nsub;
}

// ---- position expectations ---------------------------------------------------------
// Per block: sum |c|^2 and, per dimension, sum |c|^2 q_k(i_k); the DVR position
// is diagonal in the grid index with the grid point as eigenvalue (Sec. II.A).
// q holds the grid points [D][nmax].
__global__ __launch_bounds__(TB) void k_expq_partial(const uint32_t *keys, const double2 *psi, int64_t n, GridDesc g,
                                                     const double *q, int nmax, double2 *partial)
{
    double2 acc[1 + MAXD];
#pragma unroll
    for (int i = 0; i <= MAXD; ++i) acc[i] = make_double2(0.0, 0.0);
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) {
        double2 c = psi[p];
        double w = fma(c.x, c.x, c.y * c.y);
        acc[0].x += w;
        uint32_t key = keys[p];
#pragma unroll
        for (int k = 0; k < MAXD; ++k)
            if (k < g.D) {
                int d = (int)((key / g.stride[k]) % (uint32_t)g.n[k]);
                acc[1 + k].x = fma(w, q[k * nmax + d], acc[1 + k].x);
            }
    }
    block_reduce_store<1 + MAXD>(acc, partial);
}

// Fixed-order sum of the partials; out[k] = sum_k / sum_0, NaN where bit k of
// `nan_mask` is set (dimensions without a diagonal position) or the sum is 0.
__global__ __launch_bounds__(TB) void k_expq_final(const double2 *partial, int nb, int D, unsigned nan_mask,
                                                   double *out)
{
    __shared__ double red[TB];
    __shared__ double norm2;
    for (int i = 0; i <= D; ++i) {
        double s = 0.0;
        for (int b = threadIdx.x; b < nb; b += TB) s += partial[pidx(b, i)].x;
        red[threadIdx.x] = s;
        __syncthreads();
        for (int st = TB / 2; st >= 1; st >>= 1) {
            if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            if (i == 0) norm2 = red[0];
            else
                out[i - 1] = ((nan_mask >> (i - 1)) & 1u) || !(norm2 > 0.0) ? __builtin_nan("") : red[0] / norm2;
        }
        __syncthreads();
    }
}

// ---- device-side state transfer ---------------------------------------------------
// Checks caller keys (strictly ascending, below the grid size) and coefficients
// (finite) while converting them: bad[0] counts key violations, bad[1]
// non-finite coefficients (per-block counts summed by one fixed-order kernel).
__global__ void k_take_state(const uint64_t *keys, const double2 *coeff, int64_t n, uint64_t total, uint32_t *k32,
                             double2 *psi, unsigned *block_bad_keys, unsigned *block_bad_vals)
{
    int64_t p = gid();
    bool bad_key = false, bad_val = false;
    if (p < n) {
        const uint64_t k = keys[p];
        bad_key = k >= total || (p > 0 && keys[p - 1] >= k);
        const double2 c = coeff[p];
        bad_val = !isfinite(c.x) || !isfinite(c.y);
        k32[p] = (uint32_t)k;
        psi[p] = c;
    }
    count_block(bad_key, block_bad_keys);
    count_block(bad_val, block_bad_vals);
}

__global__ void k_give_keys(const uint32_t *k32, int64_t n, uint64_t *keys)
{
    int64_t p = gid();
    if (p < n) keys[p] = k32[p];
}

// host-known fields of one observable record
__global__ __launch_bounds__(TB) void k_energy_from_dot(const double2 *partial, int nb, double *rec)
{
    __shared__ double red[TB];
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += TB) s += partial[pidx(b, 0)].x;
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = TB / 2; st >= 1; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        double n2 = rec[PPQ_OBS_NORM2];
        rec[PPQ_OBS_ENERGY] = n2 > 0.0 ? red[0] / n2 : 0.0;
    }
}

// ---- adjoint ----------------------------------------------------------------------
// R^dagger of one adaption: mu (on the earlier set) from lambda (on the later
// set): mu_I = lambda_I for I in both sets, zero otherwise.
__global__ void k_gather_remap(const uint32_t *keys, int64_t n, const uint64_t *bm, const uint32_t *prefix,
                               const double2 *lam, double2 *mu)
{
    int64_t p = gid();
    if (p >= n) return;
    uint32_t key = keys[p];
    uint64_t word = bm[key >> 6];
    uint32_t b = key & 63;
    mu[p] = ((word >> b) & 1ull) ? lam[prefix[key >> 6] + (uint32_t)__popcll(word & ((1ull << b) - 1ull))]
                                 : make_double2(0.0, 0.0);
}

__global__ void k_count_diff(const double2 *a, const double2 *b, int64_t n, unsigned long long *cnt)
{
    int64_t p = gid();
    bool diff = false;
    if (p < n) {
        double2 x = a[p], y = b[p];
        diff = (__double_as_longlong(x.x) != __double_as_longlong(y.x)) ||
               (__double_as_longlong(x.y) != __double_as_longlong(y.y));
    }
    count_ballot(diff, cnt);
}

__global__ void k_mark_wave(const uint32_t *keys, int64_t n, uint64_t *bm)
{
    int64_t p = gid();
    uint32_t key = p < n ? keys[p] : 0u;
    set_bit_wave(bm, key, p < n);
}

// Time integral of the Krylov-projected Frechet derivative:
//   Q = m0 n0 [exp([[-i dt T_b, e1 e1^T], [0, -i dt T_f]])]_{12}
// (the block-triangular exponential gives int_0^1 e^{A(1-s)} X e^{Bs} ds),
// T_f, T_b the Lanczos matrices of psi_n (forward) and mu (adjoint), both of
// dimension m; 1024 lanes, one per entry of the 32 x 32 block matrix.  Bound by the
// products' LDS reads on one CU (57 us with 18 products and the squarings, 36 with 7).
constexpr int M2 = 2 * MAXM;
__global__ __launch_bounds__(1024) void k_adj_q(const KState *kf, const KState *kb, double dt, double2 *Q)
{
    __shared__ double2 A[M2][M2], E[M2][M2];
    __shared__ double rown[M2];
    __shared__ int s_sq;
    const int mf = kf->meff, mb = kb->meff;
    const int r = threadIdx.x / M2, c = threadIdx.x % M2;
    double h = 0.0;
    double2 x = make_double2(0.0, 0.0);
    // top-left: T_b (mb x mb) at [0, MAXM); bottom-right: T_f at [MAXM, 2 MAXM)
    auto tri = [](const KState *k, int mm, int i, int j) -> double {
        if (i >= mm || j >= mm) return 0.0;
        if (i == j) return k->alpha[i];
        if (i == j + 1) return k->beta[j];
        if (j == i + 1) return k->beta[i];
        return 0.0;
    };
    if (r < MAXM && c < MAXM) h = tri(kb, mb, r, c);
    else if (r >= MAXM && c >= MAXM) h = tri(kf, mf, r - MAXM, c - MAXM);
    A[r][c] = make_double2(0.0, -dt * h);
    if (r == 0 && c == MAXM) A[r][c] = make_double2(1.0, 0.0);
    (void)x;
    __syncthreads();
    if (threadIdx.x < M2) {
        double s = 0.0;
        for (int cc = 0; cc < M2; ++cc) s += sqrt(A[threadIdx.x][cc].x * A[threadIdx.x][cc].x + A[threadIdx.x][cc].y * A[threadIdx.x][cc].y);
        rown[threadIdx.x] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double nrm = 0.0;
        for (int i = 0; i < M2; ++i) nrm = rown[i] > nrm ? rown[i] : nrm;
        int sq = 0;
        while (nrm > 0.125 && sq < 1100) {  // (an infinite norm ends it too)
            nrm *= 0.5;
            ++sq;
        }
        s_sq = sq;
    }
    __syncthreads();
    const int sq = s_sq;
    const double scale = ldexp(1.0, -sq);
    A[r][c] = make_double2(A[r][c].x * scale, A[r][c].y * scale);
    // the Taylor sum of degree 19 by powers of A^4: seven products (18 term by term);
    // a lane keeps its entries of A, A^2 and A^3
    auto product = [&](const double2(*L)[M2], const double2(*R)[M2]) {
        double2 acc = make_double2(0.0, 0.0);
#pragma unroll 8
        for (int l = 0; l < M2; ++l) {
            const double2 a = L[r][l], b = R[l][c];
            acc.x += a.x * b.x - a.y * b.y;
            acc.y += a.x * b.y + a.y * b.x;
        }
        return acc;
    };
    __syncthreads();
    const double2 a1 = A[r][c], a2 = product(A, A);
    E[r][c] = a2;
    __syncthreads();
    const double2 a3 = product(E, A), a4 = product(E, E);
    __syncthreads();
    A[r][c] = a4;
    double f[20];  // 1 / k!
    f[0] = 1.0;
#pragma unroll
    for (int k = 1; k < 20; ++k) f[k] = f[k - 1] / k;
    double2 e = make_double2(0.0, 0.0);
#pragma unroll
    for (int b4 = 16; b4 >= 0; b4 -= 4) {
        if (b4 < 16) {
            E[r][c] = e;
            __syncthreads();
            e = product(E, A);
            __syncthreads();
        }
        e.x += (f[b4 + 3] * a3.x + f[b4 + 2] * a2.x) + (f[b4 + 1] * a1.x + (r == c ? f[b4] : 0.0));
        e.y += (f[b4 + 3] * a3.y + f[b4 + 2] * a2.y) + f[b4 + 1] * a1.y;
    }
    E[r][c] = e;
    __syncthreads();
    for (int q = 0; q < sq; ++q) {
        e = product(E, E);
        __syncthreads();
        E[r][c] = e;
        __syncthreads();
    }
    if (r < MAXM && c >= MAXM) {
        const double s2 = kf->n0 * kb->n0;
        Q[r * MAXM + (c - MAXM)] = (r < mb && c - MAXM < mf) ? make_double2(s2 * e.x, s2 * e.y) : make_double2(0.0, 0.0);
    }
}

// Per point S = sum_ab Q_ab conj(W_a) V_b, then for every parameter p the
// partial sums of S * G_p(I), G_p = dV/dtheta_p as a sum of products of 1D
// tables (staged in LDS).  A block per 256 points: the blocks beyond a small set
// would only reduce zeros (4D Morse training 72 us in 1024 blocks, 59 now; sums for
// the parameters there are instead of ADJ_MAXP and adjoint vectors loaded four at a
// time: 56, not kept).  V_0 / W_0 come from the FP64 master vectors
// (psi_n / n0 and mu / m0), like the propagated vectors.
template <class C>
__global__ __launch_bounds__(TB) void k_adj_reduce(const C *Vb, const C *Wb, int64_t ld, const double2 *psi,
                                                   const double2 *mu, const KState *kf, const KState *kb,
                                                   const double2 *Q, const uint32_t *keys, int64_t n, GridDesc g,
                                                   DerivDesc dd, double2 *partial)
{
    __shared__ double2 sQ[MAXM * MAXM];
    __shared__ double s_coef[POT_MAX_TERMS];
    __shared__ int s_par[POT_MAX_TERMS];
    __shared__ int s_nf[POT_MAX_TERMS];
    __shared__ int s_fac[POT_MAX_TERMS][POT_MAX_FAC];
    __shared__ double s_tab[POT_MAX_TAB];
    for (int i = threadIdx.x; i < MAXM * MAXM; i += TB) sQ[i] = Q[i];
    for (int t = threadIdx.x; t < dd.nterm; t += TB) {
        s_coef[t] = dd.coef[t];
        s_par[t] = dd.param[t];
        int nf = 0;
        for (int k = 0; k < g.D; ++k) {
            int ti = dd.tab[t * g.D + k];
            if (ti >= 0 && nf < POT_MAX_FAC) s_fac[t][nf++] = ((ti * dd.nmax) << 6) | (8 * k);
        }
        s_nf[t] = nf;
    }
    for (int i = threadIdx.x; i < dd.ntab * dd.nmax; i += TB) s_tab[i] = dd.tabs[i];
    __syncthreads();
    const int mf = kf->meff, mb = kb->meff;
    const double inv_n0 = 1.0 / kf->n0, inv_m0 = 1.0 / kb->n0;
    double2 acc[ADJ_MAXP];
#pragma unroll
    for (int i = 0; i < ADJ_MAXP; ++i) acc[i] = make_double2(0.0, 0.0);
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) {
        double2 v[MAXM];
        double2 a0 = psi[p];
        v[0] = make_double2(a0.x * inv_n0, a0.y * inv_n0);
#pragma unroll
        for (int b = 1; b < MAXM; ++b) v[b] = (b < mf) ? ld2(Vb, (int64_t)b * ld + p) : make_double2(0.0, 0.0);
        double2 S = make_double2(0.0, 0.0);
        for (int a = 0; a < mb; ++a) {
            double2 t = make_double2(0.0, 0.0);
#pragma unroll
            for (int b = 0; b < MAXM; ++b) {
                double2 q = sQ[a * MAXM + b];
                t.x += q.x * v[b].x - q.y * v[b].y;
                t.y += q.x * v[b].y + q.y * v[b].x;
            }
            double2 wa;
            if (a == 0) {
                double2 m0v = mu[p];
                wa = make_double2(m0v.x * inv_m0, m0v.y * inv_m0);
            } else {
                wa = ld2(Wb, (int64_t)a * ld + p);
            }
            cdot_acc(S, wa, t);
        }
        const uint64_t digits = packed_digits(keys[p], g);
        for (int t = 0; t < dd.nterm; ++t) {
            double f = s_coef[t];
            const int nf = __builtin_amdgcn_readfirstlane(s_nf[t]);
#pragma unroll
            for (int j = 0; j < POT_MAX_FAC; ++j) {
                if (j < nf) {
                    const int e = __builtin_amdgcn_readfirstlane(s_fac[t][j]);
                    f *= s_tab[(e >> 6) + ((uint32_t)(digits >> (e & 63)) & 255u)];
                }
            }
            const int pp = __builtin_amdgcn_readfirstlane(s_par[t]);
#pragma unroll
            for (int i = 0; i < ADJ_MAXP; ++i) {
                if (i == pp) {
                    acc[i].x += f * S.x;
                    acc[i].y += f * S.y;
                }
            }
        }
    }
    block_reduce_store<ADJ_MAXP>(acc, partial);
}

// dC[i] += coef * sum over blocks (fixed order), coef = -i dt; a block per parameter
__global__ __launch_bounds__(TB) void k_adj_accumulate(const double2 *partial, int nb, double2 coef, double2 *dC)
{
    __shared__ double2 red[TB];
    const int i = blockIdx.x;
    double2 s = make_double2(0.0, 0.0);
    for (int b = threadIdx.x; b < nb; b += TB) {
        s.x += partial[pidx(b, i)].x;
        s.y += partial[pidx(b, i)].y;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int st = TB / 2; st >= 1; st >>= 1) {
        if ((int)threadIdx.x < st) {
            red[threadIdx.x].x += red[threadIdx.x + st].x;
            red[threadIdx.x].y += red[threadIdx.x + st].y;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double2 r = red[0];
        dC[i].x += coef.x * r.x - coef.y * r.y;
        dC[i].y += coef.x * r.y + coef.y * r.x;
    }
}

// Packet-parameter terms.  For each dimension k and each of the two packet
// parameters (centre, momentum) the derivative of psi0_I is the product of
// the 1D tables with factor k replaced by its derivative table.
//   bra = 1: accumulates conj(dpsi0_I) vec_I      (<d psi0 | psi_N>)
//   bra = 0: accumulates conj(vec_I) dpsi0_I      (<lambda_0 | d psi0>)
constexpr int ADJ_MAXQ = 2 * MAXD;
__global__ __launch_bounds__(TB) void k_adj_packet(const uint32_t *keys, int64_t n, GridDesc g, const double2 *tabs,
                                                   const double2 *dtabs, int nmax, const double2 *vec, int bra,
                                                   double2 *partial)
{
    double2 acc[ADJ_MAXQ];
#pragma unroll
    for (int i = 0; i < ADJ_MAXQ; ++i) acc[i] = make_double2(0.0, 0.0);
    for (int64_t p = gid(); p < n; p += (int64_t)gridDim.x * TB) {
        uint32_t key = keys[p];
        double2 v = vec[p];
        for (int kd = 0; kd < g.D; ++kd) {
            for (int which = 0; which < 2; ++which) {
                double2 prod = make_double2(1.0, 0.0);
                for (int k = 0; k < g.D; ++k) {
                    int d = (int)((key / g.stride[k]) % (uint32_t)g.n[k]);
                    double2 f = (k == kd) ? dtabs[(2 * k + which) * nmax + d] : tabs[k * nmax + d];
                    prod = cmul(prod, f);
                }
                double2 r = make_double2(0.0, 0.0);
                if (bra) cdot_acc(r, prod, v);
                else cdot_acc(r, v, prod);
                int slot = 2 * kd + which;
#pragma unroll
                for (int i = 0; i < ADJ_MAXQ; ++i)
                    if (i == slot) {
                        acc[i].x += r.x;
                        acc[i].y += r.y;
                    }
            }
        }
    }
    block_reduce_store<ADJ_MAXQ>(acc, partial);
}

}  // namespace

// ---- launchers -------------------------------------------------------------------
void fill_u64(uint64_t *p, int64_t n, uint64_t v, hipStream_t s)
{
    if (n <= 0) return;
    unsigned b = nblocks(n);
    if (b > 8192) b = 8192;
    hipLaunchKernelGGL(k_fill<uint64_t>, dim3(b), dim3(TB), 0, s, p, n, v);
}
void fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s)
{
    if (n <= 0) return;
    unsigned b = nblocks(n);
    if (b > 8192) b = 8192;
    hipLaunchKernelGGL(k_fill<uint32_t>, dim3(b), dim3(TB), 0, s, p, n, v);
}
void fill_zero_bytes(void *p, int64_t nbytes, hipStream_t s)
{
    // callers pass 8-byte multiples
    fill_u64((uint64_t *)p, nbytes / 8, 0ull, s);
}

// (for every size up to n)
int64_t scan_tmp_words(int64_t n) { return std::max(scan_tiles(n), scan_tiles(std::min(n, SCAN_ONE))) + 16; }

void scan_popcount(const uint64_t *words, int64_t nwords, uint32_t *prefix, uint32_t *total, uint32_t *tmp,
                   hipStream_t s)
{
    scan_impl(PopLoad{words}, nwords, prefix, total, tmp, s);
}
void scan_u32(const uint32_t *in, int64_t n, uint32_t *out, uint32_t *total, uint32_t *tmp, hipStream_t s)
{
    scan_impl(U32Load{in}, n, out, total, tmp, s);
}

void init_flag(const GridDesc &g, const double2 *tabs, int nmax, double eps2, uint64_t *bm, hipStream_t s)
{
    unsigned b = nblocks(g.total);
    if (b > 65536) b = 65536;
    hipLaunchKernelGGL(k_init_flag, dim3(b), dim3(TB), 0, s, g, tabs, nmax, eps2, bm);
}
void product_values(const uint32_t *keys, int64_t n, const GridDesc &g, const double2 *tabs, int nmax,
                    double2 *out, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_product_values, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, g, tabs, nmax, out);
}
void dilate(const uint32_t *keys, const double2 *psi, int64_t n, const GridDesc &g, double eps2, uint64_t *bm,
            unsigned long long *nabove, unsigned *block_counts, hipStream_t s)
{
    if (n <= 0) return;
    const unsigned nb = nblocks(n);
    hipLaunchKernelGGL(k_dilate, dim3(nb), dim3(TB), 0, s, keys, psi, n, g, eps2, bm, block_counts);
    hipLaunchKernelGGL(k_sum_counts, dim3(1), dim3(1024), 0, s, block_counts, (int64_t)nb, nabove);
}
void dilate_words(const uint32_t *keys, const double2 *psi, int64_t n, const GridDesc &g, double eps2, uint64_t *K,
                  uint64_t *bm, int64_t nwords, unsigned long long *nabove, unsigned *block_counts, uint32_t *tile_sums,
                  hipStream_t s)
{
    const unsigned nb = n > 0 ? nblocks(n) : 0u;
    if (n > 0) hipLaunchKernelGGL(k_mark_kept, dim3(nb), dim3(TB), 0, s, keys, psi, n, eps2, K, block_counts);
    const int64_t tiles = scan_tiles(nwords);
#define L(I)                                                                                                            \
    hipLaunchKernelGGL(k_dilate_words<I>, dim3((unsigned)tiles), dim3(TB), 0, s, K, nwords, g, bm, tile_sums, block_counts, \
                       (int64_t)nb, nabove)
    if (scan_items(nwords) == 1) L(1);
    else L(SI);
#undef L
}
void scan_reduce_popcount(const uint64_t *words, int64_t nwords, uint32_t *tile_sums, hipStream_t s)
{
    const int64_t tiles = scan_tiles(nwords);
    if (scan_items(nwords) == 1)
        hipLaunchKernelGGL((k_scan_reduce<PopLoad, 1>), dim3((unsigned)tiles), dim3(SB), 0, s, PopLoad{words}, nwords, tile_sums);
    else
        hipLaunchKernelGGL((k_scan_reduce<PopLoad, SI>), dim3((unsigned)tiles), dim3(SB), 0, s, PopLoad{words}, nwords, tile_sums);
}
void scan_top(uint32_t *tile_sums, int64_t nwords, uint32_t *total, uint32_t *host_total,
              const unsigned long long *count, unsigned long long *host_count, hipStream_t s)
{
    const int64_t tiles = scan_tiles(nwords);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, tile_sums, tiles, total, host_total, count, host_count);
}
void apply_compact(const uint64_t *bm, int64_t nwords, const uint32_t *tile_off, uint32_t *prefix, uint32_t *keys_out,
                   uint64_t *K, hipStream_t s)
{
    const int64_t tiles = scan_tiles(nwords);
    if (scan_items(nwords) == 1)
        hipLaunchKernelGGL(k_apply_compact<1>, dim3((unsigned)tiles), dim3(SB), 0, s, bm, nwords, tile_off, prefix, keys_out, K);
    else
        hipLaunchKernelGGL(k_apply_compact<SI>, dim3((unsigned)tiles), dim3(SB), 0, s, bm, nwords, tile_off, prefix, keys_out, K);
}
template <class T>
void carry_over(const uint32_t *okeys, const double2 *opsi, const T *oV, int64_t n_old, const uint64_t *bm,
                const uint32_t *prefix, double2 *npsi, T *nV, int64_t n_new, hipStream_t s)
{
    if (n_new > 0)
        hipLaunchKernelGGL(k_fill_new<T>, dim3(std::min<unsigned>(nblocks(n_new), 8192u)), dim3(TB), 0, s, npsi, nV, n_new,
                           std::numeric_limits<T>::quiet_NaN());
    if (n_old > 0)
        hipLaunchKernelGGL(k_remap_all<T>, dim3(nblocks(n_old)), dim3(TB), 0, s, okeys, opsi, oV, n_old, bm, prefix, npsi,
                           nV);
}
template void carry_over<double>(const uint32_t *, const double2 *, const double *, int64_t, const uint64_t *,
                                 const uint32_t *, double2 *, double *, int64_t, hipStream_t);
template void carry_over<float>(const uint32_t *, const double2 *, const float *, int64_t, const uint64_t *,
                                const uint32_t *, double2 *, float *, int64_t, hipStream_t);
void keep_all_if_few_dropped(const uint32_t *keys, int64_t n, uint64_t *bm, double rel, unsigned *block_counts,
                             unsigned long long *dropped, hipStream_t s)
{
    if (n <= 0) return;
    const unsigned nb = nblocks(n);
    hipLaunchKernelGGL(k_count_dropped, dim3(nb), dim3(TB), 0, s, keys, n, bm, block_counts);
    hipLaunchKernelGGL(k_sum_counts, dim3(1), dim3(1024), 0, s, block_counts, (int64_t)nb, dropped);
    hipLaunchKernelGGL(k_keep_all_if, dim3(nb), dim3(TB), 0, s, keys, n, bm, dropped, rel);
}
void mark_keys(const uint32_t *keys, int64_t n, uint64_t *bm, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_mark, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, bm);
}
void remap(const uint32_t *okeys, const double2 *opsi, int64_t n_old, const uint64_t *bm, const uint32_t *prefix,
           double2 *npsi, hipStream_t s)
{
    if (n_old <= 0) return;
    hipLaunchKernelGGL(k_remap, dim3(nblocks(n_old)), dim3(TB), 0, s, okeys, opsi, n_old, bm, prefix, npsi);
}

void last_flags(const uint32_t *keys, int64_t n, int nlast, uint32_t *flags, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_last_flags, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, nlast, flags);
}
void last_fill(const uint32_t *keys, int64_t n, int nlast, const uint32_t *flags, const uint32_t *fidx,
               const uint32_t *nf, uint32_t *off, uint64_t *mask, hipStream_t s)
{
    if (nlast <= NMAX_MASK)
        hipLaunchKernelGGL(k_zero_masks, dim3(std::min<unsigned>(nblocks(n), 2048u)), dim3(TB), 0, s, mask, nf);
    hipLaunchKernelGGL(k_last_fill, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, nlast, flags, fidx, nf, off, mask);
}
void rot_set(const uint32_t *keys, int64_t n, const RotFrame &f, uint64_t *bm, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_rot_set, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, f.sk, f.nk, f.rin, f.rout, bm);
}
void rot_rank(const uint32_t *keys, int64_t n, const RotFrame &f, const uint64_t *bm, const uint32_t *prefix,
              const uint32_t *map, uint32_t *pi, uint32_t *inv, uint32_t *flags, uint64_t *tmpmask, uint8_t *info,
              hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_rot_rank, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, f.sk, f.nk, f.rin, f.rout, bm, prefix,
                       map, pi, inv, flags, tmpmask, info);
}
__global__ void k_chunk_fibers(const uint32_t *chunk, uint32_t nch, const uint32_t *fidx, const uint32_t *nf,
                               uint32_t n, uint32_t *out)
{
    int64_t t = gid();
    if (t > nch) return;
    const uint32_t c = chunk[t];
    out[t] = c < n ? fidx[c] : *nf;
}

void chunk_fibers(const uint32_t *chunk, int64_t n, uint32_t S, const uint32_t *fidx, const uint32_t *nf,
                  uint32_t *out, hipStream_t s)
{
    uint32_t nch = (uint32_t)((n + S - 1) / S);
    hipLaunchKernelGGL(k_chunk_fibers, dim3(nblocks((int64_t)nch + 1)), dim3(TB), 0, s, chunk, nch, fidx, nf,
                       (uint32_t)n, out);
}

void make_chunks(const uint32_t *keys, const uint32_t *P, int64_t n, uint32_t sin, bool inner, uint32_t S,
                 uint32_t cap, uint32_t *chunk, uint32_t *big, uint32_t *counters, hipStream_t s)
{
    uint32_t nch = (uint32_t)((n + S - 1) / S);
    hipLaunchKernelGGL(k_chunks, dim3(nblocks((int64_t)nch + 1)), dim3(TB), 0, s, keys, P, (uint32_t)n, sin,
                       inner ? 1 : 0, S, nch, cap, chunk, big, counters);
}
void last_info(const uint32_t *keys, int64_t n, int nlast, uint8_t *info, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_last_info, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, nlast, info);
}
void fiber_tables_all(const uint32_t *keys, int64_t n, const TileAll &r, int64_t nwords, uint64_t *bm, uint32_t *prefix,
                      uint32_t *cnt, uint32_t *offs, const TabPtrs &t, uint32_t *scan_tmp, uint32_t *counters,
                      uint32_t *nf, hipStream_t s)
{
    if (n <= 0 || r.nd <= 0) return;
    const int64_t nt = r.first[r.nd];
    int nmax = 0;
    for (int k = 0; k < r.nd; ++k) nmax = std::max<int>(nmax, (int)r.nk[k]);
    fill_u64(bm, nwords + 2, 0ull, s);
    mark_keys_wave(keys, n, bm, s);
    scan_popcount(bm, nwords, prefix, &counters[0], scan_tmp, s);
    const int64_t head = r.first[r.nd - 1], tail = nt - head;
    const int lanes = nt <= 1 << 16 ? 8 : 1;
    const unsigned wide = nblocks(head * lanes), last = nblocks((tail + LAST_TILES - 1) / LAST_TILES * 64);
    if (lanes == 8) hipLaunchKernelGGL(k_tile_count<8>, dim3(wide + last), dim3(TB), 0, s, r, wide, bm, cnt);
    else hipLaunchKernelGGL(k_tile_count<1>, dim3(wide + last), dim3(TB), 0, s, r, wide, bm, cnt);
    scan_u32(cnt, 2 * nt, offs, &counters[1], scan_tmp, s);
    // tiles a wavefront goes through: most hold nothing on a large grid, and a wavefront
    // of its own for each costs more than finding the next (163 us with 1, 120 with 4,
    // 115 with 8, 126 with 16 over 830K tiles); few tiles are spread over the chip (11 us
    // with 1, 40 with 8 over 5K)
    const int group = (int)std::min<int64_t>(std::max<int64_t>(nt / 8192, 1), 8);
    const int64_t per = (int64_t)(TB / 64) * group;
    hipLaunchKernelGGL(k_tile_fill, dim3((unsigned)((nt + per - 1) / per)), dim3(TB),
                       (size_t)(TB / 64) * 64 * nmax * sizeof(uint32_t), s, r, (uint32_t)n, nmax, group, bm, prefix, cnt, offs,
                       &counters[1], t, nf);
}
void fiber_tables_rotated(const uint32_t *keys, int64_t n, const RotAll &r, uint64_t *bm, uint32_t *prefix,
                          uint64_t *occ, uint32_t *oprefix, const TabPtrs &t, uint32_t *scan_tmp, uint32_t *counters,
                          uint32_t *nf, hipStream_t s)
{
    if (n <= 0 || r.nd <= 0) return;
    const int64_t words = (int64_t)(r.nd + 1) * r.nwords;  // nd rotated segments + the row-major one
    const int64_t owords = r.owoff[r.nd];
    fill_u64(bm, words + 2, 0ull, s);
    fill_u64(occ, owords + 2, 0ull, s);
    hipLaunchKernelGGL(k_rot_set_all, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, r, bm, occ);
    scan_popcount(bm, words, prefix, &counters[0], scan_tmp, s);
    scan_popcount(occ, owords, oprefix, &counters[1], scan_tmp, s);
    hipLaunchKernelGGL(k_occ_counts, dim3(1), dim3(64), 0, s, oprefix, n, r, &counters[1], t, nf);
    hipLaunchKernelGGL(k_rank_gather, dim3(nblocks((int64_t)r.nd * r.nwords)), dim3(TB), 0, s, n, r, bm, prefix, occ,
                       oprefix, t);
}
void plane_tables(const uint32_t *keys, int64_t n, const GridDesc &g, int a, uint64_t *bm, uint32_t *prefix,
                  int64_t nwords, uint32_t *P, uint16_t *dig, uint32_t *tstart, uint32_t *poff, uint32_t *pkey,
                  uint32_t *flags, uint32_t *pidx, uint32_t *scan_tmp, uint32_t *counter, hipStream_t s)
{
    if (n <= 0) return;
    const uint32_t na = (uint32_t)g.n[a], nb = (uint32_t)g.n[a + 1];
    const bool ident = (a + 2 == g.D);
    const uint32_t sk = g.stride[a + 1];
    if (!ident) {
        fill_u64(bm, nwords + 2, 0ull, s);
        hipLaunchKernelGGL(k_rot_set, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, sk, na * nb, 0u, 0u, bm);
        scan_popcount(bm, nwords, prefix, counter, scan_tmp, s);
    }
    hipLaunchKernelGGL(k_plane_rank, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, ident ? 1u : sk, na, nb,
                       ident ? nullptr : bm, ident ? nullptr : prefix, ident ? nullptr : P, dig, pkey);
    hipLaunchKernelGGL(k_plane_flags, dim3(nblocks(n)), dim3(TB), 0, s, pkey, n, flags, dig);
    scan_u32(flags, n, pidx, counter, scan_tmp, s);
    hipLaunchKernelGGL(k_plane_fill, dim3(nblocks(n)), dim3(TB), 0, s, flags, pidx, n, counter, poff);
    const uint32_t ntask = (uint32_t)((n + PLANE_WINDOW - 1) / PLANE_WINDOW);
    hipLaunchKernelGGL(k_plane_tasks, dim3(nblocks(n + 1)), dim3(TB), 0, s, poff, counter, n, PLANE_WINDOW, ntask,
                       tstart);
}

void pair_tasks(const uint32_t *keys, int64_t n, uint32_t nab, uint32_t *tstart, hipStream_t s)
{
    if (n <= 0) return;
    const uint32_t ntask = (uint32_t)((n + PAIR_WINDOW - 1) / PAIR_WINDOW);
    const int64_t threads = ((int64_t)ntask + 1) * 64;
    hipLaunchKernelGGL(k_pair_tasks, dim3((unsigned)((threads + TB - 1) / TB)), dim3(TB), 0, s, keys, n, nab,
                       PAIR_WINDOW, ntask, tstart);
}

void fib_fill(const uint32_t *flags, const uint32_t *fidx, const uint64_t *tmpmask, int64_t n, const uint32_t *nf,
              uint32_t *off, uint64_t *mask, hipStream_t s)
{
    hipLaunchKernelGGL(k_fib_fill, dim3(nblocks(n)), dim3(TB), 0, s, flags, fidx, tmpmask, n, nf, off, mask);
}

constexpr int64_t POT_DIRECT = 1 << 18;
void potential(const uint32_t *keys, int64_t n, const GridDesc &g, const PotDesc &pd, double *V, float *Vf,
               uint32_t *list, unsigned *count, hipStream_t s)
{
    if (n <= 0) return;
    const unsigned nb = std::min<unsigned>(nblocks(n), 2048u);
    // a small set's missing values are evaluated where they lie: wavefronts with
    // one run all terms, which costs less than gathering a list first (three launches)
    if (list && n <= POT_DIRECT) {
        hipLaunchKernelGGL(k_potential<1>, dim3(nb), dim3(TB), 0, s, keys, n, g, pd, V, Vf, nullptr, nullptr, 1);
        return;
    }
    if (list) {
        fill_u32(count, 1, 0u, s);
        const unsigned mb = std::min<unsigned>(nblocks(n), 1024u);
        if (V) hipLaunchKernelGGL(k_missing<double>, dim3(mb), dim3(TB), 0, s, V, n, list, count);
        else hipLaunchKernelGGL(k_missing<float>, dim3(mb), dim3(TB), 0, s, Vf, n, list, count);
    }
    // several points per thread where that leaves every SIMD its wavefronts (a list is a
    // few per cent of the set)
    if (list || n <= POT_DIRECT)
        hipLaunchKernelGGL(k_potential<1>, dim3(nb), dim3(TB), 0, s, keys, n, g, pd, V, Vf, list, count, 0);
    else
        hipLaunchKernelGGL(k_potential<4>, dim3(std::min<unsigned>(nblocks((n + 3) / 4), 2048u)), dim3(TB), 0, s, keys, n,
                           g, pd, V, Vf, list, count, 0);
}

void dot_partial(const double2 *a, const double2 *b, int64_t n, double2 *partial, hipStream_t s)
{
    hipLaunchKernelGGL(k_dot_partial, dim3(RED_BLOCKS), dim3(TB), 0, s, a, b, n, partial);
}
// a block per 256 points up to RED_BLOCKS (few partials for a small set)
static int obs_blocks(int64_t n) { return (int)std::min<int64_t>(std::max<int64_t>((n + TB - 1) / TB, 1), RED_BLOCKS); }
void obs_partial(const uint32_t *keys, const double2 *psi, int64_t n, const GridDesc &g, const double2 *bra,
                 int nmax, double eps2, double2 *partial, hipStream_t s)
{
    hipLaunchKernelGGL(k_obs_partial, dim3(obs_blocks(n)), dim3(TB), 0, s, keys, psi, n, g, bra, nmax, eps2, partial);
}
void obs_final(const double2 *partial, int64_t n, double *rec, const ObsFields &f, const KState *ks, hipStream_t s)
{
    hipLaunchKernelGGL(k_obs_final, dim3(1), dim3(TB), 0, s, partial, obs_blocks(n), rec, f, ks);
}
void expect_q(const uint32_t *keys, const double2 *psi, int64_t n, const GridDesc &g, const double *q, int nmax,
              unsigned nan_mask, double2 *partial, double *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_expq_partial, dim3(RED_BLOCKS), dim3(TB), 0, s, keys, psi, n, g, q, nmax, partial);
    hipLaunchKernelGGL(k_expq_final, dim3(1), dim3(TB), 0, s, partial, RED_BLOCKS, g.D, nan_mask, out);
}
void take_state(const uint64_t *keys, const double2 *coeff, int64_t n, uint64_t total, uint32_t *k32, double2 *psi,
                unsigned *block_counts, unsigned long long *bad, hipStream_t s)
{
    if (n <= 0) return;
    const unsigned nb = nblocks(n);
    hipLaunchKernelGGL(k_take_state, dim3(nb), dim3(TB), 0, s, keys, coeff, n, total, k32, psi, block_counts,
                       block_counts + nb);
    hipLaunchKernelGGL(k_sum_counts, dim3(1), dim3(1024), 0, s, block_counts, (int64_t)nb, bad);
    hipLaunchKernelGGL(k_sum_counts, dim3(1), dim3(1024), 0, s, block_counts + nb, (int64_t)nb, bad + 1);
}
void give_keys(const uint32_t *k32, int64_t n, uint64_t *keys, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_give_keys, dim3(nblocks(n)), dim3(TB), 0, s, k32, n, keys);
}
void sum_of_squares(const double2 *psi, int64_t n, double2 *partial, double2 *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_sq_partial, dim3(RED_BLOCKS), dim3(TB), 0, s, psi, n, partial);
    hipLaunchKernelGGL(k_sum_partial1, dim3(1), dim3(TB), 0, s, partial, RED_BLOCKS, out);
}
void gather_remap(const uint32_t *keys, int64_t n, const uint64_t *bm, const uint32_t *prefix, const double2 *lam,
                  double2 *mu, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_gather_remap, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, bm, prefix, lam, mu);
}
unsigned long long count_diff(const double2 *a, const double2 *b, int64_t n, unsigned long long *dcount,
                              unsigned long long *hcount, hipStream_t s)
{
    fill_u64((uint64_t *)dcount, 1, 0ull, s);
    if (n > 0) hipLaunchKernelGGL(k_count_diff, dim3(nblocks(n)), dim3(TB), 0, s, a, b, n, dcount);
    (void)hipMemcpyAsync(hcount, dcount, sizeof(unsigned long long), hipMemcpyDeviceToHost, s);
    (void)hipStreamSynchronize(s);
    return *hcount;
}
void mark_keys_wave(const uint32_t *keys, int64_t n, uint64_t *bm, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_mark_wave, dim3(nblocks(n)), dim3(TB), 0, s, keys, n, bm);
}
void adj_q(const KState *kf, const KState *kb, double dt, double2 *Q, hipStream_t s)
{
    hipLaunchKernelGGL(k_adj_q, dim3(1), dim3(1024), 0, s, kf, kb, dt, Q);
}
template <class C>
void adj_reduce(const C *Vb, const C *Wb, int64_t ld, const double2 *psi, const double2 *mu, const KState *kf,
                const KState *kb, const double2 *Q, const uint32_t *keys, int64_t n, const GridDesc &g,
                const DerivDesc &dd, double2 *partial, hipStream_t s)
{
    hipLaunchKernelGGL(k_adj_reduce<C>, dim3(obs_blocks(n)), dim3(TB), 0, s, Vb, Wb, ld, psi, mu, kf, kb, Q, keys, n, g,
                       dd, partial);
}
template void adj_reduce<double2>(const double2 *, const double2 *, int64_t, const double2 *, const double2 *,
                                  const KState *, const KState *, const double2 *, const uint32_t *, int64_t,
                                  const GridDesc &, const DerivDesc &, double2 *, hipStream_t);
template void adj_reduce<float2>(const float2 *, const float2 *, int64_t, const double2 *, const double2 *,
                                 const KState *, const KState *, const double2 *, const uint32_t *, int64_t,
                                 const GridDesc &, const DerivDesc &, double2 *, hipStream_t);
void adj_accumulate(const double2 *partial, int64_t n, int nparam, double2 coef, double2 *dC, hipStream_t s)
{
    if (nparam <= 0) return;
    hipLaunchKernelGGL(k_adj_accumulate, dim3(nparam), dim3(TB), 0, s, partial, obs_blocks(n), coef, dC);
}
void adj_packet(const uint32_t *keys, int64_t n, const GridDesc &g, const double2 *tabs, const double2 *dtabs,
                int nmax, const double2 *vec, int bra, double2 *partial, hipStream_t s)
{
    hipLaunchKernelGGL(k_adj_packet, dim3(obs_blocks(n)), dim3(TB), 0, s, keys, n, g, tabs, dtabs, nmax, vec, bra,
                       partial);
}

// ---- full-grid transform (C(2t) on lattice bases) ---------------------------
// y[I] = sum_j B[l][j] x[I with digit k -> j], l = i_k: the dense transform of
// a full-grid tensor along dimension k (stride of digit k, nk its size).
__global__ void k_modek(const double2 *__restrict__ x, double2 *__restrict__ y, int64_t total, int64_t stride, int nk,
                        const double2 *__restrict__ B)
{
    for (int64_t I = gid(); I < total; I += (int64_t)gridDim.x * blockDim.x) {
        const int l = (int)((I / stride) % nk);
        const int64_t base = I - (int64_t)l * stride;
        double re = 0.0, im = 0.0;
        for (int j = 0; j < nk; ++j) {
            const double2 b = B[l * nk + j], v = x[base + (int64_t)j * stride];
            re += b.x * v.x - b.y * v.y;
            im += b.x * v.y + b.y * v.x;
        }
        y[I] = make_double2(re, im);
    }
}

__global__ void k_scatter_full(const uint32_t *keys, const double2 *psi, int64_t n, double2 *full)
{
    const int64_t p = gid();
    if (p < n) full[keys[p]] = psi[p];
}

void scatter_full(const uint32_t *keys, const double2 *psi, int64_t n, double2 *full, hipStream_t s)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_scatter_full, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, keys, psi, n, full);
}

void transform_full(const double2 *x, double2 *y, int64_t total, int64_t stride, int nk, const double2 *B,
                    hipStream_t s)
{
    const int64_t nb = std::min<int64_t>((total + 255) / 256, 65536);
    hipLaunchKernelGGL(k_modek, dim3((unsigned)nb), dim3(256), 0, s, x, y, total, stride, nk, B);
}

// ---- diagonal factors of a product term -------------------------------------
// y (= or +=) w D(I) x_I with D(I) = prod over the dimensions in `use` of
// tab[k][i_k]: the diagonal (DVR) factors of a sum-of-products term.  They
// commute with the truncation to the active set, so they act on the input of
// the term's chain of dense factors.  D is formed in FP64 in increasing k.
template <class C>
__global__ void k_diag_scale(const uint32_t *keys, const C *x, int64_t n, GridDesc g, const double *tab, int nmax,
                             unsigned use, double2 w, C *y, int acc, const int *skip_if, int skip_j)
{
    if (skip_if && skip_j >= *skip_if) return;
    const int64_t p = gid();
    if (p >= n) return;
    const uint32_t key = keys[p];
    double d = 1.0;
#pragma unroll
    for (int k = 0; k < MAXD; ++k)
        if (k < g.D && ((use >> k) & 1u)) d *= tab[k * nmax + (int)((key / g.stride[k]) % (uint32_t)g.n[k])];
    const double wr = w.x * d, wi = w.y * d;
    const C v = x[p];
    const double vr = v.x, vi = v.y;
    double r = wr * vr - wi * vi, i = wr * vi + wi * vr;
    if (acc) {
        r += y[p].x;
        i += y[p].y;
    }
    C o;
    o.x = r;
    o.y = i;
    y[p] = o;
}

template <class C>
void diag_scale(const uint32_t *keys, const C *x, int64_t n, const GridDesc &g, const double *tab, int nmax,
                unsigned use, double2 w, C *y, bool acc, const int *skip_if, int skip_j, hipStream_t s)
{
    if (n <= 0) return;
    const int nb = (int)((n + 255) / 256);
    hipLaunchKernelGGL(k_diag_scale<C>, dim3(nb), dim3(256), 0, s, keys, x, n, g, tab, nmax, use, w, y, acc ? 1 : 0,
                       skip_if, skip_j);
}
template void diag_scale<double2>(const uint32_t *, const double2 *, int64_t, const GridDesc &, const double *, int,
                                  unsigned, double2, double2 *, bool, const int *, int, hipStream_t);
template void diag_scale<float2>(const uint32_t *, const float2 *, int64_t, const GridDesc &, const double *, int,
                                 unsigned, double2, float2 *, bool, const int *, int, hipStream_t);

void energy_from_dot(const double2 *partial, int nb, double *rec, hipStream_t s)
{
    hipLaunchKernelGGL(k_energy_from_dot, dim3(1), dim3(TB), 0, s, partial, nb, rec);
}

}  // namespace ppq
