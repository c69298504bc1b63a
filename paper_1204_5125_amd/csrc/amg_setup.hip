// Setup of the smoothed-aggregation preconditioner R_k = AMG_k(H, D .) with
// H = K-hat + 2 D |psi|^2 (Sec. 4.1, eq. prec2; smoothed aggregation with
// 1 + 1 symmetric Gauss-Seidel steps).  The paper leaves the aggregation and
// smoothing parameters open; this library fixes them as follows:
//   strength     every structural off-diagonal entry (theta = 0), so the
//                integer part of the hierarchy depends only on the grid
//   priorities   the smaller index first (the greedy pass of standard
//                aggregation: regular, densely packed roots; hashed priorities
//                left a V-cycle that weakened as the grid was refined)
//   roots        distance-2 maximal independent set, computed in parallel
//                rounds: an undecided node becomes a root when it has the
//                smallest index among undecided nodes within distance 2 (this
//                equals the serial greedy choice in ascending index order)
//   assignment   neighbours of a root join it; the remaining nodes join the
//                aggregate of their assigned neighbour with the smallest root
//   numbering    aggregates in ascending root index
//   prolongator  P = T - omega D^-1 A T, T = 1/sqrt|a|, omega = (4/3) / rho~,
//                rho~ the estimate of rho(D^-1 A) after 20 power-iteration
//                steps from a counter-hash start; R = P^H; A_{l+1} = R A P
//                (upper triangle, mirrored; real diagonal)
//   colours      level 0: red-black parity of the grid; coarser: Jones-Plassmann
//                rounds with index priorities (equal to greedy colouring in
//                ascending index order: 4 colours on the regular coarse grids
//                where degree or hash orders needed 7-8), then two
//                iterated-greedy passes
//   coarsest     dense Cholesky
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>

#include "amg.h"
#include "stencil.h"

namespace glk {

// ------------------------------------------------------------ scan ----
constexpr int kScanItems = 4;
constexpr int kScanTile = kBlock * kScanItems;

__global__ __launch_bounds__(kBlock) void k_scan_tile(const int *__restrict__ in, int *__restrict__ out,
                                                      int *__restrict__ bsum, int n)
{
    __shared__ int sm[kBlock];
    const int base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
    int v[kScanItems], t = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? in[base + k] : 0;
        t += v[k];
    }
    sm[threadIdx.x] = t;
    __syncthreads();
    for (int o = 1; o < kBlock; o <<= 1) {
        const int add = threadIdx.x >= (unsigned)o ? sm[threadIdx.x - o] : 0;
        __syncthreads();
        sm[threadIdx.x] += add;
        __syncthreads();
    }
    int ex = sm[threadIdx.x] - t;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) out[base + k] = ex;
        ex += v[k];
    }
    if (threadIdx.x == kBlock - 1) bsum[blockIdx.x] = sm[kBlock - 1];
}

// out[i] += the offset of i's tile, and out[n] = the total
__global__ void k_scan_add(int *out, const int *boff, const int *bsum, int n, int nb)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) {
        if (nb > 1) out[i] += boff[i / kScanTile];
    } else if (i == n) {
        out[n] = (nb > 1 ? boff[nb - 1] : 0) + bsum[nb - 1];
    }
}

// Scratch of one symbolic phase, grown as needed and kept until it ends (an
// allocation per use cost more than most of the kernels it served).
struct SymTmp {
    Arena arena;                  // of the work arrays (they do not belong to the handle)
    DevBuf<int> scan;             // tile sums and offsets
    DevBuf<int> a, b, c, d, e, f; // per-row work arrays
    DevBuf<int> flags;            // "undecided nodes are left" of a batch of rounds
    DevBuf<int> err;
};

static int *need(SymTmp &T, DevBuf<int> &b, size_t n)
{
    if (b.count < n) {
        const ArenaScope own(&T.arena);
        b.alloc(n);
    }
    return b.get();
}

static void scan_tiles(const int *in, int *out, int n, int *tmp, hipStream_t s)
{
    const int nb = (n + kScanTile - 1) / kScanTile;
    int *bsum = tmp, *boff = tmp + nb + 1;
    k_scan_tile<<<nb, kBlock, 0, s>>>(in, out, bsum, n);
    GLK_CHECK_LAUNCH();
    if (nb > 1) scan_tiles(bsum, boff, nb, tmp + 2 * (nb + 1), s);
    k_scan_add<<<blocks_for((int64_t)n + 1), kBlock, 0, s>>>(out, boff, bsum, n, nb);
    GLK_CHECK_LAUNCH();
}

// exclusive scan of in[0..n) into out[0..n], out[n] the total, which is also
// returned (synchronises s); in and out must not overlap
static int64_t scan_excl(const int *in, int *out, int n, SymTmp &T, hipStream_t s)
{
    if (n <= 0) return 0;
    scan_tiles(in, out, n, need(T, T.scan, 4 * ((size_t)n / kScanTile + 4) + 64), s);
    int total = 0;
    GLK_HIP(hipMemcpyAsync(&total, out + n, sizeof(int), hipMemcpyDeviceToHost, s));
    GLK_HIP(hipStreamSynchronize(s));
    return (int64_t)total;
}

// ---------------------------------------------------------- keys ------
__device__ __forceinline__ uint32_t fmix32(uint32_t h)
{
    h ^= h >> 16;
    h *= 0x85ebca6bu;
    h ^= h >> 13;
    h *= 0xc2b2ae35u;
    h ^= h >> 16;
    return h;
}

// aggregation priority: larger for the smaller index (0 stays free for "none")
__device__ __forceinline__ unsigned long long keyof(int i)
{
    return (unsigned long long)(0xFFFFFFFFu - (uint32_t)i);
}

// insert v into the ascending unique list buf[0..u); false on overflow
__device__ __forceinline__ bool sorted_insert(int *buf, int &u, int v)
{
    int lo = 0, hi = u;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (buf[mid] < v) lo = mid + 1; else hi = mid;
    }
    if (lo < u && buf[lo] == v) return true;
    if (u == kMaxRow) return false;
    for (int t = u; t > lo; --t) buf[t] = buf[t - 1];
    buf[lo] = v;
    ++u;
    return true;
}

__device__ __forceinline__ int find_col(const int *ci, int b, int e, int col)
{
    while (b < e) {
        const int mid = (b + e) >> 1;
        if (ci[mid] < col) b = mid + 1; else e = mid;
    }
    return b;
}

// ------------------------------------------------- level-0 CSR -------
template <int DIM>
__global__ void k_l0_count(Geom g, int *cnt)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.n) return;
    int c[3];
    node_coords<DIM>(g.N, i, c);
    int k = 1;
    for (int a = 0; a < DIM; ++a) k += (c[a] > 0) + (c[a] < g.N[a] - 1);
    cnt[i] = k;
}

// columns ascending: lower neighbours (largest stride first), i, upper neighbours
template <int DIM>
__global__ void k_l0_cols(Geom g, const int *rp, int *ci)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.n) return;
    int c[3];
    node_coords<DIM>(g.N, i, c);
    int st[3] = {1, g.N[0], g.N[0] * g.N[1]};
    int p = rp[i];
    for (int a = DIM - 1; a >= 0; --a)
        if (c[a] > 0) ci[p++] = i - st[a];
    ci[p++] = i;
    for (int a = 0; a < DIM; ++a)
        if (c[a] < g.N[a] - 1) ci[p++] = i + st[a];
}

// H = K-hat + 2 D |psi|^2 in the same entry order
template <int DIM>
struct L0Values {
    GeomT<double> g;
    const int *rp;
    LinkTab<double> U;
    const double2 *__restrict__ psi;
    double2 *v;
    double *diag;
    __device__ void operator()(int, int) const
    {
        const int i = blockIdx.x * kBlock + threadIdx.x;
        if (i >= g.n) return;
        int c[3];
        node_coords<DIM>(g.N, i, c);
        double s[3];
        const double d = node_volume<DIM, double>(g, c, s);
        int p = rp[i];
        double asum = 0.0;
        for (int a = DIM - 1; a >= 0; --a)
            if (c[a] > 0) {
                const double al = d * s[a] * g.inv_h2[a];
                v[p++] = cscale(link_u<DIM, double>(U, a, c, c[a] - 1), -al);
            }
        const int pd = p++;
        for (int a = 0; a < DIM; ++a) {
            const double al = d * s[a] * g.inv_h2[a];
            if (c[a] < g.N[a] - 1) v[p++] = cscale(cconj(link_u<DIM, double>(U, a, c, c[a])), -al);
            asum += al * ((c[a] > 0) + (c[a] < g.N[a] - 1));
        }
        const double dg = asum + 2.0 * d * cabs2(psi[i]);
        v[pd] = make_double2(dg, 0.0);
        diag[i] = dg;
    }
};

// Level 0 of a simplicial mesh: its adjacency with the diagonal inserted
// (columns ascending), H_jj = K-hat_jj + 2 |V_j| |psi_j|^2, H_jk = -kw_jk
__global__ void k_l0s_count(int n, const int *arp, int *cnt)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) cnt[i] = arp[i + 1] - arp[i] + 1;
}

__global__ void k_l0s_cols(int n, const int *arp, const int *aci, const int *rp, int *ci)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    int p = rp[i];
    bool diag = false;
    for (int q = arp[i]; q < arp[i + 1]; ++q) {
        if (!diag && aci[q] > i) {
            ci[p++] = i;
            diag = true;
        }
        ci[p++] = aci[q];
    }
    if (!diag) ci[p] = i;
}

struct L0sValues {
    GeomT<double> g;
    const int *rp, *ci;
    const double2 *__restrict__ psi;
    double2 *v;
    double *diag;
    __device__ void operator()(int, int) const
    {
        const int i = blockIdx.x * kBlock + threadIdx.x;
        if (i >= g.n) return;
        int q = g.rp[i];
        const double dg = g.ks[i] + 2.0 * g.vol[i] * cabs2(psi[i]);
        for (int p = rp[i]; p < rp[i + 1]; ++p)
            v[p] = ci[p] == i ? make_double2(dg, 0.0) : cscale(g.kw[q++], -1.0);
        diag[i] = dg;
    }
};

// --------------------------------------------------------- MIS-2 -----
__global__ void k_fill_int(int *a, int n, int val)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) a[i] = val;
}

// A word that other threads of the same kernel may be writing: an old value
// only delays a decision.
__device__ __forceinline__ int load_relaxed(const int *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void store_relaxed(int *p, int v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One round of the distance-2 independent set (state 0 undecided, 1 root, 2
// not a root).  A node is not a root once a root lies within distance 2, and is
// one once every smaller index within distance 2 is decided and no root is
// there: the outcome is the serial greedy one whatever order the threads
// decide in, so states are read and written in place, one kernel a round
// (four, with the nodes left counted by one atomic each, cost 7.4 ms of a
// 257^2 setup).  A node whose smallest neighbour is undecided is far from the
// front and waits; the others are listed in LDS and get kMisLanes lanes each,
// which take the neighbours in turn with a batch of loads in flight (a thread
// walking the 25 words of its neighbourhood one by one took 23 us a round).
// flag (nullable): set when a node was undecided before it.
constexpr int kMisLanes = 8;

__global__ __launch_bounds__(kBlock) void k_mis_round(int n, const int *__restrict__ rp, const int *__restrict__ ci,
                                                      int *state, int *flag)
{
    __shared__ int list[kBlock];
    __shared__ int count;
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    {
        const int i = blockIdx.x * kBlock + threadIdx.x;
        const bool open = i < n && load_relaxed(state + i) == 0;
        if (open) {
            const int first = ci[rp[i]];
            if (first >= i || load_relaxed(state + first) != 0) list[atomicAdd(&count, 1)] = i;
        }
        if (flag && __syncthreads_or(open) && threadIdx.x == 0) *flag = 1;
    }
    __syncthreads();
    const int lane = threadIdx.x % kMisLanes, total = count;
    for (int c = threadIdx.x / kMisLanes; c < total; c += kBlock / kMisLanes) {
        const int i = list[c];
        int seen = 0;  // bit 0: a root nearby, bit 1: a smaller undecided node
        for (int p = rp[i] + lane; p < rp[i + 1]; p += kMisLanes) {
            const int j = ci[p], e = rp[j + 1];
            for (int q = rp[j]; q < e; q += 8) {  // j itself among its columns
                int k[8], sk[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) k[u] = q + u < e ? ci[q + u] : i;
#pragma unroll
                for (int u = 0; u < 8; ++u) sk[u] = load_relaxed(state + k[u]);
#pragma unroll
                for (int u = 0; u < 8; ++u) seen |= (sk[u] == 1 ? 1 : 0) | (sk[u] == 0 && k[u] < i ? 2 : 0);
            }
        }
#pragma unroll
        for (int o = kMisLanes / 2; o > 0; o >>= 1) seen |= __shfl_xor(seen, o, 64);
        if (lane == 0 && seen != 2) store_relaxed(state + i, seen & 1 ? 2 : 1);
    }
}

__global__ void k_agg_phase_a(int n, const int *rp, const int *ci, const int *state, int *rootA)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    if (state[i] == 1) { rootA[i] = i; return; }
    int best = -1;
    for (int p = rp[i]; p < rp[i + 1]; ++p) {
        const int j = ci[p];
        if (j != i && state[j] == 1 && (best < 0 || keyof(j) > keyof(best))) best = j;
    }
    rootA[i] = best;
}

__global__ void k_agg_phase_b(int n, const int *rp, const int *ci, const int *rootA, int *root, int *err)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    int best = rootA[i];
    if (best < 0) {
        for (int p = rp[i]; p < rp[i + 1]; ++p) {
            const int j = ci[p];
            if (j == i) continue;
            const int r = rootA[j];
            if (r >= 0 && (best < 0 || keyof(r) > keyof(best))) best = r;
        }
        if (best < 0) atomicOr(err, 1);
    }
    root[i] = best;
}

__global__ void k_root_flags(int n, const int *state, int *flag)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) flag[i] = (state[i] == 1);
}

__global__ void k_agg_number(int n, const int *root, const int *id, const int *state, int *agg,
                             int *rootlist, int *aggsize)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const int r = root[i];
    const int a = r >= 0 ? id[r] : 0;
    agg[i] = a;
    if (state[i] == 1) rootlist[id[i]] = i;
    atomicAdd(&aggsize[a], 1);
}

// ------------------------------------------------------ patterns -----
__global__ void k_p_pattern(int n, const int *rp, const int *ci, const int *agg, const int *prp,
                            int *cnt, int *pci, int *err)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    int buf[kMaxRow];
    int u = 0;
    for (int p = rp[i]; p < rp[i + 1]; ++p)
        if (!sorted_insert(buf, u, agg[ci[p]])) { atomicOr(err, 2); return; }
    if (pci) {
        const int o = prp[i];
        for (int t = 0; t < u; ++t) pci[o + t] = buf[t];
    } else {
        cnt[i] = u;
    }
}

__global__ void k_col_count(int nnz, const int *col, int *cnt)
{
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p < nnz) atomicAdd(&cnt[col[p]], 1);
}

__global__ void k_transpose_fill(int n, const int *prp, const int *pci, const int *rrp, int *fill,
                                 int *rci, int *rsrc)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    for (int p = prp[i]; p < prp[i + 1]; ++p) {
        const int a = pci[p];
        const int q = rrp[a] + atomicAdd(&fill[a], 1);
        rci[q] = i;
        rsrc[q] = p;
    }
}

constexpr int kRowWaves = kBlock / 64;  // rows per work-group of the wave-per-row kernels

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// rows of the transpose in ascending column order, a wave per row: an entry's
// place is the number of smaller columns (an insertion sort by one thread per
// row took 48 ms for the 129^3 grid)
__global__ __launch_bounds__(kBlock) void k_sort_rows(int nr, const int *__restrict__ rrp,
                                                      const int *__restrict__ ci_in, const int *__restrict__ src_in,
                                                      int *__restrict__ rci, int *__restrict__ rsrc)
{
    const int r = blockIdx.x * kRowWaves + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= nr) return;
    const int b = rrp[r], e = rrp[r + 1];
    for (int p0 = b; p0 < e; p0 += 64) {
        const int p = p0 + lane;
        const int c = p < e ? ci_in[p] : 0;
        int rank = 0;
        for (int q = b; q < e; ++q) rank += ci_in[q] < c;
        if (p < e) {
            rci[b + rank] = c;
            rsrc[b + rank] = src_in[p];
        }
    }
}

// pattern of A P, a thread per row
__global__ void k_ap_pattern(int n, const int *rp, const int *ci, const int *prp, const int *pci, const int *aprp,
                             int *cnt, int *apci, int *err)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    int buf[kMaxRow];
    int u = 0;
    for (int q = rp[i]; q < rp[i + 1]; ++q) {
        const int j = ci[q];
        for (int s = prp[j]; s < prp[j + 1]; ++s)
            if (!sorted_insert(buf, u, pci[s])) { atomicOr(err, 4); return; }
    }
    if (apci) {
        const int o = aprp[i];
        for (int t = 0; t < u; ++t) apci[o + t] = buf[t];
    } else {
        cnt[i] = u;
    }
}

// The pairs (R entry p, A P entry k of row rci[p]) of coarse row I, which make
// up row I of R (A P), dealt to the lanes of a wave 64 at a time in row order:
// f(valid, p, k).  pre: 64 words of LDS.
template <class F>
__device__ __forceinline__ void wave_pairs(int b, int e, const int *__restrict__ rci, const int *__restrict__ aprp,
                                           int *pre, int lane, F &&f)
{
    for (int base = b; base < e; base += 64) {
        const int p = base + lane, i = p < e ? rci[p] : 0;
        const int o = p < e ? aprp[i] : 0, len = p < e ? aprp[i + 1] - o : 0;
        int sum = len;
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(sum, d, 64);
            if (lane >= d) sum += v;
        }
        const int total = __shfl(sum, 63, 64);
        wave_sync();
        pre[lane] = sum - len;
        wave_sync();
        for (int f0 = 0; f0 < total; f0 += 64) {
            const int idx = f0 + lane;
            int l = 0;  // the last lane whose pairs start at or before idx
#pragma unroll
            for (int d = 32; d > 0; d >>= 1)
                if (pre[l + d] <= idx) l += d;
            const int k = __shfl(o, l, 64) + idx - pre[l];
            f(idx < total, base + l, k);
        }
    }
}

// Pattern of R (A P), a wave per coarse row: the row's columns gathered in an
// LDS hash set, compacted, and placed by the number of smaller ones.  A row of
// more than kMaxRow columns is refused (err 4).  (A thread per row inserting
// the columns of R A P one by one into a sorted list took 217 ms for the first
// level of the 129^3 grid, twice; see k_rap_pairs.)
constexpr int kHash = 2 * kMaxRow;

__global__ __launch_bounds__(kBlock) void k_rap_pattern(int nc, const int *__restrict__ rrp,
                                                        const int *__restrict__ rci, const int *__restrict__ aprp,
                                                        const int *__restrict__ apci, const int *__restrict__ crp,
                                                        int *cnt, int *cci, int *err)
{
    __shared__ int s_tab[kRowWaves][kHash], s_list[kRowWaves][kMaxRow], s_pre[kRowWaves][64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, I = blockIdx.x * kRowWaves + w;
    if (I >= nc) return;
    int *tab = s_tab[w], *list = s_list[w];
    for (int t = lane; t < kHash; t += 64) tab[t] = -1;
    wave_sync();
    int fresh = 0;
    bool full = false;
    wave_pairs(rrp[I], rrp[I + 1], rci, aprp, s_pre[w], lane, [&](bool valid, int, int k) {
        if (!valid) return;
        const int c = apci[k];
        unsigned h = ((unsigned)c * 2654435761u) % kHash;
        int tries = 0;
        for (; tries < kHash; ++tries, h = (h + 1) % kHash) {
            const int old = atomicCAS(&tab[h], -1, c);
            if (old == -1) ++fresh;
            if (old == -1 || old == c) break;
        }
        full |= tries == kHash;
    });
    for (int d = 32; d > 0; d >>= 1) fresh += __shfl_xor(fresh, d, 64);
    if (__any(full) || fresh > kMaxRow) {
        if (lane == 0) atomicOr(err, 4);
        return;
    }
    if (!cci) {
        if (lane == 0) cnt[I] = fresh;
        return;
    }
    wave_sync();
    int at = 0;
    for (int t0 = 0; t0 < kHash; t0 += 64) {
        const int c = tab[t0 + lane];
        const unsigned long long m = __ballot(c >= 0);
        if (c >= 0) list[at + __popcll(m & ((1ull << lane) - 1))] = c;
        at += __popcll(m);
    }
    wave_sync();
    const int o = crp[I];
    for (int t = lane; t < at; t += 64) {
        const int c = list[t];
        int rank = 0;
        for (int k = 0; k < at; ++k) rank += list[k] < c;
        cci[o + rank] = c;
    }
}

// The pairs of every entry of the upper triangle (J >= I) of R (A P), a wave
// per coarse row: counted (pair == NULL: cnt[t]), or listed in row order
// (pair[tp[t] ..]).  A chunk of 64 pairs is ordered among itself by comparing
// every lane's entry with the earlier lanes', so the lists are the same in
// every run.
__global__ __launch_bounds__(kBlock) void k_rap_pairs(int nc, const int *__restrict__ rrp,
                                                      const int *__restrict__ rci, const int *__restrict__ aprp,
                                                      const int *__restrict__ apci, const int *__restrict__ crp,
                                                      const int *__restrict__ cci, int *__restrict__ cnt,
                                                      const int *__restrict__ tp, int2 *__restrict__ pair)
{
    __shared__ int s_col[kRowWaves][kMaxRow], s_cur[kRowWaves][kMaxRow], s_pre[kRowWaves][64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, I = blockIdx.x * kRowWaves + w;
    if (I >= nc) return;
    int *col = s_col[w], *cur = s_cur[w];
    const int cb = crp[I], u = crp[I + 1] - cb;
    for (int t = lane; t < u; t += 64) {
        col[t] = cci[cb + t];
        cur[t] = pair ? tp[cb + t] : 0;
    }
    wave_sync();
    wave_pairs(rrp[I], rrp[I + 1], rci, aprp, s_pre[w], lane, [&](bool valid, int p, int k) {
        const int J = valid ? apci[k] : -1;
        int t = -1;
        if (J >= I) t = find_col(col, 0, u, J);
        if (!pair) {
            if (t >= 0) atomicAdd(&cur[t], 1);
            return;
        }
        int before = 0, all = 0;
        for (int l = 0; l < 64; ++l) {
            const bool same = __builtin_amdgcn_readlane(t, l) == t;
            before += same && l < lane;
            all += same;
        }
        if (t >= 0) {
            const int at = cur[t];
            pair[at + before] = make_int2(p, k);
            if (before == all - 1) cur[t] = at + all;
        }
        wave_sync();
    });
    if (pair) return;
    wave_sync();
    for (int t = lane; t < u; t += 64) cnt[cb + t] = cur[t];
}

// mir[t] for an upper entry t = (I, J), J > I: the entry (J, I) (the pattern of
// R A P is symmetric); the diagonal's own index
__global__ void k_rap_mirror(int nc, const int *__restrict__ crp, const int *__restrict__ cci, int *__restrict__ mir,
                             int *err)
{
    const int g = blockIdx.x * kBlock + threadIdx.x, I = g / 8, lane = g % 8;
    if (I >= nc) return;
    for (int t = crp[I] + lane; t < crp[I + 1]; t += 8) {
        const int J = cci[t];
        if (J < I) continue;
        const int u = find_col(cci, crp[J], crp[J + 1], I);
        if (u >= crp[J + 1] || cci[u] != I) atomicOr(err, 16);
        mir[t] = u;
    }
}

// --------------------------------------------------------- colours ----
template <int DIM>
__global__ void k_parity_colour(Geom g, int *col)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= g.n) return;
    int c[3];
    node_coords<DIM>(g.N, i, c);
    col[i] = (c[0] + c[1] + c[2]) & 1;
}

constexpr int kRecolourPasses = 2;  // iterated-greedy passes after the colouring rounds

// One round of the greedy colouring in index order: a node takes the smallest
// colour free among its smaller neighbours once all of them are coloured (the
// serial result whatever order the threads decide in; see k_mis_round).
__global__ __launch_bounds__(kBlock) void k_jp_round(int n, const int *__restrict__ rp, const int *__restrict__ ci,
                                                     int *col, int *flag, int *err)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const bool open = i < n && load_relaxed(col + i) < 0;
    if (flag && __syncthreads_or(open) && threadIdx.x == 0) *flag = 1;
    if (!open) return;
    const int b = rp[i], e = rp[i + 1];
    unsigned long long used[4] = {0, 0, 0, 0};
    for (int p = b; p < e; p += 4) {  // columns ascend
        int j[4], c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) j[u] = p + u < e ? ci[p + u] : i;
        if (j[0] >= i) break;
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = j[u] < i ? load_relaxed(col + j[u]) : 256;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (c[u] < 0) return;
            if (c[u] < 256) used[c[u] >> 6] |= 1ull << (c[u] & 63);
        }
    }
    int c = 0;
    while (c < 256 && (used[c >> 6] >> (c & 63) & 1ull)) ++c;
    if (c == 256) atomicOr(err, 8);
    store_relaxed(col + i, c);
}

// Iterated greedy (Culberson): the rows of one colour class (an independent
// set, so they do not see each other) take the smallest colour not yet given
// to a neighbour in this pass; classes are visited in reverse order.
__global__ void k_ig_class(int n, const int *rp, const int *ci, const int *old, int cls, int *nw, int *err)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n || old[i] != cls) return;
    unsigned long long used[4] = {0, 0, 0, 0};
    for (int p = rp[i]; p < rp[i + 1]; ++p) {
        const int j = ci[p];
        const int c = (j != i) ? nw[j] : -1;
        if (c >= 0 && c < 256) used[c >> 6] |= 1ull << (c & 63);
    }
    int c = 0;
    while (c < 256 && (used[c >> 6] >> (c & 63) & 1ull)) ++c;
    if (c == 256) atomicOr(err, 8);
    nw[i] = c;
}

// Rows grouped by colour, ascending inside a colour: rows of each colour per
// block (cnt[c nblk + block]; a colour the block lacks counts 0), and, after an
// exclusive scan of those counts, the places.
__global__ __launch_bounds__(kBlock) void k_colour_count(int n, const int *__restrict__ col, int nblk, int ncol,
                                                         int *__restrict__ cnt)
{
    __shared__ int h[257];
    for (int c = threadIdx.x; c < 257; c += kBlock) h[c] = 0;
    __syncthreads();
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n) atomicAdd(&h[col[i]], 1);
    __syncthreads();
    for (int c = threadIdx.x; c < ncol; c += kBlock) cnt[(size_t)c * nblk + blockIdx.x] = h[c];
}

__global__ __launch_bounds__(kBlock) void k_colour_place(int n, const int *__restrict__ col, int nblk,
                                                         const int *__restrict__ off, int *__restrict__ dst)
{
    __shared__ int sc[kBlock];
    const int i = blockIdx.x * kBlock + threadIdx.x;
    const int c = i < n ? col[i] : -1;
    sc[threadIdx.x] = c;
    __syncthreads();
    if (i >= n) return;
    int before = 0;
    for (int t = 0; t < (int)threadIdx.x; ++t) before += sc[t] == c;
    dst[off[(size_t)c * nblk + blockIdx.x] + before] = i;
}

// rows of each colour: 257 counters per block in LDS, added to the totals
__global__ __launch_bounds__(kBlock) void k_colour_hist(int n, const int *__restrict__ col, int *hist)
{
    __shared__ int h[257];
    for (int c = threadIdx.x; c < 257; c += kBlock) h[c] = 0;
    __syncthreads();
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) atomicAdd(&h[col[i]], 1);
    __syncthreads();
    for (int c = threadIdx.x; c < 257; c += kBlock)
        if (h[c]) atomicAdd(&hist[c], h[c]);
}

// of rows row0[c] .. row0[c + 1] - 1 (block c of C): the longest, and where the
// places of their diagonal entries are given, at C + c the most entries before it and
// at 2 C + c the least up to and with it
__global__ __launch_bounds__(kBlock) void k_row_widths(const int *__restrict__ rp, const int *__restrict__ dpos,
                                                       const int *__restrict__ row0, int *__restrict__ width)
{
    __shared__ int sm[3][kBlock / 64];
    int m[3] = {1, 0, 0};  // (the third is INT_MAX - what is wanted, a minimum)
    for (int r = row0[blockIdx.x] + threadIdx.x; r < row0[blockIdx.x + 1]; r += kBlock) {
        m[0] = max(m[0], rp[r + 1] - rp[r]);
        if (dpos) {
            m[1] = max(m[1], dpos[r] - rp[r]);
            m[2] = max(m[2], INT_MAX - (dpos[r] - rp[r] + 1));
        }
    }
    for (int d = 32; d > 0; d >>= 1)
        for (int q = 0; q < 3; ++q) m[q] = max(m[q], __shfl_xor(m[q], d, 64));
    if ((threadIdx.x & 63) == 0)
        for (int q = 0; q < 3; ++q) sm[q][threadIdx.x >> 6] = m[q];
    __syncthreads();
    if (threadIdx.x < (dpos ? 3 : 1)) {
        int w = sm[threadIdx.x][0];
        for (int k = 1; k < kBlock / 64; ++k) w = max(w, sm[threadIdx.x][k]);
        if (threadIdx.x == 2) w = INT_MAX - w;
        width[threadIdx.x * gridDim.x + blockIdx.x] = w;
    }
}

// --------------------------------------------------------- numeric ----
struct Diag {
    int n;
    const int *rp, *ci;
    const double2 *v;
    double *diag;
    __device__ void operator()(int, int) const
    {
        const int i = blockIdx.x * kBlock + threadIdx.x;
        if (i >= n) return;
        const int p = find_col(ci, rp[i], rp[i + 1], i);
        diag[i] = (p < rp[i + 1] && ci[p] == i) ? v[p].x : 0.0;
    }
};

// Spectral radius of D^-1 A by power iteration from the counter-hash start
// s_i = (h1_i - 1/2) + i (h2_i - 1/2), h = fmix32(i ^ salt) / 2^32; the
// normalisation of each iterate is folded into the next step.
constexpr int kRhoSteps = 20;

__device__ __forceinline__ double2 pw_start(int i)
{
    const double a = (double)fmix32((uint32_t)i ^ 0x2545F491u) / 4294967296.0 - 0.5;
    const double b = (double)fmix32((uint32_t)i ^ 0x6C8E9CF5u) / 4294967296.0 - 0.5;
    return make_double2(a, b);
}

struct PwStart {
    int n;
    double2 *x;
    __device__ void operator()(int, int) const
    {
        const int i = blockIdx.x * kBlock + threadIdx.x;
        if (i < n) x[i] = pw_start(i);
    }
};

// y = D^-1 A x, divided by ||x|| where xn2 gives ||x||^2, and partial sums of
// |y|^2 where the slot is set; kPwLanes lanes share a row (lane j takes entries j,
// j + kPwLanes, ... in order, then a fixed butterfly), so long coarse rows are not
// one serial chain of gathers.  The grid is at most the partial-sum slot's size: a
// block strides over the rows by the grid (the same iterations for all its threads)
// and stores one partial.
constexpr int kPwLanes = 8;

struct PwStep {
    int n;
    const int *rp, *ci;
    const double2 *v;
    const double *diag;
    const double2 *x;
    const double *xn2;
    double2 *y;
    RedSlot slot;
    __device__ void operator()(int, int) const
    {
        __shared__ double sm[kBlock / 64];
        const int64_t total = (int64_t)n * kPwLanes;
        const double scale = xn2 ? 1.0 / sqrt(*xn2) : 1.0;
        double part = 0.0;
        for (int64_t base = (int64_t)blockIdx.x * kBlock; base < total; base += (int64_t)gridDim.x * kBlock) {
            const int64_t g = base + threadIdx.x;
            const int i = (int)(g / kPwLanes), lane = (int)(g % kPwLanes);
            const bool act = g < total;
            double2 acc = make_double2(0.0, 0.0);
            if (act)
                for (int p = rp[i] + lane; p < rp[i + 1]; p += kPwLanes) acc = cadd(acc, cmul(v[p], x[ci[p]]));
    #pragma unroll
            for (int o = kPwLanes / 2; o > 0; o >>= 1) {
                acc.x += __shfl_xor(acc.x, o, 64);
                acc.y += __shfl_xor(acc.y, o, 64);
            }
            if (act && lane == 0) {
                const double2 yi = cscale(acc, scale / diag[i]);
                y[i] = yi;
                part += cabs2(yi);
            }
        }
        if (slot.partials) block_reduce_store(part, slot, sm, blockIdx.x);
    }
};

// Level 0: the same step with H applied as the stencil (link factor tables
// and the diagonal; its CSR copy holds the same entries), so a step streams x
// and the diagonal instead of the CSR arrays.
template <int DIM>
struct PwStepL0 {
    GeomT<double> g;
    LinkTab<double> U;
    const double *diag;
    const double2 *x;
    const double *xn2;
    double2 *y;
    RedSlot slot;
    __device__ void operator()(int, int) const
    {
        __shared__ double sm[kBlock / 64];
        const int i = blockIdx.x * kBlock + threadIdx.x;
        double part = 0.0;
        if (i < g.n) {
            int c[3];
            node_coords<DIM>(g.N, i, c);
            const double di = diag[i];
            const double2 acc = cadd(cscale(x[i], di), khat_offdiag<DIM, double>(g, i, c, x, U));
            const double2 yi = cscale(acc, 1.0 / (xn2 ? di * sqrt(*xn2) : di));
            y[i] = yi;
            part = cabs2(yi);
        }
        if (slot.partials) block_reduce_store(part, slot, sm, blockIdx.x);
    }
};

struct PwRho {
    const double *yn2;
    double *rho;
    __device__ void operator()(int, int) const
    {
        if (threadIdx.x == 0) *rho = sqrt(*yn2);
    }
};

// The estimate is the growth of the last step, so only the vector before it has
// to be normalised.  The one halfway is too, to keep the squares in range: rho is
// at least 1 (the mean eigenvalue of D^-1 A), and 10 steps stay below 1e154 up to
// rho = 2e15.  (A norm per step was a second dispatch per step: 513^2, four levels,
// 1.35 ms per numeric setup, now 1.04; 97x81x65 2.70, now 2.47.)
// |y|^2 of step k is wanted
__host__ __device__ constexpr bool rho_normed(int k) { return k == kRhoSteps / 2 || k >= kRhoSteps - 1; }

// The whole estimate of a small level by one work-group, from its CSR matrix: LPR
// lanes per row, the matrix in registers (S rows of kPwEntries entries per
// thread), the vector in LDS.  A step is a few LDS reads and two barriers where a
// dispatch takes 4-5 us with its gap.  us per step by <LPR, S>: <2, 1> and <4, 1> 0.8,
// <8, 1> 1.1, <2, 2> 1.3, <8, 2> 2.0, <2, 4> 2.2, <16, 2> 2.3, <4, 4> 2.8, <8, 4> 3.4,
// <16, 4> 4.1.  33^2, two levels, 0.38 ms per numeric setup with a dispatch per step,
// 0.29 with S = 4 for every level, now 0.22.
constexpr int kPwThreads = 1024, kPwEntries = 4;

template <int LPR, int S>
struct PwSmall {
    int n;
    const int *rp, *ci;
    const double2 *v;
    const double *diag;
    double *rho;
    __device__ void operator()(int, int) const
    {
        __shared__ double2 x[kPwThreads * S / LPR];
        __shared__ double sm[kPwThreads / 64], norm;
        double2 a[S][kPwEntries], y[S];
        int j[S][kPwEntries];
        double w[S];
        const int lane = threadIdx.x % LPR;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int i = (s * kPwThreads + threadIdx.x) / LPR;
            const int b = i < n ? rp[i] : 0, e = i < n ? rp[i + 1] : 0;
            w[s] = i < n ? 1.0 / diag[i] : 0.0;
#pragma unroll
            for (int k = 0; k < kPwEntries; ++k) {
                const int p = b + lane + k * LPR;
                j[s][k] = p < e ? ci[p] : 0;
                a[s][k] = p < e ? v[p] : make_double2(0.0, 0.0);
            }
        }
        for (int i = threadIdx.x; i < n; i += kPwThreads) x[i] = pw_start(i);
        __syncthreads();
        double scale = 1.0;
        for (int step = 1; step <= kRhoSteps; ++step) {
            double part = 0.0;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                double2 acc = make_double2(0.0, 0.0);
#pragma unroll
                for (int k = 0; k < kPwEntries; ++k) acc = cadd(acc, cmul(a[s][k], x[j[s][k]]));
#pragma unroll
                for (int o = LPR / 2; o > 0; o >>= 1) {
                    acc.x += __shfl_xor(acc.x, o, 64);
                    acc.y += __shfl_xor(acc.y, o, 64);
                }
                y[s] = cscale(acc, scale * w[s]);
                if (lane == 0) part += cabs2(y[s]);
            }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int i = (s * kPwThreads + threadIdx.x) / LPR;
                if (i < n && lane == 0) x[i] = y[s];
            }
            scale = 1.0;
            if (rho_normed(step)) {
                const double s2 = block_sum(part, sm);
                if (threadIdx.x == 0) norm = sqrt(s2);
                __syncthreads();
                scale = 1.0 / norm;
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) *rho = norm;
    }
};

static void rho_estimate(gl_precond *pre, Level &lev, const Launch &L)
{
    const gl_mesh *m = pre->mesh;
    const int n = lev.n, nb = blocks_for(n);
    const RedSlot slot = red_slot(m, 0);
    double2 *x = pre->vin.get(), *y = pre->cyc_r.get();
    double *nrm = pre->pwn.get();
    const int width = lev.ewidth.empty() ? 2 * m->g.dim + 1 : *std::max_element(lev.ewidth.begin(), lev.ewidth.end());
    const auto small = [&](auto lpr, auto slots) {
        constexpr int LPR = decltype(lpr)::value, S = decltype(slots)::value;
        if (width > LPR * kPwEntries || (int64_t)n * LPR > kPwThreads * S) return false;
        L.run<PwSmall<LPR, S>, kPwThreads>(
            1, PwSmall<LPR, S>{n, lev.A.rp.get(), lev.A.ci.get(), lev.A.v64.get(), lev.diag64.get(), lev.rho.get()});
        return true;
    };
    const auto small_rows = [&](auto lpr) {
        return small(lpr, std::integral_constant<int, 1>{}) || small(lpr, std::integral_constant<int, 2>{}) ||
               small(lpr, std::integral_constant<int, 4>{});
    };
    if (small_rows(std::integral_constant<int, 2>{}) || small_rows(std::integral_constant<int, 4>{}) ||
        small_rows(std::integral_constant<int, 8>{}) || small_rows(std::integral_constant<int, 16>{}) ||
        small_rows(std::integral_constant<int, 32>{}))
        return;
    L.run(nb, PwStart{n, x});
    // level 0 of a grid as the stencil, every other level (and level 0 of a
    // simplicial mesh) through its CSR matrix
    const bool l0 = &lev == &pre->L[0] && !m->g.simplicial;
    const GeomT<double> g = geom_t<double>(m->g);
    // CSR levels: kPwLanes threads per row, at most one partial per level-0 block
    const int nbl = std::min(blocks_for((int64_t)n * kPwLanes), blocks_for(m->g.n));
    for (int k = 1; k <= kRhoSteps; ++k) {
        const double *xn2 = k > 1 && rho_normed(k - 1) ? nrm + ((k - 1) & 1) : nullptr;
        const RedSlot sum = rho_normed(k) ? slot : RedSlot{nullptr};
        if (l0 && m->g.dim == 2)
            L.run(nb, PwStepL0<2>{g, link_tab<double>(m), lev.diag64.get(), x, xn2, y, sum});
        else if (l0)
            L.run(nb, PwStepL0<3>{g, link_tab<double>(m), lev.diag64.get(), x, xn2, y, sum});
        else
            L.run(nbl, PwStep{n, lev.A.rp.get(), lev.A.ci.get(), lev.A.v64.get(), lev.diag64.get(), x, xn2, y, sum});
        if (rho_normed(k))
            launch_finalize(slot.partials, l0 ? nb : nbl, FIN_STORE, nullptr, nrm + (k & 1), nullptr, L);
        std::swap(x, y);
    }
    L.run<PwRho, 64>(1, PwRho{nrm + (kRhoSteps & 1), lev.rho.get()});
}

// whether any lane of the wave is left (lanes of a wave that share shuffles stay together)
__device__ __forceinline__ bool wave_any(bool p) { return __any(p); }

// P = T - omega D^-1 A T.  LPR lanes share a row, a lane per entry of P's row: each
// loads one entry of A's row with the aggregate of its column, and every lane adds
// those of its own aggregate, in the order of the row, as they are passed round.
// (A thread per row that walked A's row once per entry of P's: 97x81x65, three
// levels, 550 us per numeric setup, now 84.)
constexpr int kPLanes = 8;

struct PValues {
    static constexpr int LPR = kPLanes;
    int n;
    const int *__restrict__ arp, *__restrict__ aci;
    const double2 *__restrict__ av;
    const double *diag;
    const int *__restrict__ agg, *aggsize;
    const double *rho;
    const int *__restrict__ prp, *__restrict__ pci;
    double2 *__restrict__ pv;
    __device__ void operator()(int, int) const
    {
        const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
        const int i = (int)(g / LPR), lane = (int)(g % LPR);
        const bool act = i < n;
        const int b = act ? arp[i] : 0, e = act ? arp[i + 1] : 0;
        const int pb = act ? prp[i] : 0, pe = act ? prp[i + 1] : 0;
        const double f = act ? (4.0 / 3.0) / *rho / diag[i] : 0.0;
        const int ai = act ? agg[i] : -1;
        for (int p0 = pb; wave_any(p0 < pe); p0 += LPR) {
            const int p = p0 + lane;
            const int a = p < pe ? pci[p] : -1;
            const double ta = a >= 0 ? 1.0 / sqrt((double)aggsize[a]) : 0.0;
            double2 at = make_double2(0.0, 0.0);
            for (int q0 = p0 < pe ? b : e; wave_any(q0 < e); q0 += LPR) {
                const int q = q0 + lane;
                const int mine = q < e ? agg[aci[q]] : -2;
                const double2 v = q < e ? av[q] : make_double2(0.0, 0.0);
#pragma unroll
                for (int t = 0; t < LPR; ++t) {
                    const int c = __shfl(mine, t, LPR);
                    const double2 u = make_double2(__shfl(v.x, t, LPR), __shfl(v.y, t, LPR));
                    if (c == a) at = cadd(at, cscale(u, ta));
                }
            }
            if (p < pe) pv[p] = make_double2((ai == a ? ta : 0.0) - f * at.x, -f * at.y);
        }
    }
};

struct RValues {
    int nnz;
    const int *rsrc;
    const double2 *pv;
    double2 *rv;
    __device__ void operator()(int, int) const
    {
        const int q = blockIdx.x * kBlock + threadIdx.x;
        if (q < nnz) rv[q] = cconj(pv[rsrc[q]]);
    }
};

// A_{l+1} = R (A P) in two products: A P is formed once (a fine row's entry is
// used by every coarse row of its R column), so the second product has about a
// third of the terms that R A P has term by term, and lists two indices per
// term instead of three.
// (A P)_ik = sum of A_ij P_jk over the row's j, LPR lanes per row, a lane per
// entry of A P.  The row's products are formed LPR at a time, a lane each (the
// lanes load an entry of A each, count the entries of P's rows below them and find
// their own) and put into LDS: every lane adds those of its column, in the order of
// the row.  (Each lane searching every P row for its column: chains of dependent
// loads, 97x81x65 807 us per numeric setup, now 218; 129^3 2.7 ms, now 0.76.  The
// products passed round by shuffles, five words each: 750 us and 2.65 ms.)
template <int LPR>
struct ApValues {
    int n;
    const int *__restrict__ rp, *__restrict__ ci;
    const double2 *__restrict__ av;
    const int *__restrict__ prp, *__restrict__ pci;
    const double2 *__restrict__ pv;
    const int *__restrict__ aprp, *__restrict__ apci;
    double2 *__restrict__ apv;
    __device__ void operator()(int, int) const
    {
        __shared__ double2 s_a[kBlock], s_v[kBlock];
        __shared__ int s_at[kBlock];
        __shared__ int4 s_c[kBlock / 4];
        const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
        const int i = (int)(g / LPR), lane = (int)(g % LPR), own = threadIdx.x - lane;  // own: the row's first place
        const bool act = i < n;
        const int b = act ? rp[i] : 0, e = act ? rp[i + 1] : 0;
        const int kb = act ? aprp[i] : 0, ke = act ? aprp[i + 1] : 0;
        for (int k0 = kb; wave_any(k0 < ke); k0 += LPR) {
            const int k = k0 + lane;
            const int mine = k < ke ? apci[k] : -1;
            double2 acc = make_double2(0.0, 0.0);
            for (int q0 = k0 < ke ? b : e; wave_any(q0 < e); q0 += LPR) {
                const int q = q0 + lane;
                const int j = q < e ? ci[q] : 0;
                const double2 a = q < e ? av[q] : make_double2(0.0, 0.0);
                const int s0 = q < e ? prp[j] : 0, len = q < e ? prp[j + 1] - s0 : 0;
                int upto = len;  // products of this lane's entry and those before it
#pragma unroll
                for (int o = 1; o < LPR; o *= 2) {
                    const int x = __shfl_up(upto, o, LPR);
                    if (lane >= o) upto += x;
                }
                const int total = __shfl(upto, LPR - 1, LPR);
                s_a[threadIdx.x] = a;
                s_at[threadIdx.x] = s0 - (upto - len);  // product m is entry s_at + m of P
                wave_sync();
                for (int m0 = 0; wave_any(m0 < total); m0 += LPR) {
                    const int m = m0 + lane;
                    int src = 0;  // the first lane with upto > m
#pragma unroll
                    for (int o = LPR / 2; o > 0; o /= 2)
                        if (__shfl(upto, src + o - 1, LPR) <= m) src += o;
                    const bool in = m < total;
                    const int at = s_at[own + src] + m;
                    reinterpret_cast<int *>(s_c)[threadIdx.x] = in ? pci[at] : -2;
                    s_v[threadIdx.x] = in ? cmul(s_a[own + src], pv[at]) : make_double2(0.0, 0.0);
                    wave_sync();
                    unsigned hit = 0;
#pragma unroll
                    for (int t = 0; t < LPR; t += 4) {
                        const int4 c = s_c[(own + t) / 4];
                        hit |= ((c.x == mine) | (c.y == mine) << 1 | (c.z == mine) << 2 | (c.w == mine) << 3) << t;
                    }
                    for (; hit; hit &= hit - 1) acc = cadd(acc, s_v[own + __ffs(hit) - 1]);
                    wave_sync();
                }
                wave_sync();
            }
            if (k < ke) apv[k] = acc;
        }
    }
};

// Upper triangle (J >= I) of R (A P), mirrored: entry t = the sum of R_p (A P)_k
// over its pairs, which are listed once per hierarchy (symbolic) in the order
// of the row.  kRapLanes lanes share an entry: lane j sums pairs j, j +
// kRapLanes, ... in order, then the lanes are added by a fixed butterfly, so a
// setup is bit-reproducible; neighbouring lanes read neighbouring pairs.
constexpr int kRapLanes = 8;

struct RapValues {
    int nnz;
    const int *__restrict__ tp;
    const int2 *__restrict__ pair;
    const int *__restrict__ mir;
    const double2 *__restrict__ rv, *__restrict__ apv;
    double2 *__restrict__ cv;
    __device__ void operator()(int, int) const
    {
        const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
        const int t = (int)(g / kRapLanes), lane = (int)(g % kRapLanes);
        const int b = t < nnz ? tp[t] : 0, e = t < nnz ? tp[t + 1] : 0;
        double2 acc = make_double2(0.0, 0.0);
        for (int k = b + lane; k < e; k += kRapLanes) {
            const int2 q = pair[k];
            acc = cadd(acc, cmul(rv[q.x], apv[q.y]));
        }
    #pragma unroll
        for (int o = kRapLanes / 2; o > 0; o >>= 1) {
            acc.x += __shfl_xor(acc.x, o, 64);
            acc.y += __shfl_xor(acc.y, o, 64);
        }
        if (lane != 0 || b == e) return;  // a lower entry has no pairs
        const int u = mir[t];
        if (u == t) {
            cv[t] = make_double2(acc.x, 0.0);
        } else {
            cv[t] = acc;
            cv[u] = cconj(acc);
        }
    }
};

struct ToF32c {
    int n;
    const double2 *a;
    float2 *b;
    __device__ void operator()(int, int) const
    {
        const int i = blockIdx.x * kBlock + threadIdx.x;
        if (i < n) b[i] = make_float2((float)a[i].x, (float)a[i].y);
    }
};

struct ToF32r {
    int n;
    const double *a;
    float *b;
    __device__ void operator()(int, int) const
    {
        const int i = blockIdx.x * kBlock + threadIdx.x;
        if (i < n) b[i] = (float)a[i];
    }
};

struct DenseFromCsr {
    int n;
    const int *rp, *ci;
    const double2 *v;
    double2 *M;
    __device__ void operator()(int, int) const
    {
        const int i = blockIdx.x * kBlock + threadIdx.x;
        if (i >= n) return;
        for (int j = 0; j < n; ++j) M[(size_t)i * n + j] = make_double2(0.0, 0.0);
        for (int p = rp[i]; p < rp[i + 1]; ++p) M[(size_t)i * n + ci[p]] = v[p];
    }
};

// Cholesky factor M = L L^H of the Hermitian coarsest operator, in place
// (row-major, lower triangle; the upper part zeroed at the end), blocked
// right-looking: a panel of pw columns is factored in LDS by one work-group
// (k_chol_panel), then every work-group updates its share of the trailing
// lower triangle with that panel (k_chol_update).  status = 1 when a pivot is
// not positive relative to the largest diagonal entry of M (k_chol_init);
// every later kernel returns at once then.
constexpr int kCholLds = (65536 - 1024) / sizeof(double2);  // panel entries held in LDS

int chol_panel_width(int n) { return std::max(1, std::min(32, kCholLds / std::max(n, 1))); }

struct CholInit {
    int n;
    const double2 *M;
    double *dmax;
    int *status;
    __device__ void operator()(int, int) const
    {
        __shared__ double sm[1024 / 64];
        double m = 0.0;
        for (int i = threadIdx.x; i < n; i += blockDim.x) m = fmax(m, fabs(M[(size_t)i * n + i].x));
        for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_down(m, o, 64));
        if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
        __syncthreads();
        if (threadIdx.x == 0) {
            double r = 0.0;
            for (int w = 0; w < (int)(blockDim.x >> 6); ++w) r = fmax(r, sm[w]);
            *dmax = r;
            *status = 0;
        }
    }
};

// columns p0 .. p0 + pw - 1, rows p0 .. n - 1 (already updated by the
// earlier panels): P[r * pw + c] = M[p0 + r][p0 + c]
struct CholPanel {
    int n, p0, pw;
    double2 *M;
    const double *dmaxp;
    int *status;
    __device__ void operator()(int, int) const
    {
        __shared__ double2 P[kCholLds];
        __shared__ double piv;
        __shared__ int bad;
        if (*status) return;
        const int rows = n - p0;
        const double dmax = *dmaxp;
        for (int t = threadIdx.x; t < rows * pw; t += blockDim.x)
            P[t] = M[(size_t)(p0 + t / pw) * n + p0 + t % pw];
        if (threadIdx.x == 0) bad = 0;
        __syncthreads();
        for (int c = 0; c < pw; ++c) {
            if (threadIdx.x == 0) {
                const double d = P[c * pw + c].x;
                if (!(d > 1e-12 * dmax)) bad = 1;
                else {
                    piv = sqrt(d);
                    P[c * pw + c] = make_double2(piv, 0.0);
                }
            }
            __syncthreads();
            if (bad) break;
            const double inv = 1.0 / piv;
            for (int r = c + 1 + threadIdx.x; r < rows; r += blockDim.x) P[r * pw + c] = cscale(P[r * pw + c], inv);
            __syncthreads();
            // the panel's remaining columns c' > c, rows r >= c'
            const int w = pw - c - 1;
            for (int t = threadIdx.x; t < (rows - c - 1) * w; t += blockDim.x) {
                const int r = c + 1 + t / w, q = c + 1 + t % w;
                if (r >= q) P[r * pw + q] = csub(P[r * pw + q], cmul(P[r * pw + c], cconj(P[q * pw + c])));
            }
            __syncthreads();
        }
        if (bad) {
            if (threadIdx.x == 0) *status = 1;
            return;
        }
        for (int t = threadIdx.x; t < rows * pw; t += blockDim.x) {
            const int r = t / pw, c = t % pw;
            if (r >= c) M[(size_t)(p0 + r) * n + p0 + c] = P[t];
        }
    }
};

// M[i][k] -= sum_c L[i][p0 + c] conj(L[k][p0 + c]) for p0 + pw <= k <= i < n
// One 16 x 16 tile of the trailing matrix per work-group of 256 threads:
// tile bx = (tile row) * tiles + (tile column), tiles = ceil((n - p0 - pw) / 16).
struct CholUpdate {
    int n, p0, pw, tiles;
    double2 *M;
    const int *status;
    __device__ void operator()(int bx, int) const
    {
        if (*status) return;
        const int b = p0 + pw;
        const int i = b + (bx / tiles) * 16 + (int)(threadIdx.x >> 4);
        const int k = b + (bx % tiles) * 16 + (int)(threadIdx.x & 15);
        if (i >= n || k > i) return;
        const double2 *li = M + (size_t)i * n + p0, *lk = M + (size_t)k * n + p0;
        double2 acc = make_double2(0.0, 0.0);
        for (int c = 0; c < pw; ++c) acc = cadd(acc, cmul(li[c], cconj(lk[c])));
        M[(size_t)i * n + k] = csub(M[(size_t)i * n + k], acc);
    }
};

struct CholZeroUpper {
    int n;
    double2 *M;
    __device__ void operator()(int, int) const
    {
        const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
        if (t >= (int64_t)n * n) return;
        if (t % n > t / n) M[t] = make_double2(0.0, 0.0);
    }
};

static void cholesky(int n, double2 *M, double *dmax, int *status, const Launch &L)
{
    L.run<CholInit, 1024>(1, CholInit{n, M, dmax, status});
    const int pb = chol_panel_width(n);
    for (int p0 = 0; p0 < n; p0 += pb) {
        const int pw = std::min(pb, n - p0);
        L.run<CholPanel, 1024>(1, CholPanel{n, p0, pw, M, dmax, status});
        const int m = n - p0 - pw;
        const int tiles = (m + 15) / 16;
        if (m > 0) L.run(tiles * tiles, CholUpdate{n, p0, pw, tiles, M, status});
    }
    L.run(blocks_for((int64_t)n * n), CholZeroUpper{n, M});
}

// Column j of (L L^H)^-1 (one work-group per column), stored row-major.
struct CholInverse {
    int n;
    const double2 *__restrict__ Lf;
    double2 *inv;
    const int *status;  // nonzero: the factorisation failed, nothing to invert
    __device__ void operator()(int, int) const
    {
        if (*status) return;
        __shared__ double2 y[kMaxDense];
        const int j = blockIdx.x;
        for (int i = threadIdx.x; i < n; i += blockDim.x) y[i] = make_double2(i == j ? 1.0 : 0.0, 0.0);
        __syncthreads();
        for (int k = j; k < n; ++k) {  // L y = e_j
            const double2 yk = cscale(y[k], 1.0 / Lf[(size_t)k * n + k].x);
            __syncthreads();
            for (int i = k + 1 + threadIdx.x; i < n; i += blockDim.x) y[i] = csub(y[i], cmul(Lf[(size_t)i * n + k], yk));
            if (threadIdx.x == 0) y[k] = yk;
            __syncthreads();
        }
        for (int k = n - 1; k >= 0; --k) {  // L^H x = y
            const double2 yk = cscale(y[k], 1.0 / Lf[(size_t)k * n + k].x);
            __syncthreads();
            for (int i = threadIdx.x; i < k; i += blockDim.x) y[i] = csub(y[i], cmulc(Lf[(size_t)k * n + i], yk));
            if (threadIdx.x == 0) y[k] = yk;
            __syncthreads();
        }
        for (int i = threadIdx.x; i < n; i += blockDim.x) inv[(size_t)i * n + j] = y[i];
    }
};

// ------------------------------------------------- colour renumbering --
__global__ void k_iperm(int n, const int *perm, int *iperm)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r < n) iperm[perm[r]] = r;
}

// length of old row rowperm[r] (identity when rowperm is NULL)
__global__ void k_perm_count(int nrows, const int *rowperm, const int *rp, int *cnt)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= nrows) return;
    const int o = rowperm ? rowperm[r] : r;
    cnt[r] = rp[o + 1] - rp[o];
}

// row r of the copy = old row rowperm[r] with columns relabelled by colmap
__global__ void k_perm_fill(int nrows, const int *rowperm, const int *rp, const int *ci, const int *colmap,
                            const int *nrp, int *nci, int *map)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= nrows) return;
    const int o = rowperm ? rowperm[r] : r;
    int q = nrp[r];
    for (int p = rp[o]; p < rp[o + 1]; ++p, ++q) {
        nci[q] = colmap ? colmap[ci[p]] : ci[p];
        map[q] = p;
    }
}

// place of the diagonal entry of each sorted row
__global__ void k_diag_place(int n, const int *rp, const int *ci, int *dpos)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= n) return;
    int p = rp[r];
    while (p < rp[r + 1] && ci[p] < r) ++p;
    dpos[r] = p;
}

// Level-0 restriction without the red columns: the level-0 residual the
// V-cycle restricts is zero on red nodes (their last pre-smoothing update
// zeroes it), so those entries only ever multiply zeros.  Row r keeps the
// entries of columns i with (c0 + c1 + c2) odd; map composes the copy's entry
// with the value map of the source copy.
__device__ __forceinline__ bool black_node(const GeomT<double> &g, int i)
{
    const int c0 = i % g.N[0], r = i / g.N[0];
    const int c1 = r % g.N[1], c2 = r / g.N[1];
    return ((c0 + c1 + c2) & 1) != 0;
}

__global__ void k_black_count(int nrows, GeomT<double> g, const int *rp, const int *ci, int *cnt)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= nrows) return;
    int c = 0;
    for (int p = rp[r]; p < rp[r + 1]; ++p) c += black_node(g, ci[p]);
    cnt[r] = c;
}

// columns numbered as the V-cycle stores level-0 vectors: black node i of
// red-black pair t at npair + t
__global__ void k_black_fill(int nrows, GeomT<double> g, const int *rp, const int *ci, const int *srcmap,
                             const int *nrp, int *nci, int *map)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= nrows) return;
    int q = nrp[r];
    for (int p = rp[r]; p < rp[r + 1]; ++p) {
        const int i = ci[p];
        if (black_node(g, i)) {
            nci[q] = g.npair + (i / g.N[0]) * g.hr + (i % g.N[0]) / 2;
            map[q] = srcmap[p];
            ++q;
        }
    }
}

// Level-0 prolongation rows of the black nodes only, row t = the black node
// of red-black pair t (empty where the pair has none): the V-cycle corrects
// only black nodes from the coarse level, and the copy keeps those rows
// contiguous.  map composes with the value map of the source copy.
__device__ __forceinline__ int pair_black(const GeomT<double> &g, int t)
{
    const int row = t / g.hr, c0 = 2 * (t - row * g.hr);
    const int c1 = row % g.N[1], c2 = row / g.N[1];
    const int s = (1 + c1 + c2) & 1;
    return c0 + s < g.N[0] ? c0 + s + g.N[0] * row : -1;
}

__global__ void k_pblack_count(GeomT<double> g, const int *rp, int *cnt)
{
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= g.npair) return;
    const int i = pair_black(g, t);
    cnt[t] = i < 0 ? 0 : rp[i + 1] - rp[i];
}

__global__ void k_pblack_fill(GeomT<double> g, const int *rp, const int *ci, const int *srcmap, const int *nrp,
                              int *nci, int *map)
{
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= g.npair) return;
    const int i = pair_black(g, t);
    if (i < 0) return;
    int q = nrp[t];
    for (int p = rp[i]; p < rp[i + 1]; ++p, ++q) {
        nci[q] = ci[p];
        map[q] = srcmap[p];
    }
}

// the level-0 diagonal in the colour-split layout (an absent odd node's slot
// holds 1)
struct SplitDiag {
    GeomT<double> g;
    const double *d;
    double *s64;
    float *s32;
    __device__ void operator()(int, int) const
    {
        const int t = blockIdx.x * kBlock + threadIdx.x;
        if (t >= g.npair) return;
        const int row = t / g.hr, c0 = 2 * (t - row * g.hr);
        const int c1 = row % g.N[1], c2 = row / g.N[1];
        const int ie = c0 + g.N[0] * row, ce = (c0 + c1 + c2) & 1;
        const double de = d[ie], dodd = c0 + 1 < g.N[0] ? d[ie + 1] : 1.0;
        s64[ce * g.npair + t] = de;
        s32[ce * g.npair + t] = (float)de;
        s64[(1 - ce) * g.npair + t] = dodd;
        s32[(1 - ce) * g.npair + t] = (float)dodd;
    }
};

struct GatherC {
    int nnz;
    const int *map;
    const double2 *src;
    double2 *d64;
    float2 *d32;
    __device__ void operator()(int, int) const
    {
        const int q = blockIdx.x * kBlock + threadIdx.x;
        if (q >= nnz) return;
        const double2 v = src[map[q]];
        d64[q] = v;
        d32[q] = make_float2((float)v.x, (float)v.y);
    }
};

// padded block of one colour (rows row0 .. row0 + count - 1 of Aa), row-major:
// entry k of row r at r W + k
__global__ void k_ell_fill(int row0, int count, int W, const int *rp, const int *ci, int *eci, int *emap)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= count) return;
    const int i = row0 + r;
    const int b = rp[i], len = rp[i + 1] - rp[i];
    for (int k = 0; k < W; ++k) {
        eci[(size_t)r * W + k] = k < len ? ci[b + k] : i;
        emap[(size_t)r * W + k] = k < len ? b + k : -1;
    }
}

// the rows of the prolongation padded to W entries: (column 0, no entry)
__global__ void k_pell_fill(int n, int W, const int *rp, const int *ci, int *pci, int *pmap)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= n) return;
    const int b = rp[r], len = rp[r + 1] - rp[r];
    for (int k = 0; k < W; ++k) {
        pci[(size_t)r * W + k] = k < len ? ci[b + k] : 0;
        pmap[(size_t)r * W + k] = k < len ? b + k : -1;
    }
}

struct EllValues {
    int n;
    const int *emap;
    const double2 *src;
    double2 *d64;
    float2 *d32;
    __device__ void operator()(int, int) const
    {
        const int q = blockIdx.x * kBlock + threadIdx.x;
        if (q >= n) return;
        const int p = emap[q];
        const double2 v = p >= 0 ? src[p] : make_double2(0.0, 0.0);
        d64[q] = v;
        d32[q] = make_float2((float)v.x, (float)v.y);
    }
};

// ----------------------------------------------------------- patches --
// The level-0 node of every aggregate's root, through the levels' roots.
__global__ void k_origin(int nc, const int *root, const int *origin, int *out)
{
    const int a = blockIdx.x * kBlock + threadIdx.x;
    if (a < nc) out[a] = origin ? origin[root[a]] : root[a];
}

// Tile of each row (new order): the place of its level-0 node in a kx x ky
// grid of tiles over the domain.
struct TileGrid {
    int simplicial;
    int N0, N1;            // grid
    const double *x;       // simplicial: node coordinates (3 per node)
    double lo[2], inv[2];  // simplicial: lower corner, 1 / extent
    int k[2];
};

__global__ void k_tile_of(int n, const int *perm, const int *origin, TileGrid t, int *tile)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= n) return;
    const int o = perm[r], i = origin ? origin[o] : o;
    int c[2];
    if (t.simplicial) {
        for (int a = 0; a < 2; ++a)
            c[a] = min(t.k[a] - 1, max(0, (int)((t.x[3 * (size_t)i + a] - t.lo[a]) * t.inv[a] * t.k[a])));
    } else {
        c[0] = (int)((int64_t)(i % t.N0) * t.k[0] / t.N0);
        c[1] = (int)((int64_t)(i / t.N0 % t.N1) * t.k[1] / t.N1);
    }
    tile[r] = c[1] * t.k[0] + c[0];
}

__global__ void k_tile_fill(int n, const int *tile, const int *rp, int *fill, int *rows)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= n) return;
    const int t = tile[r];
    rows[rp[t] + atomicAdd(&fill[t], 1)] = r;
}

// Patch blockIdx.x from its own rows own[beg .. end): going back from the end
// of the sweep, pass t needs every value its rows read, so a row joins the
// patch when the first of its neighbours' passes after which it is needed is
// met, and is then updated in every earlier pass of its colour.  (Rows of one
// colour are not adjacent, so a pass widens the patch only around its own
// colour: a symmetric sweep of 5-8 colours on the 2D hierarchies reaches three
// or four rows out, not one per pass.)  The residual and the own rows' last
// pass need the neighbours' final values.  Overflow: err 32.
template <int NR>
__global__ __launch_bounds__(NR) void k_patch_build(const int *__restrict__ tile_rp,
                                                            const int *__restrict__ tile_rows,
                                                            const int *__restrict__ rp, const int *__restrict__ ci,
                                                            const int *__restrict__ perm, const int *__restrict__ color,
                                                            int ncol, int W, int *size, int *rowid, int *info,
                                                            unsigned short *idx, int *map, int *total, int *err)
{
    constexpr int NS = 2 * NR, H = 2 * NS;
    __shared__ int key[H], val[H], row[NS], last[NS], place[NS];
    __shared__ unsigned char col[NS], done[NS];
    __shared__ int cnt, nrows, bad;
    const int p = blockIdx.x, tid = threadIdx.x;
    const int beg = tile_rp[p], end = tile_rp[p + 1];
    for (int t = tid; t < H; t += NR) key[t] = -1;
    for (int t = tid; t < NS; t += NR) {
        done[t] = 0;
        rowid[(size_t)p * NS + t] = 0;  // slots without a row read row 0 and write nothing
    }
    info[(size_t)p * NR + tid] = 255;
    if (tid == 0) cnt = nrows = bad = 0;
    __syncthreads();
    auto insert = [&](int g, int e) {
        if (load_relaxed(&bad)) return;  // (a full table would be walked round by every further row)
        unsigned h = ((unsigned)g * 2654435761u) % H;
        for (int tries = 0; tries < H; ++tries, h = (h + 1) % H) {
            const int old = atomicCAS(&key[h], -1, g);
            if (old == g) return;
            if (old != -1) continue;
            const int slot = atomicAdd(&cnt, 1);
            if (slot >= NS) {
                store_relaxed(&bad, 1);
                return;
            }
            val[h] = slot;
            row[slot] = g;
            last[slot] = e;
            col[slot] = (unsigned char)color[perm[g]];
            return;
        }
        store_relaxed(&bad, 1);
    };
    const int T = 2 * ncol - 1;
    for (int q = beg + tid; q < end; q += NR) insert(tile_rows[q], T);
    __syncthreads();
    for (int q = beg + tid; q < end; q += NR) {
        const int g = tile_rows[q];
        for (int k = rp[g]; k < rp[g + 1]; ++k) insert(ci[k], T);
    }
    __syncthreads();
    for (int t = T - 1; t >= 0; --t) {
        const int c = t < ncol ? t : 2 * ncol - 2 - t;
        const int n0 = min(cnt, NS), over = bad;
        __syncthreads();
        if (over) break;
        for (int s = tid; s < n0; s += NR)
            if (col[s] == c && last[s] > t && !done[s]) {
                done[s] = 1;
                const int g = row[s];
                for (int k = rp[g]; k < rp[g + 1]; ++k) insert(ci[k], t);
            }
        __syncthreads();
    }
    __syncthreads();
    const int n = min(cnt, NS);
    if (!bad)
        for (int s = tid; s < n; s += NR)
            if (done[s]) atomicAdd(&nrows, 1);
    __syncthreads();
    const int nr = nrows;
    if (bad || nr > NR) {
        if (tid == 0) atomicOr(err, 32);
        return;
    }
    // the places: updated rows first, then the others, each in row order
    for (int s = tid; s < n; s += NR) {
        int rank = done[s] ? 0 : nr;
        for (int q = 0; q < n; ++q) rank += done[q] == done[s] && row[q] < row[s];
        place[s] = rank;
        rowid[(size_t)p * NS + rank] = row[s];
    }
    if (tid == 0) {
        size[2 * p] = nr;
        size[2 * p + 1] = n;
        atomicAdd(total, nr);
    }
    __syncthreads();
    const size_t base = (size_t)p * W * NR;
    for (int t = tid; t < W * NR; t += NR) {
        idx[base + t] = NS;
        map[base + t] = -1;
    }
    __syncthreads();
    for (int s = tid; s < n; s += NR) {
        if (!done[s]) continue;
        const int g = row[s], r = place[s];
        int own = 0;
        for (int q = beg; q < end; ++q) own |= tile_rows[q] == g;
        int k = 0;
        for (int q = rp[g]; q < rp[g + 1]; ++q) {
            const int j = ci[q];
            if (j == g) continue;
            unsigned h = ((unsigned)j * 2654435761u) % H;
            for (int tries = 0; tries < H && key[h] != j; ++tries) h = (h + 1) % H;
            idx[base + (size_t)k * NR + r] = (unsigned short)place[val[h]];
            map[base + (size_t)k * NR + r] = q;
            ++k;
        }
        info[(size_t)p * NR + r] = col[s] | last[s] << 8 | own << 16 | k << 20;
    }
}

struct GatherR {
    int n;
    const int *perm;
    const double *src;
    double *d64;
    float *d32;
    __device__ void operator()(int, int) const
    {
        const int r = blockIdx.x * kBlock + threadIdx.x;
        if (r >= n) return;
        const double v = src[perm[r]];
        d64[r] = v;
        d32[r] = (float)v;
    }
};

// ------------------------------------------------------------- host ---
static int read_int(const int *d, hipStream_t s)
{
    int h = 0;
    GLK_HIP(hipMemcpyAsync(&h, d, sizeof(int), hipMemcpyDeviceToHost, s));
    GLK_HIP(hipStreamSynchronize(s));
    return h;
}

static void check_err(const DevBuf<int> &err, hipStream_t s, const char *what)
{
    const int e = read_int(err.get(), s);
    if (e & 2 || e & 4) fail(GL_ERR_UNSUPPORTED, std::string(what) + ": a coarse row exceeds the setup row limit");
    if (e & 8) fail(GL_ERR_UNSUPPORTED, std::string(what) + ": more than 256 colours");
    if (e & 16) fail(GL_ERR_HIP, std::string(what) + ": a coarse pattern is not symmetric");
    if (e) fail(GL_ERR_HIP, std::string(what) + ": aggregation left a node unassigned");
}

// CSR pattern (rp from counts, then columns) helper
static void alloc_rowptr(Csr &M, const int *cnt, SymTmp &T, hipStream_t s)
{
    M.rp.alloc((size_t)M.n + 1);
    const int64_t nnz = scan_excl(cnt, M.rp.get(), M.n, T, s);
    if (nnz > INT32_MAX - 1) fail(GL_ERR_UNSUPPORTED, "sparse matrix too large");
    M.nnz = (int)nnz;
    M.ci.alloc((size_t)std::max(1, M.nnz));
}

// Launches rounds of a wave-like decision until none of its nodes is
// undecided: round(flag) enqueues one round, which sets *flag when nodes are
// left.  The host looks after a batch of rounds only (rounds after the last
// decision change nothing), and a batch grows with the rounds already run.
template <class Round>
static void run_rounds(int n, SymTmp &T, hipStream_t s, const char *what, Round &&round)
{
    constexpr int slots = 256;
    int *flags = need(T, T.flags, slots), slot = 0;
    int64_t done = 0;
    for (;;) {
        if (done > (int64_t)n + 8) fail(GL_ERR_HIP, std::string(what) + " did not terminate");
        if (slot == 0) k_fill_int<<<1, slots, 0, s>>>(flags, slots, 0);
        const int batch = 8 + (int)std::min<int64_t>(done / 4, 64);
        for (int r = 0; r < batch; ++r) round(r + 1 == batch ? flags + slot : nullptr);
        GLK_CHECK_LAUNCH();
        done += batch;
        if (read_int(flags + slot, s) == 0) return;
        slot = (slot + 1) % slots;
    }
}

static void colour_level(gl_precond *pre, int l, SymTmp &T, hipStream_t s)
{
    Level &L = pre->L[l];
    const int n = L.n, nb = blocks_for(n);
    L.color.alloc(n);
    const gl_mesh *m = pre->mesh;
    if (l == 0 && !m->g.simplicial) {
        if (m->g.dim == 2) k_parity_colour<2><<<nb, kBlock, 0, s>>>(m->g, L.color.get());
        else k_parity_colour<3><<<nb, kBlock, 0, s>>>(m->g, L.color.get());
        GLK_CHECK_LAUNCH();
        L.ncolors = n > 1 ? 2 : 1;
    } else {
        int *err = need(T, T.err, 1);
        k_fill_int<<<1, 64, 0, s>>>(err, 1, 0);
        k_fill_int<<<nb, kBlock, 0, s>>>(L.color.get(), n, -1);
        run_rounds(n, T, s, "colouring", [&](int *flag) {
            k_jp_round<<<nb, kBlock, 0, s>>>(n, L.A.rp.get(), L.A.ci.get(), L.color.get(), flag, err);
        });
        check_err(T.err, s, "colouring");
        // class sizes and the number of colours
        int *hist = need(T, T.a, 257);
        std::vector<int> h;
        int nc = 0;
        auto count = [&] {
            k_fill_int<<<2, kBlock, 0, s>>>(hist, 257, 0);
            k_colour_hist<<<std::min(nb, 256), kBlock, 0, s>>>(n, L.color.get(), hist);
            GLK_CHECK_LAUNCH();
            h = to_host(hist, 257, s);
            nc = 0;
            for (int c = 0; c < 257; ++c)
                if (h[c]) nc = c + 1;
        };
        count();
        // iterated greedy: never more colours, often fewer (each colour costs
        // two dependent passes per symmetric sweep)
        int *nw = need(T, T.b, n);
        for (int pass = 0; pass < kRecolourPasses; ++pass) {
            k_fill_int<<<nb, kBlock, 0, s>>>(nw, n, -1);
            for (int c = nc - 1; c >= 0; --c)
                k_ig_class<<<nb, kBlock, 0, s>>>(n, L.A.rp.get(), L.A.ci.get(), L.color.get(), c, nw, err);
            GLK_CHECK_LAUNCH();
            GLK_HIP(hipMemcpyAsync(L.color.get(), nw, sizeof(int) * (size_t)n, hipMemcpyDeviceToDevice, s));
            count();
        }
        check_err(T.err, s, "recolouring");
        L.ncolors = nc;
        // rows grouped by colour
        L.cperm.alloc(n);
        L.coff.assign(nc + 1, 0);
        for (int c = 0; c < nc; ++c) L.coff[c + 1] = L.coff[c] + h[c];
        int *bc = need(T, T.b, (size_t)nc * nb), *off = need(T, T.c, (size_t)nc * nb + 1);
        k_colour_count<<<nb, kBlock, 0, s>>>(n, L.color.get(), nb, nc, bc);
        scan_excl(bc, off, nc * nb, T, s);
        k_colour_place<<<nb, kBlock, 0, s>>>(n, L.color.get(), nb, off, L.cperm.get());
        GLK_CHECK_LAUNCH();
    }
}

// aggregation of level l; returns the number of aggregates
static int aggregate_level(gl_precond *pre, int l, SymTmp &T, hipStream_t s)
{
    Level &L = pre->L[l];
    const int n = L.n, nb = blocks_for(n);
    const int *rp = L.A.rp.get(), *ci = L.A.ci.get();
    int *state = need(T, T.a, n), *rootA = need(T, T.b, n), *rootB = need(T, T.c, n), *flag = need(T, T.d, n);
    int *id = need(T, T.e, (size_t)n + 1), *err = need(T, T.err, 1);
    k_fill_int<<<nb, kBlock, 0, s>>>(state, n, 0);
    k_fill_int<<<1, 64, 0, s>>>(err, 1, 0);
    run_rounds(n, T, s, "aggregation",
               [&](int *left) { k_mis_round<<<nb, kBlock, 0, s>>>(n, rp, ci, state, left); });
    k_agg_phase_a<<<nb, kBlock, 0, s>>>(n, rp, ci, state, rootA);
    k_agg_phase_b<<<nb, kBlock, 0, s>>>(n, rp, ci, rootA, rootB, err);
    k_root_flags<<<nb, kBlock, 0, s>>>(n, state, flag);
    GLK_CHECK_LAUNCH();
    check_err(T.err, s, "aggregation");
    const int nc = (int)scan_excl(flag, id, n, T, s);
    L.nc = nc;
    L.agg.alloc(n);
    L.root.alloc(std::max(1, nc));
    L.aggsize.alloc(std::max(1, nc));
    k_fill_int<<<blocks_for(std::max(1, nc)), kBlock, 0, s>>>(L.aggsize.get(), std::max(1, nc), 0);
    k_agg_number<<<nb, kBlock, 0, s>>>(n, rootB, id, state, L.agg.get(), L.root.get(), L.aggsize.get());
    GLK_CHECK_LAUNCH();
    return nc;
}

static void transfer_patterns(gl_precond *pre, int l, SymTmp &T, hipStream_t s)
{
    Level &L = pre->L[l];
    Level &Nx = pre->L[l + 1];
    const int n = L.n, nc = L.nc, nb = blocks_for(n);
    const int nbw = (nc + kRowWaves - 1) / kRowWaves;  // a wave per coarse row
    int *cnt = need(T, T.a, std::max(n, nc)), *err = need(T, T.err, 1);
    k_fill_int<<<1, 64, 0, s>>>(err, 1, 0);
    // P: n x nc
    L.P.n = n;
    L.P.m = nc;
    k_p_pattern<<<nb, kBlock, 0, s>>>(n, L.A.rp.get(), L.A.ci.get(), L.agg.get(), nullptr, cnt, nullptr, err);
    GLK_CHECK_LAUNCH();
    check_err(T.err, s, "prolongator pattern");
    alloc_rowptr(L.P, cnt, T, s);
    k_p_pattern<<<nb, kBlock, 0, s>>>(n, L.A.rp.get(), L.A.ci.get(), L.agg.get(), L.P.rp.get(), nullptr, L.P.ci.get(),
                                      err);
    // R = P^H: nc x n
    L.R.n = nc;
    L.R.m = n;
    k_fill_int<<<blocks_for(nc), kBlock, 0, s>>>(cnt, nc, 0);
    k_col_count<<<blocks_for(L.P.nnz), kBlock, 0, s>>>(L.P.nnz, L.P.ci.get(), cnt);
    GLK_CHECK_LAUNCH();
    alloc_rowptr(L.R, cnt, T, s);
    L.rsrc.alloc(std::max(1, L.R.nnz));
    int *fill = need(T, T.b, nc), *tci = need(T, T.c, std::max(1, L.R.nnz)), *tsrc = need(T, T.d, std::max(1, L.R.nnz));
    k_fill_int<<<blocks_for(nc), kBlock, 0, s>>>(fill, nc, 0);
    k_transpose_fill<<<nb, kBlock, 0, s>>>(n, L.P.rp.get(), L.P.ci.get(), L.R.rp.get(), fill, tci, tsrc);
    k_sort_rows<<<nbw, kBlock, 0, s>>>(nc, L.R.rp.get(), tci, tsrc, L.R.ci.get(), L.rsrc.get());
    GLK_CHECK_LAUNCH();
    // A P pattern
    L.AP.n = n;
    L.AP.m = nc;
    k_ap_pattern<<<nb, kBlock, 0, s>>>(n, L.A.rp.get(), L.A.ci.get(), L.P.rp.get(), L.P.ci.get(), nullptr, cnt, nullptr,
                                       err);
    GLK_CHECK_LAUNCH();
    check_err(T.err, s, "Galerkin pattern");
    alloc_rowptr(L.AP, cnt, T, s);
    k_ap_pattern<<<nb, kBlock, 0, s>>>(n, L.A.rp.get(), L.A.ci.get(), L.P.rp.get(), L.P.ci.get(), L.AP.rp.get(), nullptr,
                                       L.AP.ci.get(), err);
    // A_{l+1} = R A P pattern
    Nx.n = nc;
    Nx.A.n = nc;
    Nx.A.m = nc;
    k_rap_pattern<<<nbw, kBlock, 0, s>>>(nc, L.R.rp.get(), L.R.ci.get(), L.AP.rp.get(), L.AP.ci.get(), nullptr, cnt,
                                         nullptr, err);
    GLK_CHECK_LAUNCH();
    check_err(T.err, s, "Galerkin pattern");
    alloc_rowptr(Nx.A, cnt, T, s);
    k_rap_pattern<<<nbw, kBlock, 0, s>>>(nc, L.R.rp.get(), L.R.ci.get(), L.AP.rp.get(), L.AP.ci.get(), Nx.A.rp.get(),
                                         nullptr, Nx.A.ci.get(), err);
    GLK_CHECK_LAUNCH();
    // the pairs of the upper triangle for the numeric Galerkin product
    const int nnzc = Nx.A.nnz;
    int *pc = need(T, T.b, std::max(1, nnzc));
    k_rap_pairs<<<nbw, kBlock, 0, s>>>(nc, L.R.rp.get(), L.R.ci.get(), L.AP.rp.get(), L.AP.ci.get(), Nx.A.rp.get(),
                                       Nx.A.ci.get(), pc, nullptr, nullptr);
    GLK_CHECK_LAUNCH();
    L.rap_tp.alloc((size_t)nnzc + 1);
    const int64_t npair = scan_excl(pc, L.rap_tp.get(), nnzc, T, s);
    if (npair < 0 || npair > (int64_t)1 << 30) fail(GL_ERR_UNSUPPORTED, "Galerkin product: too many products");
    L.rap_pair.alloc((size_t)std::max<int64_t>(1, npair));
    L.rap_mir.alloc(std::max(1, nnzc));
    k_rap_pairs<<<nbw, kBlock, 0, s>>>(nc, L.R.rp.get(), L.R.ci.get(), L.AP.rp.get(), L.AP.ci.get(), Nx.A.rp.get(),
                                       Nx.A.ci.get(), nullptr, L.rap_tp.get(), L.rap_pair.get());
    k_rap_mirror<<<blocks_for((int64_t)nc * 8), kBlock, 0, s>>>(nc, Nx.A.rp.get(), Nx.A.ci.get(), L.rap_mir.get(), err);
    GLK_CHECK_LAUNCH();
    check_err(T.err, s, "Galerkin product");
}

static void alloc_values(gl_precond *pre)
{
    const bool simp = pre->mesh->g.simplicial;
    const int ns = simp ? 0 : 2 * geom_t<double>(pre->mesh->g).npair;  // level-0 split layout of a grid
    for (int l = 0; l < pre->nlev; ++l) {
        Level &L = pre->L[l];
        const int nv = l == 0 ? std::max(L.n, ns) : L.n;
        L.A.v64.alloc(std::max(1, L.A.nnz));
        L.A.v32.alloc(std::max(1, L.A.nnz));
        L.diag64.alloc(L.n);
        L.diag32.alloc(L.n);
        L.b64.alloc(nv);
        L.x64.alloc(nv);
        L.r64.alloc(nv);
        L.b32.alloc(nv);
        L.x32.alloc(nv);
        L.r32.alloc(nv);
        if (l > 0 || simp) {
            L.t64.alloc(nv);
            L.t32.alloc(nv);
        }
        if (l == 0 && !simp) {
            L.hs64.alloc(ns);
            L.hs32.alloc(ns);
        }
        if (l < pre->nlev - 1) {
            L.P.v64.alloc(std::max(1, L.P.nnz));
            L.P.v32.alloc(std::max(1, L.P.nnz));
            L.AP.v64.alloc(std::max(1, L.AP.nnz));
            L.R.v64.alloc(std::max(1, L.R.nnz));
            L.R.v32.alloc(std::max(1, L.R.nnz));
            L.rho.alloc(1);
        }
    }
    const int nl = pre->L[pre->nlev - 1].n;
    pre->cfac.alloc((size_t)nl * nl);
    pre->cinv64.alloc((size_t)nl * nl);
    pre->cinv32.alloc((size_t)nl * nl);
    pre->status.alloc(1);
    pre->cdmax.alloc(1);
    const int n0 = pre->L[0].n;
    pre->cyc_r.alloc(n0);
    pre->vin.alloc(n0);
    pre->pwn.alloc(2);
}

// copy of M with rows taken in the order rowperm and columns relabelled by colmap
// (sorted: rows in ascending order of the new columns)
static void permuted_copy(const Csr &M, const int *rowperm, const int *colmap, Csr &out, DevBuf<int> &map,
                          SymTmp &T, hipStream_t s, bool sorted = false)
{
    out.n = M.n;
    out.m = M.m;
    int *cnt = need(T, T.a, std::max(1, M.n));
    k_perm_count<<<blocks_for(M.n), kBlock, 0, s>>>(M.n, rowperm, M.rp.get(), cnt);
    GLK_CHECK_LAUNCH();
    alloc_rowptr(out, cnt, T, s);
    map.alloc(std::max(1, out.nnz));
    int *fci = sorted ? need(T, T.b, std::max(1, out.nnz)) : out.ci.get();
    int *fmap = sorted ? need(T, T.c, std::max(1, out.nnz)) : map.get();
    k_perm_fill<<<blocks_for(M.n), kBlock, 0, s>>>(M.n, rowperm, M.rp.get(), M.ci.get(), colmap, out.rp.get(), fci, fmap);
    if (sorted)
        k_sort_rows<<<(M.n + kRowWaves - 1) / kRowWaves, kBlock, 0, s>>>(M.n, out.rp.get(), fci, fmap, out.ci.get(),
                                                                         map.get());
    GLK_CHECK_LAUNCH();
    out.v64.alloc(std::max(1, out.nnz));
    out.v32.alloc(std::max(1, out.nnz));
}

static void build_patches(gl_precond *pre, int l, SymTmp &T, hipStream_t s);

// the colour-ordered copies the V-cycle works on
static void build_apply_copies(gl_precond *pre, SymTmp &T, hipStream_t s)
{
    // level 0 of a simplicial mesh is a CSR level like the coarse ones (when
    // it is not the coarsest, which is applied as a dense inverse in node order)
    const bool simp = pre->mesh->g.simplicial && pre->nlev > 1;
    const int lfirst = simp ? 0 : 1;
    for (int l = 1; l < pre->nlev; ++l) {
        Level &L = pre->L[l];
        L.origin.alloc(L.n);
        k_origin<<<blocks_for(L.n), kBlock, 0, s>>>(L.n, pre->L[l - 1].root.get(), pre->L[l - 1].origin.get(),
                                                    L.origin.get());
        GLK_CHECK_LAUNCH();
    }
    for (int l = lfirst; l < pre->nlev; ++l) {
        Level &L = pre->L[l];
        L.perm.alloc(L.n);
        GLK_HIP(hipMemcpyAsync(L.perm.get(), L.cperm.get(), sizeof(int) * L.n, hipMemcpyDeviceToDevice, s));
        L.iperm.alloc(L.n);
        k_iperm<<<blocks_for(L.n), kBlock, 0, s>>>(L.n, L.perm.get(), L.iperm.get());
        GLK_CHECK_LAUNCH();
        L.dg64.alloc(L.n);
        L.dg32.alloc(L.n);
    }
    for (int l = 0; l < pre->nlev; ++l) {
        Level &L = pre->L[l];
        const bool generic = l >= lfirst;
        const int *rowp = generic ? L.perm.get() : nullptr;
        const int *colp = generic ? L.iperm.get() : nullptr;
        if (generic) {
            permuted_copy(L.A, rowp, colp, L.Aa, L.amap, T, s, true);
            L.dpos.alloc(L.n);
            k_diag_place<<<blocks_for(L.n), kBlock, 0, s>>>(L.n, L.Aa.rp.get(), L.Aa.ci.get(), L.dpos.get());
            GLK_CHECK_LAUNCH();
        }
        if (l + 1 < pre->nlev) {
            Level &Nx = pre->L[l + 1];
            permuted_copy(L.P, rowp, Nx.iperm.get(), L.Pa, L.pmap, T, s);
            permuted_copy(L.R, Nx.perm.get(), colp, L.Ra, L.rmap, T, s);
            if (l == 0 && !generic) {
                const GeomT<double> g = geom_t<double>(pre->mesh->g);
                Csr &B = L.Rb;
                B.n = L.Ra.n;
                B.m = 2 * g.npair;
                int *cnt = need(T, T.a, std::max(1, B.n));
                k_black_count<<<blocks_for(B.n), kBlock, 0, s>>>(B.n, g, L.Ra.rp.get(), L.Ra.ci.get(), cnt);
                GLK_CHECK_LAUNCH();
                alloc_rowptr(B, cnt, T, s);
                L.bmap.alloc(std::max(1, B.nnz));
                k_black_fill<<<blocks_for(B.n), kBlock, 0, s>>>(B.n, g, L.Ra.rp.get(), L.Ra.ci.get(), L.rmap.get(),
                                                                B.rp.get(), B.ci.get(), L.bmap.get());
                GLK_CHECK_LAUNCH();
                B.v64.alloc(std::max(1, B.nnz));
                B.v32.alloc(std::max(1, B.nnz));
                Csr &Q = L.Pb;
                Q.n = g.npair;
                Q.m = L.Pa.m;
                int *qcnt = need(T, T.a, std::max(1, Q.n));
                k_pblack_count<<<blocks_for(Q.n), kBlock, 0, s>>>(g, L.Pa.rp.get(), qcnt);
                GLK_CHECK_LAUNCH();
                alloc_rowptr(Q, qcnt, T, s);
                L.pbmap.alloc(std::max(1, Q.nnz));
                k_pblack_fill<<<blocks_for(Q.n), kBlock, 0, s>>>(g, L.Pa.rp.get(), L.Pa.ci.get(), L.pmap.get(),
                                                                 Q.rp.get(), Q.ci.get(), L.pbmap.get());
                GLK_CHECK_LAUNCH();
                Q.v64.alloc(std::max(1, Q.nnz));
                Q.v32.alloc(std::max(1, Q.nnz));
            }
        }
        if (generic) {
            // padded colour blocks for the Gauss-Seidel sweeps
            int *row0 = need(T, T.a, (size_t)L.ncolors + 1), *wid = need(T, T.b, 3 * (size_t)L.ncolors);
            to_device(row0, L.coff, s);
            k_row_widths<<<L.ncolors, kBlock, 0, s>>>(L.Aa.rp.get(), L.dpos.get(), row0, wid);
            GLK_CHECK_LAUNCH();
            L.ewidth = to_host(wid, 3 * (size_t)L.ncolors, s);
            L.elow.assign(L.ewidth.begin() + L.ncolors, L.ewidth.begin() + 2 * L.ncolors);
            L.eup.assign(L.ewidth.begin() + 2 * L.ncolors, L.ewidth.end());
            L.ewidth.resize(L.ncolors);
            L.eoff.assign(L.ncolors + 1, 0);
            for (int c = 0; c < L.ncolors; ++c) L.eoff[c + 1] = L.eoff[c] + L.ewidth[c] * (L.coff[c + 1] - L.coff[c]);
            const int ne = std::max(1, L.eoff[L.ncolors]);
            L.eci.alloc(ne);
            L.emap.alloc(ne);
            L.ev64.alloc(ne);
            L.ev32.alloc(ne);
            for (int c = 0; c < L.ncolors; ++c) {
                const int cnt = L.coff[c + 1] - L.coff[c];
                if (cnt == 0) continue;
                k_ell_fill<<<blocks_for(cnt), kBlock, 0, s>>>(L.coff[c], cnt, L.ewidth[c], L.Aa.rp.get(),
                                                             L.Aa.ci.get(), L.eci.get() + L.eoff[c],
                                                             L.emap.get() + L.eoff[c]);
                GLK_CHECK_LAUNCH();
            }
            if (l + 1 < pre->nlev) build_patches(pre, l, T, s);
        }
    }
    GLK_HIP(hipStreamSynchronize(s));
}

// Patches of level l (its colour-ordered copy Aa exists): tiles of about
// `own` rows by the rows' places in the plane.  A level keeps its dispatch per
// colour pass where patches do not pay or do not fit: rows of more than
// kPatchWidth neighbours (the 3D hierarchies: 30 entries and 15-30 colours reach
// over the whole level), a patch of more than 1024 rows, or more than kPatchMost
// updated rows per row of the level.  On every level measured that fits there are
// fewer (3-5 with 96 rows of a patch's own, 2.6-2.7 with 256-380; a disc whose rings
// crowd, 5 419 rows, 4.8), and up to there patches win (us per iteration with levels
// of more than 3 in passes / in patches: disc of 49 537 nodes 121 / 79, 1025^2 341 /
// 258), so the bound keeps only unmeasured levels out.  kPatchLevel is where they stop
// winning (us per iteration, passes / patches: level 1 of 394 113 rows FP64 547 / 509,
// FP32 418 / 386, of 700 587 rows 976 / 957 and 766 / 748, of 1 094 000 rows 1188 /
// 1212 and 897 / 888).
constexpr double kPatchMost = 8.0;
constexpr int kPatchLevel = 1 << 20;  // rows of a level in patches at most
constexpr int kPatchLarge = 65536;    // rows from which a level takes the largest patches that fit

static void build_patches(gl_precond *pre, int l, SymTmp &T, hipStream_t s)
{
    Level &L = pre->L[l];
    const gl_mesh *m = pre->mesh;
    const int n = L.n, nb = blocks_for(n);
    int wmax = 0;
    for (int w : L.ewidth) wmax = std::max(wmax, w - 1);
    if (n > kPatchLevel || m->g.dim != 2 || wmax > kPatchWidth || L.ncolors < 2 || L.ncolors > kMaxColors) return;
    PatchSet &S = L.patch;
    TileGrid t{};
    t.simplicial = m->g.simplicial;
    double ext[2];
    if (t.simplicial) {
        t.x = m->s_x.get();
        for (int a = 0; a < 2; ++a) {
            t.lo[a] = m->s_lo[a];
            ext[a] = m->s_hi[a] - m->s_lo[a];
            t.inv[a] = ext[a] > 0.0 ? 1.0 / ext[a] : 0.0;
        }
    } else {
        t.N0 = m->g.N[0];
        t.N1 = m->g.N[1];
        ext[0] = t.N0;
        ext[1] = t.N1;
    }
    // (rows of a patch, of these its own): smaller patches where 512 rows do not
    // hold a patch's reach, then 1024 rows (513^2 FP64, its level of 4 923 rows:
    // 169 us per MINRES iteration with 64 rows of 512, 175 with 112 of 1024;
    // 769^2 FP32, its level of 1 121 rows: 288 without patches, 238 with 1024).
    // A level that fills the chip several times over is bound by the rows that
    // patches share, so it starts from the largest (us per iteration with 96
    // rows of 512, then the first of these that fits: 1025^2 FP32, 175 446
    // rows, 253 and 225; 769^2 FP64, 98 000 rows, 216 and 186; 601^2, below
    // the line, 147 either way; 513^2, 44 075 rows, 143 and 141)
    const int tries[8][2] = {{1024, 380}, {1024, 340}, {1024, 300}, {1024, 256},
                             {512, 96}, {512, 64}, {1024, 112}, {1024, 64}};
    const Arena::Mark before = pre->arena.mark();
    const auto drop = [&] {  // (a try's kernels are done when its outcome has been read)
        S = PatchSet();
        pre->arena.rewind(before);
    };
    for (int k = n >= kPatchLarge ? 0 : 4; k < 8; ++k) {
        const int NR = tries[k][0], own = tries[k][1];
        S.rows = NR;
        S.W = wmax <= 8 ? 8 : wmax <= 12 ? 12 : wmax <= 16 ? 16 : 24;
        const double tiles = std::max(1.0, (double)n / own);
        t.k[0] = (int)std::max(1.0, std::min(tiles, std::round(std::sqrt(tiles * ext[0] / std::max(ext[1], 1e-300)))));
        t.k[1] = std::max(1, (int)std::round(tiles / t.k[0]));
        const int nt = t.k[0] * t.k[1];
        int *tile = need(T, T.a, n), *cnt = need(T, T.b, nt), *trp = need(T, T.c, (size_t)nt + 1);
        int *rows = need(T, T.d, n), *srt = need(T, T.e, 2 * (size_t)n), *err = need(T, T.err, 1);
        int *range = need(T, T.f, 3);
        k_fill_int<<<1, 64, 0, s>>>(err, 1, 0);
        k_fill_int<<<blocks_for(nt), kBlock, 0, s>>>(cnt, nt, 0);
        k_tile_of<<<nb, kBlock, 0, s>>>(n, L.perm.get(), L.origin.get(), t, tile);
        k_col_count<<<nb, kBlock, 0, s>>>(n, tile, cnt);
        GLK_CHECK_LAUNCH();
        scan_tiles(cnt, trp, nt, need(T, T.scan, 4 * ((size_t)nt / kScanTile + 4) + 64), s);
        // tiles are equal parts of the plane: on a graded mesh one may hold most of
        // the level, which no patch can (and whose rows would be sorted by one wave,
        // at a cost that grows with their square)
        k_fill_int<<<1, 64, 0, s>>>(range, 1, 0);
        k_fill_int<<<1, 64, 0, s>>>(range + 1, 1, nt);
        k_row_widths<<<1, kBlock, 0, s>>>(trp, nullptr, range, range + 2);
        GLK_CHECK_LAUNCH();
        if (read_int(range + 2, s) > NR) continue;
        k_fill_int<<<blocks_for(nt), kBlock, 0, s>>>(cnt, nt, 0);
        k_tile_fill<<<nb, kBlock, 0, s>>>(n, tile, trp, cnt, rows);
        k_sort_rows<<<(nt + kRowWaves - 1) / kRowWaves, kBlock, 0, s>>>(nt, trp, rows, rows, srt, srt + n);
        S.size.alloc(2 * (size_t)nt + 1);
        S.rowid.alloc((size_t)nt * 2 * NR);
        S.info.alloc((size_t)nt * NR);
        S.idx.alloc((size_t)nt * S.W * NR);
        S.map.alloc((size_t)nt * S.W * NR);
        int *total = S.size.get() + 2 * (size_t)nt;
        k_fill_int<<<1, 64, 0, s>>>(total, 1, 0);
        auto build = [&](auto kern) {
            kern<<<nt, S.rows, 0, s>>>(trp, srt, L.Aa.rp.get(), L.Aa.ci.get(), L.perm.get(), L.color.get(), L.ncolors,
                                       S.W, S.size.get(), S.rowid.get(), S.info.get(), S.idx.get(), S.map.get(), total,
                                       err);
        };
        if (NR == 512) build(k_patch_build<512>);
        else build(k_patch_build<1024>);
        GLK_CHECK_LAUNCH();
        const bool fits = read_int(err, s) == 0;
        if (fits && read_int(total, s) <= kPatchMost * n) {
            S.np = nt;
            S.v64.alloc((size_t)nt * S.W * NR);
            S.v32.alloc((size_t)nt * S.W * NR);
            int *row0 = need(T, T.a, 2), *wid = need(T, T.b, 1);
            to_device(row0, std::vector<int>{0, n}, s);
            k_row_widths<<<1, kBlock, 0, s>>>(L.Pa.rp.get(), nullptr, row0, wid);
            GLK_CHECK_LAUNCH();
            S.PW = read_int(wid, s);
            const size_t np = (size_t)n * S.PW;
            S.pci.alloc(np);
            S.pmap.alloc(np);
            S.pv64.alloc(np);
            S.pv32.alloc(np);
            k_pell_fill<<<nb, kBlock, 0, s>>>(n, S.PW, L.Pa.rp.get(), L.Pa.ci.get(), S.pci.get(), S.pmap.get());
            GLK_CHECK_LAUNCH();
            return;
        }
        drop();
        if (fits) break;
    }
}

void precond_symbolic(gl_precond *pre, hipStream_t s)
{
    const gl_mesh *m = pre->mesh;
    const int n0 = m->g.n, nb0 = blocks_for(n0);
    Level &L0 = pre->L[0];
    L0.n = n0;
    L0.A.n = L0.A.m = n0;
    SymTmp T;
    T.arena.spare = pre->arena.spare;
    {
        int *cnt = need(T, T.a, n0);
        if (m->g.simplicial) k_l0s_count<<<nb0, kBlock, 0, s>>>(n0, m->g.rp, cnt);
        else if (m->g.dim == 2) k_l0_count<2><<<nb0, kBlock, 0, s>>>(m->g, cnt);
        else k_l0_count<3><<<nb0, kBlock, 0, s>>>(m->g, cnt);
        GLK_CHECK_LAUNCH();
        alloc_rowptr(L0.A, cnt, T, s);
        if (m->g.simplicial)
            k_l0s_cols<<<nb0, kBlock, 0, s>>>(n0, m->g.rp, m->g.ci, L0.A.rp.get(), L0.A.ci.get());
        else if (m->g.dim == 2) k_l0_cols<2><<<nb0, kBlock, 0, s>>>(m->g, L0.A.rp.get(), L0.A.ci.get());
        else k_l0_cols<3><<<nb0, kBlock, 0, s>>>(m->g, L0.A.rp.get(), L0.A.ci.get());
        GLK_CHECK_LAUNCH();
    }
    const int max_levels = std::min(pre->opts.max_levels, kMaxLevels);
    int l = 0;
    for (;;) {
        colour_level(pre, l, T, s);
        Level &L = pre->L[l];
        if (L.n <= pre->opts.max_coarse || l == max_levels - 1) break;
        const int nc = aggregate_level(pre, l, T, s);
        if ((double)nc > 0.85 * (double)L.n) {
            L.agg.release();
            L.root.release();
            L.aggsize.release();
            L.nc = 0;
            break;
        }
        transfer_patterns(pre, l, T, s);
        ++l;
    }
    pre->nlev = l + 1;
    if (pre->L[l].n > kMaxDense)
        fail(GL_ERR_UNSUPPORTED, "coarsest level too large for the dense solve");
    alloc_values(pre);
    build_apply_copies(pre, T, s);
    bottom_descriptors(pre, s);
    GLK_HIP(hipStreamSynchronize(s));
}

// The patches' copies of the matrix values, for the levels above the bottom
// kernel and the dense operator.
void patch_values_enqueue(gl_precond *pre, const Launch &L)
{
    for (int l = 0; l < std::max(pre->bottom, pre->stail); ++l) {
        Level &lv = pre->L[l];
        if (lv.patch.np == 0) continue;
        const int ne = lv.patch.np * lv.patch.W * lv.patch.rows;
        L.run(blocks_for(ne), EllValues{ne, lv.patch.map.get(), lv.Aa.v64.get(), lv.patch.v64.get(), lv.patch.v32.get()});
        const int nq = lv.n * lv.patch.PW;
        L.run(blocks_for(nq), EllValues{nq, lv.patch.pmap.get(), lv.Pa.v64.get(), lv.patch.pv64.get(), lv.patch.pv32.get()});
    }
}

void precond_numeric_enqueue(gl_precond *pre, const double2 *psi, const Launch &L)
{
    const gl_mesh *m = pre->mesh;
    Level &L0 = pre->L[0];
    const int n0 = L0.n;
    const GeomT<double> g = geom_t<double>(m->g);
    const bool simp = m->g.simplicial;
    pre->stail_current = false;
    if (simp)
        L.run(blocks_for(n0), L0sValues{g, L0.A.rp.get(), L0.A.ci.get(), psi, L0.A.v64.get(), L0.diag64.get()});
    else if (m->g.dim == 2)
        L.run(blocks_for(n0), L0Values<2>{g, L0.A.rp.get(), link_tab<double>(m), psi, L0.A.v64.get(), L0.diag64.get()});
    else
        L.run(blocks_for(n0), L0Values<3>{g, L0.A.rp.get(), link_tab<double>(m), psi, L0.A.v64.get(), L0.diag64.get()});
    for (int l = 0; l + 1 < pre->nlev; ++l) {
        Level &lv = pre->L[l];
        Level &Nx = pre->L[l + 1];
        const int n = lv.n, nb = blocks_for(n);
        if (l > 0) L.run(nb, Diag{n, lv.A.rp.get(), lv.A.ci.get(), lv.A.v64.get(), lv.diag64.get()});
        rho_estimate(pre, lv, L);
        L.run(blocks_for((int64_t)n * kPLanes),
              PValues{n, lv.A.rp.get(), lv.A.ci.get(), lv.A.v64.get(), lv.diag64.get(), lv.agg.get(), lv.aggsize.get(),
                      lv.rho.get(), lv.P.rp.get(), lv.P.ci.get(), lv.P.v64.get()});
        L.run(blocks_for(lv.R.nnz), RValues{lv.R.nnz, lv.rsrc.get(), lv.P.v64.get(), lv.R.v64.get()});
        // A P: eight lanes a row on the finest levels in 2D (five-point and triangle
        // rows, at most 5 entries of A P), 16 on denser ones.  us by 4 / 8 / 16 lanes:
        // level 0 of 1025^2 122 / 90 / 134, of a disc of 49 537 nodes 11.5 / 7.5 / 11;
        // level 0 of 129^3 657 / 448 / 378, of a tetrahedron of 12 001 nodes 54 / 21 /
        // 10; levels 1 of 1025^2 54 / 38 / 32, of 129^3 1006 / 425 / 305.
        auto ap = [&](auto lanes) {
            constexpr int LPR = decltype(lanes)::value;
            L.run(blocks_for((int64_t)n * LPR),
                  ApValues<LPR>{n, lv.A.rp.get(), lv.A.ci.get(), lv.A.v64.get(), lv.P.rp.get(), lv.P.ci.get(),
                                lv.P.v64.get(), lv.AP.rp.get(), lv.AP.ci.get(), lv.AP.v64.get()});
        };
        if (lv.AP.nnz <= 5 * (int64_t)n) ap(std::integral_constant<int, 8>{});
        else ap(std::integral_constant<int, 16>{});
        L.run(blocks_for((int64_t)Nx.A.nnz * kRapLanes),
              RapValues{Nx.A.nnz, lv.rap_tp.get(), lv.rap_pair.get(), lv.rap_mir.get(), lv.R.v64.get(), lv.AP.v64.get(),
                        Nx.A.v64.get()});
    }
    const int last = pre->nlev - 1;
    Level &Lc = pre->L[last];
    if (last > 0) L.run(blocks_for(Lc.n), Diag{Lc.n, Lc.A.rp.get(), Lc.A.ci.get(), Lc.A.v64.get(), Lc.diag64.get()});
    // level 0 in single precision (its stencil diagonal; the CSR copy serves export only)
    L.run(blocks_for(n0), ToF32r{n0, L0.diag64.get(), L0.diag32.get()});
    if (!simp) L.run(blocks_for(g.npair), SplitDiag{g, L0.diag64.get(), L0.hs64.get(), L0.hs32.get()});
    // colour-ordered copies for the V-cycle, FP64 and rounded to FP32
    for (int l = 0; l < pre->nlev; ++l) {
        Level &lv = pre->L[l];
        if (l >= 1 || (simp && last > 0)) {
            L.run(blocks_for(lv.Aa.nnz), GatherC{lv.Aa.nnz, lv.amap.get(), lv.A.v64.get(), lv.Aa.v64.get(), lv.Aa.v32.get()});
            L.run(blocks_for(lv.n), GatherR{lv.n, lv.perm.get(), lv.diag64.get(), lv.dg64.get(), lv.dg32.get()});
            const int ne = lv.eoff.empty() ? 0 : lv.eoff.back();
            if (ne > 0) L.run(blocks_for(ne), EllValues{ne, lv.emap.get(), lv.Aa.v64.get(), lv.ev64.get(), lv.ev32.get()});
        }
        if (l < last) {
            L.run(blocks_for(lv.Pa.nnz), GatherC{lv.Pa.nnz, lv.pmap.get(), lv.P.v64.get(), lv.Pa.v64.get(), lv.Pa.v32.get()});
            L.run(blocks_for(lv.Ra.nnz), GatherC{lv.Ra.nnz, lv.rmap.get(), lv.R.v64.get(), lv.Ra.v64.get(), lv.Ra.v32.get()});
            if (l == 0 && !simp) {
                L.run(blocks_for(lv.Rb.nnz),
                      GatherC{lv.Rb.nnz, lv.bmap.get(), lv.R.v64.get(), lv.Rb.v64.get(), lv.Rb.v32.get()});
                L.run(blocks_for(lv.Pb.nnz),
                      GatherC{lv.Pb.nnz, lv.pbmap.get(), lv.P.v64.get(), lv.Pb.v64.get(), lv.Pb.v32.get()});
            }
        }
    }
    patch_values_enqueue(pre, L);
    // coarsest: Cholesky in FP64 (positive definiteness check), then the inverse
    // in the V-cycle's row order, applied as a dense product
    const Csr &Mc = last > 0 ? Lc.Aa : Lc.A;
    L.run(blocks_for(Lc.n), DenseFromCsr{Lc.n, Mc.rp.get(), Mc.ci.get(), Mc.v64.get(), pre->cfac.get()});
    cholesky(Lc.n, pre->cfac.get(), pre->cdmax.get(), pre->status.get(), L);
    L.run(Lc.n, CholInverse{Lc.n, pre->cfac.get(), pre->cinv64.get(), pre->status.get()});
    L.run(blocks_for((int64_t)Lc.n * Lc.n), ToF32c{Lc.n * Lc.n, pre->cinv64.get(), pre->cinv32.get()});
}

void precond_numeric_finish(gl_precond *pre, bool singular, hipStream_t s)
{
    if (singular) fail(GL_ERR_SINGULAR, "gl_precond_setup: coarsest operator is not positive definite");
    pre->has_values = true;
    form_tail(pre, s);
    if (pre->opts.cycles == 0) pcg_calibrate(pre, s);
}

void precond_numeric(gl_precond *pre, const double2 *psi, hipStream_t s)
{
    precond_numeric_enqueue(pre, psi, Launch{s});
    precond_numeric_finish(pre, read_int(pre->status.get(), s) != 0, s);
}

}  // namespace glk

using namespace glk;

namespace glk {
void check_amg_opts(const gl_amg_opts *opts, const char *who)
{
    const std::string w(who);
    if (opts->precision != GL_FP64 && opts->precision != GL_FP32 && opts->precision != GL_MIXED)
        fail(GL_ERR_INVALID_ARGUMENT, w + ": precision");
    if (opts->cycles < 0 || opts->cycles > 1000) fail(GL_ERR_INVALID_ARGUMENT, w + ": cycles must be in 0..1000");
    if (opts->cycles == 0 && opts->precision != GL_FP64)
        fail(GL_ERR_INVALID_ARGUMENT, w + ": R_inf (cycles 0) needs the FP64 V-cycle");
    if (opts->max_coarse < 1 || opts->max_coarse > kMaxDense)
        fail(GL_ERR_INVALID_ARGUMENT, w + ": max_coarse must be in 1..2048");
    if (opts->max_levels < 1 || opts->max_levels > kMaxLevels)
        fail(GL_ERR_INVALID_ARGUMENT, w + ": max_levels must be in 1..16");
}

gl_precond *precond_new(const gl_mesh *mesh, const double2 *psi, const gl_amg_opts &opts,
                        const std::shared_ptr<SpareChunks> &spare, hipStream_t s)
{
    std::unique_ptr<gl_precond> pre(new gl_precond());
    pre->uid = new_precond_uid();
    pre->mesh = mesh;
    pre->opts = opts;
    pre->arena.spare = spare;
    {
        const ArenaScope small(&pre->arena);
        precond_symbolic(pre.get(), s);
    }
    precond_numeric(pre.get(), psi, s);
    return pre.release();
}

uint64_t new_precond_uid()
{
    static std::atomic<uint64_t> next{1};
    return next++;
}
}  // namespace glk

extern "C" {

gl_status gl_precond_setup(const gl_mesh *mesh, const void *psi, const gl_amg_opts *opts,
                           gl_precond **inout, gl_stream stream)
{
    return guarded([&] {
        if (!mesh || !psi || !inout) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_setup: NULL argument");
        hipStream_t s = as_stream(stream);
        gl_precond *pre = *inout;
        if (pre && pre->mesh != mesh)
            fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_setup: handle belongs to another mesh");
        if (!pre && !opts) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_setup: opts required for a new handle");
        if (opts) check_amg_opts(opts, "gl_precond_setup");
        if (!pre) {
            *inout = precond_new(mesh, (const double2 *)psi, *opts, mesh->spare, s);
        } else {
            if (opts) {
                if (opts->max_coarse != pre->opts.max_coarse || opts->max_levels != pre->opts.max_levels)
                    fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_setup: hierarchy limits differ from the handle's");
                pre->opts.precision = opts->precision;
                pre->opts.cycles = opts->cycles;
            }
            precond_numeric(pre, (const double2 *)psi, s);
        }
    });
}

gl_status gl_precond_inner_steps(const gl_precond *pre, int *steps)
{
    return guarded([&] {
        if (!pre || !steps) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_inner_steps: NULL argument");
        *steps = pre->opts.cycles == 0 ? pre->pcg_m : pre->opts.cycles;
    });
}

gl_status gl_precond_info(const gl_precond *pre, int *nlev, int64_t *sizes, int64_t *nnz, int *ncolors)
{
    return guarded([&] {
        if (!pre) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_info: NULL handle");
        if (nlev) *nlev = pre->nlev;
        for (int l = 0; l < pre->nlev; ++l) {
            if (sizes) sizes[l] = pre->L[l].n;
            if (nnz) nnz[l] = pre->L[l].A.nnz;
            if (ncolors) ncolors[l] = pre->L[l].ncolors;
        }
    });
}

gl_status gl_precond_export(const gl_precond *pre, int level, int what, void *host_buf, size_t *bytes)
{
    return guarded([&] {
        if (!pre || !bytes) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_export: NULL argument");
        if (level < 0 || level >= pre->nlev) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_export: level");
        const Level &L = pre->L[level];
        const bool last = level == pre->nlev - 1;
        if (last && ((what >= 6 && what <= 11) || what == 0 || what == 1))
            fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_export: the coarsest level has no transfer operators");
        const void *src = nullptr;
        size_t need = 0;
        switch (what) {
        case 0: src = L.agg.get(); need = sizeof(int) * L.n; break;
        case 1: src = L.root.get(); need = sizeof(int) * L.nc; break;
        case 2: src = L.color.get(); need = sizeof(int) * L.n; break;
        case 3: src = L.A.rp.get(); need = sizeof(int) * (L.n + 1); break;
        case 4: src = L.A.ci.get(); need = sizeof(int) * L.A.nnz; break;
        case 5: src = L.A.v64.get(); need = sizeof(double2) * L.A.nnz; break;
        case 6: src = L.P.rp.get(); need = sizeof(int) * (L.n + 1); break;
        case 7: src = L.P.ci.get(); need = sizeof(int) * L.P.nnz; break;
        case 8: src = L.P.v64.get(); need = sizeof(double2) * L.P.nnz; break;
        case 9: src = L.R.rp.get(); need = sizeof(int) * (L.nc + 1); break;
        case 10: src = L.R.ci.get(); need = sizeof(int) * L.R.nnz; break;
        case 11: src = L.R.v64.get(); need = sizeof(double2) * L.R.nnz; break;
        default: fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_export: unknown array");
        }
        if (!host_buf) { *bytes = need; return; }
        if (*bytes < need) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_export: buffer too small");
        *bytes = need;
        GLK_HIP(hipDeviceSynchronize());
        if (need) GLK_HIP(hipMemcpy(host_buf, src, need, hipMemcpyDeviceToHost));
    });
}

gl_status gl_precond_set_tiles(gl_precond *pre, const gl_tiles *tiles)
{
    return guarded([&] {
        if (!pre || !tiles) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_set_tiles: NULL argument");
        if (tiles->lane_shift < -2 || tiles->lane_shift > 2 || tiles->bottom_rows < 0 || tiles->bottom_rows > 65536 ||
            tiles->dense_rows < 0 || tiles->dense_rows > kMaxTail || tiles->l0_tiled < 0 || tiles->l0_tiled > 3)
            fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_set_tiles: lane_shift in -2..2, bottom_rows in 0..65536, "
                                          "dense_rows in 0..8192, l0_tiled 0..3");
        // (the request alone decides, not what was set before it)
        const bool automatic = !tiles->lane_shift && !tiles->bottom_rows && !tiles->dense_rows && !tiles->l0_tiled;
        const int rows = tiles->bottom_rows ? tiles->bottom_rows : kBottomRows;
        if (automatic == pre->auto_tiles && rows == pre->bottom_rows && tiles->lane_shift == pre->lane_shift &&
            tiles->dense_rows == pre->dense_rows && tiles->l0_tiled == pre->l0_tiled)
            return;
        pre->bottom_rows = rows;
        pre->lane_shift = tiles->lane_shift;
        pre->dense_rows = tiles->dense_rows;
        pre->l0_tiled = tiles->l0_tiled;
        pre->auto_tiles = automatic;
        pre->uid = new_precond_uid();  // captured graphs of the old shape are stale
        hipStream_t s = pre->mesh->ws;
        GLK_HIP(hipStreamSynchronize(s));  // no pending use of the buffers re-made here
        bottom_descriptors(pre, s);
        if (pre->has_values) patch_values_enqueue(pre, Launch{s});  // levels that were below the split
        form_tail(pre, s);
        GLK_HIP(hipStreamSynchronize(s));
    });
}

gl_status gl_precond_get_tiles(const gl_precond *pre, gl_tiles *tiles)
{
    return guarded([&] {
        if (!pre || !tiles) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_get_tiles: NULL argument");
        tiles->lane_shift = pre->lane_shift;
        tiles->bottom_rows = pre->auto_tiles ? 0 : pre->bottom_rows;
        tiles->dense_rows = pre->dense_rows;
        tiles->l0_tiled = pre->l0_tiled;
    });
}

void gl_precond_destroy(gl_precond *pre) { delete pre; }

}  // extern "C"
