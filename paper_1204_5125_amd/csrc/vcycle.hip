// Application of the preconditioner R_k = AMG_k(H, D .) (eq. prec2): k
// V-cycles from zero on H x = v with one symmetric Gauss-Seidel sweep before
// and after the coarse correction (Sec. 4.1).  A symmetric sweep visits the
// colours 0 .. C-1 and then C-2 .. 0; on level 0 (red-black, red = even index
// sum) that is red, black, red.  Every kernel is templated on the storage and
// arithmetic type (double or float); the input v and the output z are FP64.
//
// Level 0 needs six stencil passes instead of seven because a Gauss-Seidel
// update of a red node does not read the node's previous value:
//   - the first red update from x = 0 is x_r = b_r / H_rr, folded into the
//     black update that follows (which evaluates it for its red neighbours);
//   - after the pre-smoothing sweep the red residual is zero (the last update
//     made it so), and only black residuals are formed;
//   - after the coarse correction only the black values x_b + (P x_c)_b are
//     read (by the first red update), so only black nodes are prolonged.
// In 2D these passes run on tiles in LDS, two kernels a cycle (L0PreTile,
// L0PostTile).  The coarser levels run a whole symmetric sweep per dispatch on
// patches of rows (PatchPre, PatchPost) where the patches fit, and a dispatch per
// colour and half a sweep (SgsPass) where they do not.  Below the first level with at most dense_rows rows (a tile choice), or that
// solver_tail picks for solves, the cycle is a fixed linear map of that level's
// right-hand side; it is formed as a dense matrix and applied as one product, like
// the coarsest inverse.
#include <cstring>
#include <type_traits>

#include "amg.h"
#include "stencil.h"

namespace glk {

#define GATE()                               \
    if (gate && *gate == 0) return

// The gate flag read together with a kernel's data and checked right before
// its stores, so that its load overlaps the others instead of delaying them;
// the flag is uniform, so every thread takes the same branch.
#define GATE_LOAD() const bool gate_go = gate == nullptr || *gate != 0

// a seeded right-hand side in [-1, 1]^2 per node (MurmurHash3 finaliser of
// the node index), for calibrating R_inf
__global__ void k_hash_rhs(int n, double2 *v)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    auto mix = [](uint32_t h) {
        h ^= h >> 16;
        h *= 0x85ebca6bu;
        h ^= h >> 13;
        h *= 0xc2b2ae35u;
        h ^= h >> 16;
        return h;
    };
    const uint32_t a = mix(2u * (uint32_t)i + 0x9e3779b9u), b = mix(2u * (uint32_t)i + 1u + 0x9e3779b9u);
    v[i] = make_double2(a * (2.0 / 4294967295.0) - 1.0, b * (2.0 / 4294967295.0) - 1.0);
}

// Level-0 colour passes run one thread per red-black pair: thread t owns the
// nodes c0 = 2k and 2k + 1 of x-row `row` (k = t mod hr, row = t / hr), one
// of each colour, so every thread updates a node (a thread per node would
// leave half of them idle and need twice the waves).
struct Pair {
    int ie;      // index of the even node (c0 = 2k)
    int c[3];    // its coordinates
    bool odd;    // the odd node c0 = 2k + 1 exists
};

template <int DIM, class T>
__device__ __forceinline__ Pair pair_at(const GeomT<T> &g, int t)
{
    Pair P;
    const int row = t / g.hr, k = t - row * g.hr;
    P.c[0] = 2 * k;
    P.c[1] = DIM == 3 ? row % g.N[1] : row;
    P.c[2] = DIM == 3 ? row / g.N[1] : 0;
    P.ie = 2 * k + g.N[0] * row;
    P.odd = 2 * k + 1 < g.N[0];
    return P;
}

// the pair's node of colour col: offset s from the even node (false: absent)
__device__ __forceinline__ bool pair_colour(const Pair &P, int col, int &s)
{
    s = (col + P.c[1] + P.c[2]) & 1;
    return s == 0 || P.odd;
}

// The V-cycle's level-0 vectors (b, x, r) and the diagonal it divides by are
// stored split by colour: the node of colour col in pair t sits at
// col * npair + t.  A colour pass then reads and writes one contiguous half,
// and the neighbours of a node, all of the other colour, sit in the other
// half at pairs t +- 1 (x), t +- hr (y) and t +- hr N1 (z).  The sum below
// takes the terms in the order of khat_offdiag, so the results do not change.
template <int DIM, class T>
__device__ __forceinline__ C<T> khat_offdiag_rb(const GeomT<T> &g, const int c[3], int t,
                                                const C<T> *__restrict__ xo, const LinkTab<T> &U)
{
    T s[3];
    const T d = node_volume<DIM, T>(g, c, s);
    C<T> acc = mk<T>(0, 0);
    const int row0 = t - (c[0] >> 1);  // first pair of the node's x-row
    int pstride = g.hr;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const T al = d * s[a] * g.inv_h2[a];
        int tl, tu;
        if (a == 0) {
            tl = row0 + ((c[0] - 1) >> 1);
            tu = row0 + ((c[0] + 1) >> 1);
        } else {
            tl = t - pstride;
            tu = t + pstride;
            pstride *= g.N[a];
        }
        if (c[a] > 0) acc = csub(acc, cscale(cmul(link_u<DIM, T>(U, a, c, c[a] - 1), xo[tl]), al));
        if (c[a] < g.N[a] - 1) acc = csub(acc, cscale(cmulc(link_u<DIM, T>(U, a, c, c[a]), xo[tu]), al));
    }
    return acc;
}

// pre-smoothing: b = round(v) into the split layout, and the black pass from
// zero (the red pass from zero, x_red = b / diag, folded in: it reads v and
// the natural-order diagonal hd at the red neighbours)
template <int DIM, class T>
struct L0PreBlack {
    GeomT<T> g;
    const double2 *v;
    C<T> *b, *x;
    LinkTab<T> U;
    const T *hd;
    const int *gate;
    __device__ void operator()(int bx, int nbx) const
    {
        GATE_LOAD();
        const int t = xcd_tile(bx, nbx) * kBlock + threadIdx.x;
        if (t >= g.npair) return;
        const Pair P = pair_at<DIM, T>(g, t);
        const int np = g.npair, ce = (P.c[1] + P.c[2]) & 1;  // colour of the even node
        const C<T> b0 = narrow<T>(v[P.ie]);
        const C<T> b1 = P.odd ? narrow<T>(v[P.ie + 1]) : mk<T>(0, 0);
        if (gate_go) {
            b[ce * np + t] = b0;
            if (P.odd) b[(1 - ce) * np + t] = b1;
        }
        int sb;
        if (!pair_colour(P, 1, sb)) return;
        const int i = P.ie + sb;
        const int c[3] = {P.c[0] + sb, P.c[1], P.c[2]};
        const C<T> bi = sb ? b1 : b0;
        T s[3];
        const T d = node_volume<DIM, T>(g, c, s);
        C<T> off = mk<T>(0, 0);
        int stride = 1;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            const T al = d * s[a] * g.inv_h2[a];
            if (c[a] > 0) {
                const int k = i - stride;
                const C<T> xk = cscale(narrow<T>(v[k]), (T)1 / hd[k]);
                off = csub(off, cscale(cmul(link_u<DIM, T>(U, a, c, c[a] - 1), xk), al));
            }
            if (c[a] < g.N[a] - 1) {
                const int k = i + stride;
                const C<T> xk = cscale(narrow<T>(v[k]), (T)1 / hd[k]);
                off = csub(off, cscale(cmulc(link_u<DIM, T>(U, a, c, c[a]), xk), al));
            }
            stride *= g.N[a];
        }
        const C<T> xi = cscale(csub(bi, off), (T)1 / hd[i]);
        if (!gate_go) return;
        x[np + t] = xi;
    }
};

// x_i = (b_i - sum_{j != i} H_ij x_j) / H_ii on one colour (split layout; hs:
// the diagonal in that layout)
template <int DIM, class T>
struct L0Sweep {
    GeomT<T> g;
    int colour;
    const C<T> *b;
    C<T> *x;
    LinkTab<T> U;
    const T *hs;
    const int *gate;
    __device__ void operator()(int bx, int nbx) const
    {
        GATE_LOAD();
        const int t = xcd_tile(bx, nbx) * kBlock + threadIdx.x;
        if (t >= g.npair) return;
        const Pair P = pair_at<DIM, T>(g, t);
        int sc;
        if (!pair_colour(P, colour, sc)) return;
        const int c[3] = {P.c[0] + sc, P.c[1], P.c[2]};
        const int q = colour * g.npair + t;
        const C<T> bi = b[q];
        const T di = hs[q];
        const C<T> off = khat_offdiag_rb<DIM, T>(g, c, t, x + (1 - colour) * g.npair, U);
        const C<T> xi = cscale(csub(bi, off), (T)1 / di);
        if (!gate_go) return;
        x[q] = xi;
    }
};

// r = b - H x on the black nodes (split layout); the red residual is zero and
// is neither stored nor read (the restriction has no red columns)
template <int DIM, class T>
struct L0Residual {
    GeomT<T> g;
    const C<T> *b, *x;
    LinkTab<T> U;
    const T *hs;
    C<T> *r;
    const int *gate;
    __device__ void operator()(int bx, int nbx) const
    {
        GATE_LOAD();
        const int t = xcd_tile(bx, nbx) * kBlock + threadIdx.x;
        if (t >= g.npair) return;
        const Pair P = pair_at<DIM, T>(g, t);
        int sb;
        if (!pair_colour(P, 1, sb)) return;
        const int c[3] = {P.c[0] + sb, P.c[1], P.c[2]};
        const int q = g.npair + t;
        const C<T> bi = b[q];
        const C<T> xi = x[q];
        const T di = hs[q];
        const C<T> off = khat_offdiag_rb<DIM, T>(g, c, t, x, U);
        const C<T> ri = csub(csub(bi, cscale(xi, di)), off);
        if (!gate_go) return;
        r[q] = ri;
    }
};

// r = v - H z on every node, FP64 (between cycles of R_k, k > 1)
template <int DIM>
struct L0ResidualFull {
    GeomT<double> g;
    const double2 *v, *z;
    LinkTab<double> U;
    const double *hd;
    double2 *r;
    const int *gate;
    __device__ void operator()(int bx, int nbx) const
    {
        GATE();
        const int i = xcd_tile(bx, nbx) * kBlock + threadIdx.x;
        if (i >= g.n) return;
        int c[3];
        node_coords<DIM>(g.N, i, c);
        const double2 off = khat_offdiag<DIM, double>(g, i, c, z, U);
        r[i] = csub(csub(v[i], cscale(z[i], hd[i])), off);
    }
};

// (P x_c)_k for one fine row
template <class T>
__device__ __forceinline__ C<T> prolong_row(const int *__restrict__ prp, const int *__restrict__ pci,
                                            const C<T> *__restrict__ pv, const C<T> *__restrict__ xc, int k)
{
    C<T> s = mk<T>(0, 0);
    for (int p = prp[k]; p < prp[k + 1]; ++p) s = cadd(s, cmul(pv[p], xc[pci[p]]));
    return s;
}

// coarse correction of the black nodes: x_b += (P x_c)_b (the red nodes are
// overwritten by the red pass that follows, which reads only black values);
// x in the split layout, P's black rows by pair (row t: the black node of
// pair t)
template <int DIM, class T, class TC = T>
struct L0ProlongBlack {
    GeomT<T> g;
    C<T> *x;
    const int *prp, *pci;
    const C<TC> *pv, *xc;
    const int *gate;
    __device__ void operator()(int bx, int nbx) const
    {
        GATE_LOAD();
        const int t = xcd_tile(bx, nbx) * kBlock + threadIdx.x;
        if (t >= g.npair) return;
        const Pair P = pair_at<DIM, T>(g, t);
        int sb;
        if (!pair_colour(P, 1, sb)) return;
        const int q = g.npair + t;
        const C<T> xo = x[q];
        const C<T> xi = cadd(xo, as_c<T>(prolong_row<TC>(prp, pci, pv, xc, t)));
        if (!gate_go) return;
        x[q] = xi;
    }
};

// last red pass; z = x (ADD: z += x) on every node and partial sums of Re<vdot, z>
template <int DIM, class T, int ADD>
struct L0Last {
    GeomT<T> g;
    const C<T> *b;
    C<T> *x;
    LinkTab<T> U;
    const T *hs;
    double2 *z;
    const double2 *vdot;
    RedSlot slot;
    int want_dot;
    DeflDot dd;
    const int *gate;
    __device__ void operator()(int bx, int nbx) const
    {
        GATE_LOAD();
        __shared__ double sm[kBlock / 64];
        const int t = xcd_tile(bx, nbx) * kBlock + threadIdx.x;
        const bool in = t < g.npair;
        const Pair P = pair_at<DIM, T>(g, in ? t : 0);
        // the red node's update, then z on both nodes (even first, natural
        // order); every load before the (uniform) gate check, every store
        // after it.  The red update goes to z only: the next cycle starts
        // from zero and writes every node before it reads it.
        int sr, sb;
        const bool red = in && pair_colour(P, 0, sr);
        const bool black = in && pair_colour(P, 1, sb);
        C<T> xr = mk<T>(0, 0);
        const C<T> xb = black ? x[g.npair + t] : mk<T>(0, 0);
        double2 zq[2] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
        double part = 0.0, part_u = 0.0;
        if (red) {
            const int c[3] = {P.c[0] + sr, P.c[1], P.c[2]};
            const C<T> bi = b[t];
            const T di = hs[t];
            const C<T> off = khat_offdiag_rb<DIM, T>(g, c, t, x + g.npair, U);
            xr = cscale(csub(bi, off), (T)1 / di);
        }
        if (in) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (q == 1 && !P.odd) break;
                const int i = P.ie + q;
                double2 zi = widen(red && q == sr ? xr : xb);
                if (ADD) zi = cadd(z[i], zi);
                zq[q] = zi;
                if (want_dot) part += redot(vdot[i], zi);
                if (dd.psi) {
                    const int c[3] = {P.c[0] + q, P.c[1], P.c[2]};
                    part_u += dd.term<DIM>(i, c, zi);
                }
            }
        }
        if (!gate_go) return;
        if (in) {
            z[P.ie] = zq[0];
            if (P.odd) z[P.ie + 1] = zq[1];
        }
        if (want_dot) block_reduce_store(part, slot, sm, bx);
        if (dd.psi) block_reduce_store(part_u, dd.slot, sm, bx);
    }
};

// ------------------------------------------- level 0 in LDS tiles (2D) ---
// The level-0 passes of a V-cycle fused into two kernels, each over a tile
// of S::TX x S::TY nodes held in LDS with a halo of three nodes: the three
// colour passes of a sweep need neighbours' values of the previous pass, so
// a pass is exact one node further inside than the one before, and three
// passes (or two and the residual) are exact on the tile itself.  Every node
// value is the same expression, in the same order, as in the
// one-pass-per-dispatch kernels above (red from zero folded, khat_offdiag
// order), so the cycle's output agrees with theirs to rounding (the compiler
// may contract multiply-adds differently in the two); the partial sums of
// Re<vdot, z> are grouped by tile.
// A thread has one red-black pair in registers (right-hand side, diagonal and its
// reciprocal, links, coefficients); LDS holds the iterate alone, by colour and
// pair, so a pass is three conflict-free LDS reads, the update and a barrier.
// The halo is three rows below and above and four columns left and right (pairs stay
// whole).  A link across the grid's edge is zero, so its term drops out without a
// branch.
// Tile shapes (gl_tiles.l0_tiled 1, 2, 3): smaller tiles keep more of them resident
// per CU at the price of a larger halo share.
// What bounds it: on large grids the traffic (up with both dot products 89 MB for
// 1025^2 in FP32 by the counters, 17 us at the rate of a copy) and the halo's share
// of the instructions; on small ones the chain row pointers - P's row - x_c, the
// passes and the launch.  Down / up, us per dispatch, against threads that looped
// over single nodes with every operand in LDS: 1025^2 FP32 18.5 / 33.1 (19.8 /
// 45.3), twelve grids of 129-513^2 FP64 13.0 / 21.4 (18 / 28), 33^2 FP64 4.5 /
// 7.8 (5.5 / 9.8).
template <int X, int Y>
struct L0Shape {
    static constexpr int TX = X, TY = Y, HX = 4, HY = 3, LX = X + 2 * HX, LY = Y + 2 * HY;
    static constexpr int PX = LX / 2, pairs = PX * LY, threads = (pairs + 63) / 64 * 64;
};
using L0Shape1 = L0Shape<32, 32>;
using L0Shape2 = L0Shape<32, 16>;
using L0Shape3 = L0Shape<16, 16>;

// a or b by value (a choice between lvalues is one between addresses, and puts
// both in memory)
template <class V>
__device__ __forceinline__ V l0_pick(bool which, V a, V b)
{
    return V{which ? a.x : b.x, which ? a.y : b.y};
}

// one node of a pair
template <class T>
struct L0Node {
    int gx, ring;  // ring: distance from the border of the tile's halo
    bool in, odd;  // in the grid; the pair's second node
    T a0, a1;      // edge coefficients alpha = |V| s_a / h_a^2 along x and y
    C<T> ul, ur, ud, uu;  // links of the edges to the lower and upper neighbours along x, y
    T d, w;        // diagonal, 1 / d
    C<T> b, x;

    // sum_{j != i} H_ij x_j; far: x of the neighbour in the next pair
    __device__ __forceinline__ C<T> offdiag(C<T> own, C<T> far, C<T> dn, C<T> up) const
    {
        const C<T> xl = l0_pick(odd, own, far), xr = l0_pick(odd, far, own);
        C<T> acc = mk<T>(0, 0);
        acc = csub(acc, cscale(cmul(ul, xl), a0));
        acc = csub(acc, cscale(cmulc(ur, xr), a0));
        acc = csub(acc, cscale(cmul(ud, dn), a1));
        acc = csub(acc, cscale(cmulc(uu, up), a1));
        return acc;
    }
};

template <class T, class S>
struct L0Pair {
    int p, t, gy;   // place in LDS; pair of the grid; row
    bool act, own;  // a pair of the tile with its halo; of the tile
    L0Node<T> n[2];  // red, black

    __device__ __forceinline__ L0Pair(const GeomT<T> &g, const LinkTab<T> &U, const T *hs, int tile, int ntx)
    {
        p = threadIdx.x;
        act = p < S::pairs;
        const int lp = p % S::PX, ly = p / S::PX;
        const int ge = (tile % ntx) * S::TX - S::HX + 2 * lp;  // the pair's even node
        gy = (tile / ntx) * S::TY - S::HY + ly;
        own = act && lp >= S::HX / 2 && lp < (S::HX + S::TX) / 2 && ly >= S::HY && ly < S::HY + S::TY;
        const int nx = g.N[0], ny = g.N[1];
        const bool row = act && gy >= 0 && gy < ny;
        t = row && ge >= 0 && ge < nx ? (ge >> 1) + g.hr * gy : 0;
        // links of the pair's seven edges (coordinates clamped into the grid,
        // those across its edge zeroed)
        const int cy = min(max(gy, 0), ny - 1), dy = max(cy - 1, 0);
        C<T> ux[3], ud[2], uu[2];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int cx = min(max(ge - 1 + k, 0), nx - 1);
            const int c[3] = {cx, cy, 0};
            ux[k] = link_u<2, T>(U, 0, c, cx);
            if (ge - 1 + k < 0 || ge - 1 + k >= nx - 1) ux[k] = mk<T>(0, 0);
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int c[3] = {min(max(ge + k, 0), nx - 1), cy, 0};
            ud[k] = gy > 0 ? link_u<2, T>(U, 1, c, dy) : mk<T>(0, 0);
            uu[k] = gy < ny - 1 ? link_u<2, T>(U, 1, c, cy) : mk<T>(0, 0);
        }
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            L0Node<T> &m = n[col];
            m.odd = (col ^ gy) & 1;
            m.gx = ge + m.odd;
            m.in = row && m.gx >= 0 && m.gx < nx;
            const int lx = 2 * lp + m.odd;
            m.ring = m.in ? min(min(lx, S::LX - 1 - lx), min(ly, S::LY - 1 - ly)) : -1;
            m.ul = l0_pick(m.odd, ux[1], ux[0]);
            m.ur = l0_pick(m.odd, ux[2], ux[1]);
            m.ud = l0_pick(m.odd, ud[1], ud[0]);
            m.uu = l0_pick(m.odd, uu[1], uu[0]);
            const int c[3] = {m.gx, gy, 0};
            T sc[3];
            const T vol = node_volume<2, T>(g, c, sc);
            m.a0 = vol * sc[0] * g.inv_h2[0];
            m.a1 = vol * sc[1] * g.inv_h2[1];
            m.d = m.in ? hs[col * g.npair + t] : (T)1;
            m.w = (T)1 / m.d;
            m.b = m.x = mk<T>(0, 0);
        }
    }
    // the sum above for the node of colour col, given the other colour's values
    __device__ __forceinline__ C<T> offdiag(int col, const C<T> *other) const
    {
        const L0Node<T> &m = n[col];
        return m.offdiag(n[1 - col].x, other[m.odd ? p + 1 : p - 1], other[p - S::PX], other[p + S::PX]);
    }
    // x = (b - sum) / d where the node is at least rmin rings in
    __device__ __forceinline__ void update(int col, int rmin, const C<T> *other)
    {
        L0Node<T> &m = n[col];
        if (m.ring >= rmin) m.x = cscale(csub(m.b, offdiag(col, other)), m.w);
    }
};

// Down: b = round(v), red from zero, black, red, black residual (L0PreBlack,
// L0Sweep(0), L0Residual); writes b and x of the tile's nodes and r of its
// black nodes in the split layout.
template <class T, class S>
struct L0PreTile {
    GeomT<T> g;
    const double2 *v;
    const T *hs;
    LinkTab<T> U;
    C<T> *b, *x, *r;
    int ntx;
    const int *gate;
    __device__ void operator()(int bx, int nbx) const
    {
        GATE_LOAD();
        __shared__ C<T> sr[S::pairs], sb[S::pairs];
        const int tile = xcd_tile(bx, nbx);
        L0Pair<T, S> P(g, U, hs, tile, ntx);
#pragma unroll
        for (int col = 0; col < 2; ++col)
            if (P.n[col].in) P.n[col].b = narrow<T>(v[P.n[col].gx + g.N[0] * P.gy]);
        P.n[0].x = cscale(P.n[0].b, P.n[0].w);  // red from zero: x = b / d
        if (P.act) sr[P.p] = P.n[0].x;
        __syncthreads();
        P.update(1, 1, sr);
        if (P.act) sb[P.p] = P.n[1].x;
        __syncthreads();
        P.update(0, 2, sb);
        if (P.act) sr[P.p] = P.n[0].x;
        __syncthreads();
        if (!P.own || !gate_go) return;
        const int np = g.npair;
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            if (!P.n[col].in) continue;
            b[col * np + P.t] = P.n[col].b;
            x[col * np + P.t] = P.n[col].x;
        }
        const L0Node<T> &m = P.n[1];
        if (m.in) r[np + P.t] = csub(csub(m.b, cscale(m.x, m.d)), P.offdiag(1, sr));
    }
};

// (P x_c)_k with four entries in flight
template <class T>
__device__ __forceinline__ C<T> prolong_row4(const int *__restrict__ prp, const int *__restrict__ pci,
                                             const C<T> *__restrict__ pv, const C<T> *__restrict__ xc, int k)
{
    C<T> s = mk<T>(0, 0);
    const int p1 = prp[k + 1];
    for (int p = prp[k]; p < p1; p += 4) {
        C<T> a[4], x[4];
        int j[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int pe = min(p + e, p1 - 1);
            j[e] = pci[pe];
            a[e] = pv[pe];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = xc[j[e]];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (p + e < p1) s = cadd(s, cmul(a[e], x[e]));
    }
    return s;
}

// Up: black += (P x_c)_b, red, black, last red; z = x on the tile's nodes (ADD:
// z += x) and partial sums of Re<vdot, z> (L0ProlongBlack, L0Sweep(0),
// L0Sweep(1), L0Last).
template <class T, class TC, int ADD, class S>
struct L0PostTile {
    GeomT<T> g;
    const C<T> *b, *x;
    const T *hs;
    LinkTab<T> U;
    const int *prp, *pci;
    const C<TC> *pv, *xc;
    double2 *z;
    const double2 *vdot;
    RedSlot slot;
    int want_dot;
    DeflDot dd;
    int ntx;
    const int *gate;
    __device__ void operator()(int bx, int nbx) const
    {
        GATE_LOAD();
        __shared__ C<T> sr[S::pairs], sb[S::pairs];
        __shared__ double sm[S::threads / 64];
        const int tile = xcd_tile(bx, nbx), np = g.npair;
        L0Pair<T, S> P(g, U, hs, tile, ntx);
#pragma unroll
        for (int col = 0; col < 2; ++col)
            if (P.n[col].in) P.n[col].b = b[col * np + P.t];
        // red values are recomputed from the black ones before any use
        if (P.n[1].in) P.n[1].x = cadd(x[np + P.t], as_c<T>(prolong_row4<TC>(prp, pci, pv, xc, P.t)));
        // what the tile's own nodes are multiplied with, loaded behind the passes
        double2 vd[2], ps[2], zo[2];
#pragma unroll
        for (int col = 0; col < 2; ++col) {
            vd[col] = ps[col] = zo[col] = make_double2(0.0, 0.0);
            if (!P.own || !P.n[col].in) continue;
            const int i = P.n[col].gx + g.N[0] * P.gy;
            if (want_dot) vd[col] = vdot[i];
            if (dd.psi) ps[col] = dd.psi[i];
            if (ADD) zo[col] = z[i];
        }
        if (P.act) sb[P.p] = P.n[1].x;
        __syncthreads();
        P.update(0, 1, sb);
        if (P.act) sr[P.p] = P.n[0].x;
        __syncthreads();
        P.update(1, 2, sr);
        if (P.act) sb[P.p] = P.n[1].x;
        __syncthreads();
        // last red on the tile, into z only; z on every node of the tile
        double part = 0.0, part_u = 0.0;
        if (P.own) {
            P.update(0, 3, sb);
#pragma unroll
            for (int col = 0; col < 2; ++col) {
                const L0Node<T> &m = P.n[col];
                if (!m.in) continue;
                double2 zi = widen(m.x);
                if (ADD) zi = cadd(zo[col], zi);
                if (want_dot) part += redot(vd[col], zi);
                if (dd.psi) {
                    const int c[3] = {m.gx, P.gy, 0};
                    part_u += dd.weight<2>(0, c) * (ps[col].x * zi.y - ps[col].y * zi.x);
                }
                if (gate_go) z[m.gx + g.N[0] * P.gy] = zi;
            }
        }
        if (want_dot && gate_go) block_reduce_store(part, slot, sm, bx);
        if (dd.psi && gate_go) block_reduce_store(part_u, dd.slot, sm, bx);
    }
};

// --------------------------------------------------------------- CSR ---
// LPR lanes of one wave share a row; partial sums are combined by shuffles.
template <class T, int LPR>
__device__ __forceinline__ C<T> lanes_sum(C<T> s)
{
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) {
        s.x += __shfl_xor(s.x, o, 64);
        s.y += __shfl_xor(s.y, o, 64);
    }
    return s;
}

// Symmetric Gauss-Seidel sweeps on a level in colour order, A = L + D + U by that
// order.  What a pass needs of a row is the part whose product is not known yet:
//   down, from zero  forward   t = D^-1 (b - L t)
//                    backward  e = D^-1 U x,  x = t - e
//                    residual  t = b - A x = L e
//   up               right-hand side of the forward half  r = b - U x
//                    forward   t = D^-1 (r - L t), then r = b - L t
//                    backward  x = D^-1 (r - U x)
// (e is kept in r.)  That is three reads of the matrix a cycle instead of five, and a
// pass writes a vector that it reads only at rows already final, so nothing is
// updated in place.  The rows are padded blocks per colour (ELL), sorted by column:
// the lower part of a row of colour c lies within its first elow[c] entries, the
// upper part from entry eup[c] on.
// A pass of a few thousand rows is bound by its launch and two dependent trips to
// memory (5.5-6 us), one of a large level by the rows' traffic, so passes with
// nothing to gather are not dispatches of their own: the first colour from zero
// (t = D^-1 b) is formed by the kernel that writes b, in the sweep of x by that of r =
// b - U x, and the last colour's backward value is its forward one (its rows have no
// U).  C colours take 2 C - 1 dispatches each way, as many as whole rows updated in
// place with a residual of their own.  us per MINRES iteration, automatic tiles, whole
// rows / halves with 2 C + 1 dispatches / now: tetrahedron of 3 101 nodes 186 / 81 /
// 73 FP64, 97^3 1151 / 920 / 900, 129^3 1596 / 1310 / 1291 and FP32 1364 / 1149 /
// 1132; one application (gl_precond_apply) to 5x5x3001 204 / 214 / 206, to 129^3 1488
// / 1199 / 1182.  (Two colours per dispatch, the second forming the values it needs of
// the first itself: 97^3 1942, 129^3 FP32 1340 against 910 and 836; the first colour
// alone that way: 129^3 2 % slower, its FP64 divisions.)
enum { SGS_FWD0 = 0, SGS_FWD = 1, SGS_BWD0 = 2, SGS_BWD = 3 };

// One colour: its rows and the entries [lo, hi) of them that hold the part.  LPR
// lanes share a row, with kSgsBatch entries of each in flight; the gate is loaded
// alongside the data and checked only before the store.
constexpr int kSgsBatch = 4;

// last: no later colour, so x is the forward value.
template <class T, int LPR, int MODE>
struct SgsPass {
    const int *eci;
    const C<T> *ev;
    int W, lo, hi, row0, cnt;
    bool last;
    const T *diag;
    const C<T> *b;
    C<T> *x, *r, *t;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        constexpr bool fwd = MODE == SGS_FWD0 || MODE == SGS_FWD;
        const int go = gate ? *gate : 1;
        const int g = bx * kBlock + threadIdx.x;
        const int row = g / LPR, lane = g % LPR;
        const bool act = row < cnt;
        const int i = row0 + (act ? row : 0);
        // the row's own terms do not depend on the gathers
        const bool own = act && lane == 0;
        C<T> p = mk<T>(0, 0), q = p;
        T d = (T)1;
        if (own) {
            d = diag[i];
            p = MODE == SGS_FWD0 ? b[i] : MODE == SGS_BWD0 ? t[i] : r[i];
            if (MODE == SGS_FWD) q = b[i];
        }
        const C<T> *from = fwd ? t : x;
        C<T> s = mk<T>(0, 0);
        if (act) {
            const size_t base = (size_t)row * W;
            for (int k = lo + lane; k < hi; k += kSgsBatch * LPR) {
                int c[kSgsBatch];
                C<T> a[kSgsBatch], v[kSgsBatch];
#pragma unroll
                for (int u = 0; u < kSgsBatch; ++u) {
                    const int e = min(k + u * LPR, hi - 1);
                    c[u] = eci[base + e];
                    a[u] = ev[base + e];
                }
#pragma unroll
                for (int u = 0; u < kSgsBatch; ++u) v[u] = from[c[u]];
#pragma unroll
                for (int u = 0; u < kSgsBatch; ++u)
                    if (k + u * LPR < hi && (fwd ? c[u] < row0 : c[u] >= row0 + cnt)) s = cadd(s, cmul(a[u], v[u]));
            }
        }
        s = lanes_sum<T, LPR>(s);
        if (!own || !go) return;
        const T w = (T)1 / d;
        if (MODE == SGS_BWD0) {
            const C<T> e = cscale(s, w);
            r[i] = e;
            x[i] = csub(p, e);
        } else {
            const C<T> n = cscale(csub(p, s), w);
            (fwd ? t : x)[i] = n;
            if (fwd && last) x[i] = n;
            if (MODE == SGS_FWD) r[i] = csub(q, s);
        }
    }
};

// y = L e (UP = 0) or y = b - U x (UP = 1) from the sorted rows; UP: the rows of
// colour 0, the first `first`, also take their forward value t = D^-1 (b - U x), and y = b
template <class T, int LPR, int UP>
struct SgsProduct {
    int n, first;
    const int *rp, *ci, *dpos;
    const C<T> *v, *b, *x;
    const T *diag;
    C<T> *y, *t;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE_LOAD();
        const int g = bx * kBlock + threadIdx.x;
        const int i = g / LPR, lane = g % LPR;
        const bool act = i < n;
        const C<T> bi = UP && act && lane == 0 ? b[i] : mk<T>(0, 0);
        C<T> s = mk<T>(0, 0);
        if (act) {
            const int p0 = UP ? dpos[i] + 1 : rp[i], p1 = UP ? rp[i + 1] : dpos[i];
            for (int p = p0 + lane; p < p1; p += LPR) s = cadd(s, cmul(v[p], x[ci[p]]));
        }
        s = lanes_sum<T, LPR>(s);
        if (!act || lane != 0 || !gate_go) return;
        const C<T> yi = UP ? csub(bi, s) : s;
        if (UP && i < first) {  // (the diagonal loaded ahead of the sum: 80 us for 255 871 rows, 35 here)
            t[i] = cscale(yi, (T)1 / diag[i]);
            y[i] = bi;
        } else {
            y[i] = yi;
        }
    }
};

// The rows of colour 0 of a level that runs its sweeps by colour passes, for the
// kernel that writes its right-hand side b: t = D^-1 b there (n = 0: none)
template <class T>
struct FirstColour {
    int n = 0;
    const T *diag = nullptr;
    C<T> *t = nullptr;
};

// y = A x (ADD = 0) or y += A x (ADD = 1); x may be held in the other precision
template <class T, int LPR, int ADD, class TX = T>
struct CsrSpmv {
    int n;
    const int *rp, *ci;
    const C<T> *v;
    const C<TX> *x;
    C<T> *y;
    FirstColour<T> fc;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE_LOAD();
        const int t = bx * kBlock + threadIdx.x;
        const int i = t / LPR, lane = t % LPR;
        const bool act = i < n;
        const C<T> yi = ADD && act && lane == 0 ? y[i] : mk<T>(0, 0);
        const T d = !ADD && lane == 0 && i < fc.n ? fc.diag[i] : (T)1;
        C<T> s = mk<T>(0, 0);
        if (act)
            for (int p = rp[i] + lane; p < rp[i + 1]; p += LPR) s = cadd(s, cmul(v[p], as_c<T>(x[ci[p]])));
        s = lanes_sum<T, LPR>(s);
        if (!act || lane != 0 || !gate_go) return;
        y[i] = ADD ? cadd(yi, s) : s;
        if (!ADD && i < fc.n) fc.t[i] = cscale(s, (T)1 / d);
    }
};

// ----------------------------------------------------- patch sweeps ---
// A whole symmetric Gauss-Seidel sweep of a level in one dispatch: a
// work-group runs every colour pass on its patch (PatchSet), a thread per row
// with the row's entries in registers and the iterate in LDS.  A pass is a
// handful of LDS reads, a chain of FP64 adds and a barrier (0.5 us) where a
// dispatch per pass took 3-4 us, most of it launch and two dependent round trips
// to memory; loading the patch takes 4-6 us (latency: rows, then what they
// index), and the price is the rows that more than one patch updates (3-5 per
// row of the level; 2.3-2.7 in the large patches of large levels, which that
// traffic bounds).  FP64, down / up: 4 923 and 545 rows of 7 and 8 colours 12 /
// 14 us (46 / 50 as 14-16 dispatches), 44 075 rows of 5 colours 13 / 19 us (35 /
// 31); FP32, 175 446 rows of 4 colours 14 / 22 us (42 / 40; 21 / 38 in patches of 512).
// Every row's value is the update of the per-pass kernels, so the sweep is the
// same up to the order of the row sums.  The starting value of a row beyond
// the patch is read, never written, and the sweep's result goes to another
// vector (r, whose content is used up by then), so patches do not disturb one
// another.
template <class T, int W, int NR>
struct PatchArrays {
    const int *size, *rowid, *info;
    const unsigned short *idx;
    const C<T> *v;
    const T *diag;
    int ncol;
    int planes;  // entries per row in the arrays, W of them held in registers
};

template <class T, int W, int NR>
struct PatchRow {
    int g, colour, last, cnt;
    bool own;
    int wide;  // entries of the wave's longest row: 8, 12, 16, or more than W
    T d;
    C<T> b, v[W];
    unsigned idx[W / 2];  // two slots each
    const C<T> *vg;
    const unsigned short *ig;
};

// Every load that depends on no other first, then those through the row's
// index.  Most waves have no row of more than eight neighbours (the interior of
// the 2D hierarchies): the entries after the eighth are read, and summed, by the
// others only.  The few rows with more than 16 read the rest in every pass
// (24 held entries leave one work-group per CU, and spill with 1024 rows: 66 us
// instead of 25 for 1 121 rows in FP64).
template <class T, int W, int NR>
__device__ __forceinline__ PatchRow<T, W, NR> patch_load(const PatchArrays<T, W, NR> &A, int p, const C<T> *b)
{
    PatchRow<T, W, NR> R;
    const int i = threadIdx.x;
    const size_t base = (size_t)p * A.planes * NR + i;
    R.vg = A.v + base;
    R.ig = A.idx + base;
    R.g = A.rowid[(size_t)p * 2 * NR + i];
    const int inf = A.info[(size_t)p * NR + i];
    auto part = [&](auto k0, auto k1) {
#pragma unroll
        for (int k = decltype(k0)::value; k < decltype(k1)::value; ++k) {
            R.v[k] = R.vg[(size_t)k * NR];
            const unsigned at = R.ig[(size_t)k * NR];
            R.idx[k / 2] = k & 1 ? R.idx[k / 2] | at << 16 : at;
        }
    };
    part(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{});
    R.d = A.diag[R.g];
    R.b = b[R.g];
    R.colour = inf & 255;
    R.last = (inf >> 8) & 255;
    R.own = (inf >> 16 & 1) != 0;
    R.cnt = inf >> 20;
    R.wide = 8;
    if constexpr (W > 8)
        if (__any(R.cnt > 8)) {
            R.wide = 12;
            part(std::integral_constant<int, 8>{}, std::integral_constant<int, 12>{});
        }
    if constexpr (W > 12)
        if (__any(R.cnt > 12)) {
            R.wide = __any(R.cnt > 16) ? W + 1 : 16;
            part(std::integral_constant<int, 12>{}, std::integral_constant<int, 16>{});
        }
    return R;
}

// sum of the row's products
template <class T, int W, int NR>
__device__ __forceinline__ C<T> patch_sum(const PatchRow<T, W, NR> &R, const C<T> *xs)
{
    C<T> s = mk<T>(0, 0);
    auto part = [&](auto k0, auto k1) {
#pragma unroll
        for (int k = decltype(k0)::value; k < decltype(k1)::value; ++k)
            s = cadd(s, cmul(R.v[k], xs[k & 1 ? R.idx[k / 2] >> 16 : R.idx[k / 2] & 0xFFFFu]));
    };
    part(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{});
    if constexpr (W > 8)
        if (R.wide > 8) part(std::integral_constant<int, 8>{}, std::integral_constant<int, 12>{});
    if constexpr (W > 12) {
        if (R.wide > 12) part(std::integral_constant<int, 12>{}, std::integral_constant<int, 16>{});
        if (R.wide > W)
            for (int k = W; k < R.cnt; ++k) s = cadd(s, cmul(R.vg[(size_t)k * NR], xs[R.ig[(size_t)k * NR]]));
    }
    return s;
}

template <class T, int W, int NR>
__device__ __forceinline__ void patch_sweep(const PatchRow<T, W, NR> &R, int ncol, C<T> *xs)
{
    const T inv = (T)1 / R.d;
    for (int t = 0; t < 2 * ncol - 1; ++t) {
        const int c = t < ncol ? t : 2 * ncol - 2 - t;
        if (R.colour == c && t < R.last) xs[threadIdx.x] = cscale(csub(R.b, patch_sum<T, W, NR>(R, xs)), inv);
        __syncthreads();
    }
}

// x = the sweep from zero, r = b - A x, on the patch's own rows
template <class T, int W, int NR>
struct PatchPre {
    PatchArrays<T, W, NR> A;
    const C<T> *b;
    C<T> *x, *r;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE_LOAD();
        __shared__ C<T> xs[2 * NR + 1];
        const PatchRow<T, W, NR> R = patch_load<T, W, NR>(A, bx, b);
        for (int q = threadIdx.x; q <= 2 * NR; q += NR) xs[q] = mk<T>(0, 0);
        __syncthreads();
        patch_sweep<T, W, NR>(R, A.ncol, xs);
        if (!R.own || !gate_go) return;
        const C<T> xi = xs[threadIdx.x];
        x[R.g] = xi;
        r[R.g] = csub(csub(R.b, cscale(xi, R.d)), patch_sum<T, W, NR>(R, xs));
    }
};

// xo = the sweep from x + P x_c on the patch's own rows (TX: the precision of
// x_c; P's rows padded to PW entries)
template <class T, class TX, int W, int NR>
struct PatchPost {
    PatchArrays<T, W, NR> A;
    const C<T> *b, *x;
    int PW;
    const int *pci;
    const C<T> *pv;
    const C<TX> *xc;
    C<T> *xo;
    const int *gate;
    __device__ C<T> start(int g) const
    {
        C<T> s = x[g];
        const size_t o = (size_t)g * PW;
        for (int k = 0; k < PW; k += 4) {
            int c[4];
            C<T> pk[4], xk[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                c[u] = k + u < PW ? pci[o + k + u] : 0;
                pk[u] = k + u < PW ? pv[o + k + u] : mk<T>(0, 0);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) xk[u] = as_c<T>(xc[c[u]]);
#pragma unroll
            for (int u = 0; u < 4; ++u) s = cadd(s, cmul(pk[u], xk[u]));
        }
        return s;
    }
    __device__ void operator()(int bx, int) const
    {
        GATE_LOAD();
        __shared__ C<T> xs[2 * NR + 1];
        const int ns = A.size[2 * bx + 1];
        const int g1 = A.rowid[(size_t)bx * 2 * NR + NR + threadIdx.x];
        const PatchRow<T, W, NR> R = patch_load<T, W, NR>(A, bx, b);
        xs[threadIdx.x] = start(R.g);
        if (NR + (int)threadIdx.x < ns) xs[NR + threadIdx.x] = start(g1);
        if (threadIdx.x == 0) xs[2 * NR] = mk<T>(0, 0);
        __syncthreads();
        patch_sweep<T, W, NR>(R, A.ncol, xs);
        if (R.own && gate_go) xo[R.g] = xs[threadIdx.x];
    }
};

template <class T>
struct Narrow {
    int n;
    const double2 *v;
    C<T> *b;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE();
        const int i = bx * kBlock + threadIdx.x;
        if (i < n) b[i] = narrow<T>(v[i]);
    }
};

// z = x (ADD = 0) or z += x (ADD = 1); partial sums of Re<vdot, z>
template <int DIM, class T, int ADD>
struct Output {
    int n;
    const C<T> *x;
    const double2 *vdot;
    double2 *z;
    RedSlot slot;
    int want_dot;
    DeflDot dd;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE();
        __shared__ double sm[kBlock / 64];
        const int i = bx * kBlock + threadIdx.x;
        double part = 0.0, part_u = 0.0;
        if (i < n) {
            double2 zi = widen(x[i]);
            if (ADD) zi = cadd(z[i], zi);
            z[i] = zi;
            if (want_dot) part = redot(vdot[i], zi);
            if (dd.psi) {
                int c[3];
                node_coords<DIM>(dd.N, i, c);
                part_u = dd.term<DIM>(i, c, zi);
            }
        }
        if (want_dot) block_reduce_store(part, slot, sm, bx);
        if (dd.psi) block_reduce_store(part_u, dd.slot, sm, bx);
    }
};

// b[r] = round(v[perm[r]]): level 0 of a simplicial mesh, whose V-cycle
// vectors are in colour order (row r is node perm[r])
template <class T>
struct NarrowPerm {
    int n;
    const double2 *v;
    const int *perm;
    C<T> *b;
    FirstColour<T> fc;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE();
        const int r = bx * kBlock + threadIdx.x;
        if (r >= n) return;
        const C<T> br = narrow<T>(v[perm[r]]);
        b[r] = br;
        if (r < fc.n) fc.t[r] = cscale(br, (T)1 / fc.diag[r]);
    }
};

// z[perm[r]] = x[r] (ADD: +=), partial sums of Re<vdot, z> in row order
template <class T, int ADD>
struct OutputPerm {
    int n;
    const C<T> *x;
    const int *perm;
    const double2 *vdot;
    double2 *z;
    RedSlot slot;
    int want_dot;
    DeflDot dd;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE();
        __shared__ double sm[kBlock / 64];
        const int r = bx * kBlock + threadIdx.x;
        double part = 0.0, part_u = 0.0;
        if (r < n) {
            const int i = perm[r];
            double2 zi = widen(x[r]);
            if (ADD) zi = cadd(z[i], zi);
            z[i] = zi;
            if (want_dot) part = redot(vdot[i], zi);
            if (dd.psi) {
                const int c[3] = {i, 0, 0};
                part_u = dd.term<0>(i, c, zi);
            }
        }
        if (want_dot) block_reduce_store(part, slot, sm, bx);
        if (dd.psi) block_reduce_store(part_u, dd.slot, sm, bx);
    }
};

// x = M b for a dense row-major operator (the coarsest inverse or an explicit
// sub-cycle), a wave per row.  Each lane issues kDenseUnroll loads before it
// uses any (a row of a few thousand entries is otherwise one memory round
// trip per 64 entries); the sum still runs over j = lane, lane + 64, ... in
// that order.
constexpr int kDenseUnroll = 8;

template <class T>
struct DenseApply {
    int n;
    const C<T> *M, *b;
    C<T> *x;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE_LOAD();
        const int t = bx * kBlock + threadIdx.x;
        const int i = t / 64, lane = t % 64;
        const bool act = i < n;
        C<T> s = mk<T>(0, 0);
        if (act) {
            const C<T> *row = M + (size_t)i * n;
            for (int j0 = 0; j0 < n; j0 += 64 * kDenseUnroll) {
                C<T> m[kDenseUnroll], v[kDenseUnroll];
#pragma unroll
                for (int u = 0; u < kDenseUnroll; ++u) {
                    const int j = j0 + u * 64 + lane;
                    m[u] = j < n ? row[j] : mk<T>(0, 0);
                    v[u] = j < n ? b[j] : mk<T>(0, 0);
                }
#pragma unroll
                for (int u = 0; u < kDenseUnroll; ++u)
                    if (j0 + u * 64 + lane < n) s = cadd(s, cmul(m[u], v[u]));
            }
        }
        s = lanes_sum<T, 64>(s);
        if (act && lane == 0 && gate_go) x[i] = s;
    }
};

// ------------------------------------------------------------ bottom ---
// Every level from D.first down to the coarsest, in one work-group of
// kBottomThreads threads: the same V-cycle steps as the multi-kernel levels,
// separated by work-group barriers, and the dense solve.  One work-group
// avoids a dispatch per colour pass, but a step costs about 3 us even over a
// handful of rows (a dependent global load is about 1 us away, measured on
// MI355X) and one compute unit streams about 20-25 GB/s, so this pays only for
// levels of a few hundred rows; the tile autotuner chooses the bound
// (bottom_rows).  Eight lanes share a row, so a colour pass of such a level
// is one round of loads.
constexpr int kBottomThreads = 1024;
constexpr int kBottomLpr = 8;

// one colour of a level, from its ELL block; x in LDS or global memory
template <class T>
__device__ __forceinline__ void bottom_rows_sgs(const BottomLevel<T> &L, int colour, const C<T> *b, C<T> *x)
{
    const int cnt = L.coff[colour + 1] - L.coff[colour];
    const int row0 = L.coff[colour];
    const int W = L.ewidth[colour];
    const int *eci = L.eci + L.eoff[colour];
    const C<T> *ev = L.ev + L.eoff[colour];
    const int per = kBottomThreads / kBottomLpr;
    const int lane = threadIdx.x % kBottomLpr;
    for (int base = 0; base < cnt; base += per) {
        const int r = base + threadIdx.x / kBottomLpr;
        const bool act = r < cnt;
        const int i = row0 + (act ? r : 0);
        C<T> s = mk<T>(0, 0);
        if (act)
            for (int k = lane; k < W; k += kBottomLpr) {
                const int j = eci[(size_t)r * W + k];
                if (j != i) s = cadd(s, cmul(ev[(size_t)r * W + k], x[j]));
            }
        s = lanes_sum<T, kBottomLpr>(s);
        if (act && lane == 0) x[i] = cscale(csub(b[i], s), (T)1 / L.diag[i]);
    }
}

// MODE 0: y = M x, 1: y += M x, 2: y = b - M x
template <class T, int MODE>
__device__ __forceinline__ void bottom_rows_spmv(int nrows, const int *rp, const int *ci, const C<T> *v,
                                                 const C<T> *x, const C<T> *b, C<T> *y)
{
    const int per = kBottomThreads / kBottomLpr;
    const int lane = threadIdx.x % kBottomLpr;
    for (int base = 0; base < nrows; base += per) {
        const int i = base + threadIdx.x / kBottomLpr;
        const bool act = i < nrows;
        C<T> s = mk<T>(0, 0);
        if (act)
            for (int p = rp[i] + lane; p < rp[i + 1]; p += kBottomLpr) s = cadd(s, cmul(v[p], x[ci[p]]));
        s = lanes_sum<T, kBottomLpr>(s);
        if (act && lane == 0) {
            if (MODE == 0) y[i] = s;
            else if (MODE == 1) y[i] = cadd(y[i], s);
            else y[i] = csub(b[i], s);
        }
    }
}

// y = M b for a dense row-major n x n matrix
template <class T>
__device__ __forceinline__ void bottom_dense(int n, const C<T> *M, const C<T> *b, C<T> *y)
{
    const int per = kBottomThreads / kBottomLpr;
    const int lane = threadIdx.x % kBottomLpr;
    for (int base = 0; base < n; base += per) {
        const int i = base + threadIdx.x / kBottomLpr;
        const bool act = i < n;
        C<T> s = mk<T>(0, 0);
        if (act)
            for (int j = lane; j < n; j += kBottomLpr) s = cadd(s, cmul(M[(size_t)i * n + j], b[j]));
        s = lanes_sum<T, kBottomLpr>(s);
        if (act && lane == 0) y[i] = s;
    }
}

template <class T>
__device__ __forceinline__ void bottom_sgs(const BottomLevel<T> &L, const C<T> *b, C<T> *x)
{
    for (int t = 0; t < 2 * L.ncolors - 1; ++t) {
        bottom_rows_sgs<T>(L, t < L.ncolors ? t : 2 * L.ncolors - 2 - t, b, x);
        __syncthreads();
    }
}

// The V-cycle over levels D.first .. D.last in one work-group: the same
// steps as the multi-kernel levels, then the dense operator of level D.last.
// vec(l, k) is level l's right-hand side (k = 0), iterate (1) or residual (2).
template <class T, class V>
__device__ __forceinline__ void bottom_cycle(const BottomDesc<T> &D, V vec)
{
    for (int l = D.first; l < D.last; ++l) {
        const BottomLevel<T> &L = D.L[l];
        C<T> *b = vec(l, 0), *x = vec(l, 1), *r = vec(l, 2);
        for (int i = threadIdx.x; i < L.n; i += kBottomThreads) x[i] = mk<T>(0, 0);
        __syncthreads();
        bottom_sgs<T>(L, b, x);
        bottom_rows_spmv<T, 2>(L.n, L.rp, L.ci, L.v, x, b, r);
        __syncthreads();
        bottom_rows_spmv<T, 0>(L.nc, L.rrp, L.rci, L.rv, r, nullptr, vec(l + 1, 0));
        __syncthreads();
    }
    bottom_dense<T>(D.L[D.last].n, D.cinv, vec(D.last, 0), vec(D.last, 1));
    __syncthreads();
    for (int l = D.last - 1; l >= D.first; --l) {
        const BottomLevel<T> &L = D.L[l];
        C<T> *x = vec(l, 1);
        bottom_rows_spmv<T, 1>(L.n, L.prp, L.pci, L.pv, vec(l + 1, 1), nullptr, x);
        __syncthreads();
        bottom_sgs<T>(L, vec(l, 0), x);
    }
}

// The level D.lds_level (the largest one handled here, when it fits) keeps
// its iterate in LDS for the whole cycle and writes it out at the end.
template <class T>
struct Bottom {
    const BottomDesc<T> *Dp;
    const int *gate;
    __device__ void operator()(int, int) const
    {
        GATE();
        extern __shared__ double2 glk_bottom_lds[];
        const BottomDesc<T> &D = *Dp;
        C<T> *xs = reinterpret_cast<C<T> *>(glk_bottom_lds);
        bottom_cycle<T>(D, [&](int l, int k) -> C<T> * {
            const BottomLevel<T> &L = D.L[l];
            return k == 0 ? L.b : k == 1 ? (l == D.lds_level ? xs : L.x) : L.r;
        });
        if (D.lds_level >= 0) {
            const BottomLevel<T> &L = D.L[D.lds_level];
            for (int i = threadIdx.x; i < L.n; i += kBottomThreads) L.x[i] = xs[i];
            __syncthreads();
        }
    }
};

// Forming an explicit sub-cycle kTailBlock columns at a time: vectors are
// [n][kTailBlock] blocks (the columns of a row contiguous), thread t works on row
// t / kTailBlock and column t % kTailBlock, and the kTailBlock threads of a row
// read the same matrix entries, so a level's matrix is read once per block of
// columns instead of once per column.  A thread takes its row's entries in groups
// of kTailUnroll, every gather of a group issued before any is used, and sums them
// in order.  A null right-hand side stands for columns bid .. bid + kTailBlock - 1
// of the identity.
// What bounds it is the gathers' traffic (the blocks' vectors are far larger than
// L2), so each row is split at its diagonal, A = L + D + U by the order of the
// colours, and no product that a pass has already formed is formed again:
//   forward from zero   y = (D + L)^-1 b                    reads L
//   backward            e = D^-1 U x,  x = y - e            reads U
//   residual            r = b - A x = L e                   reads L
//   forward again       s = b - L x,  x = D^-1 (s - U x)    reads L and U
//   backward            x = D^-1 (s - U x)                  reads U
// three reads of the matrix in place of five.  The sub-cycle is Hermitian, so
// a block whose first column has colour k also skips colours below k in the first
// pass (y = 0 there) and in the last (those rows are mirrored from the columns that
// compute them).  5 592 rows of 31 colours, 58 entries each: 11.9 ms (21.8 with whole
// rows and all columns); 2 173 rows of the 1025^2 hierarchy: 0.88 (1.19).  1024
// threads and 8 columns: 512 threads 15.7 and 0.92, 16 columns 14.4 and 0.99, 4
// columns of 256 threads 19.4 and 0.82, groups of four entries 14.8 and 0.89.
constexpr int kTailBlock = 8;
constexpr int kTailThreads = 1024;
constexpr int kTailRows = kTailThreads / kTailBlock;  // rows per round
constexpr int kTailUnroll = 8;

template <class T>
__device__ __forceinline__ C<T> blk_rhs(const C<T> *b, int bid, int i, int c)
{
    return b ? b[(size_t)i * kTailBlock + c] : mk<T>(i == bid + c ? 1 : 0, 0);
}

// acc += sum over k in [k0, k1) of v[k] x[idx[k]][c]
template <class T>
__device__ __forceinline__ void blk_row_sum(const int *idx, const C<T> *v, int k0, int k1, const C<T> *x, int c,
                                            C<T> &acc)
{
    for (int k = k0; k < k1; k += kTailUnroll) {
        int j[kTailUnroll];
        C<T> a[kTailUnroll], xv[kTailUnroll];
#pragma unroll
        for (int u = 0; u < kTailUnroll; ++u) {
            const int q = min(k + u, k1 - 1);
            j[u] = idx[q];
            a[u] = v[q];
        }
#pragma unroll
        for (int u = 0; u < kTailUnroll; ++u) xv[u] = x[(size_t)j[u] * kTailBlock + c];
#pragma unroll
        for (int u = 0; u < kTailUnroll; ++u)
            if (k + u < k1) acc = cadd(acc, cmul(a[u], xv[u]));
    }
}

// f(i) for the thread's rows of [r0, r1)
template <class F>
__device__ __forceinline__ void blk_rows(int r0, int r1, F &&f)
{
    for (int i = r0 + threadIdx.x / kTailBlock; i < r1; i += kTailRows) f(i);
}

// y = M x, or y += M x
template <class T, bool ADD>
__device__ __forceinline__ void blk_spmv(int nrows, const int *rp, const int *ci, const C<T> *v, const C<T> *x, C<T> *y)
{
    const int c = threadIdx.x % kTailBlock;
    blk_rows(0, nrows, [&](int i) {
        C<T> &yi = y[(size_t)i * kTailBlock + c];
        C<T> acc = mk<T>(0, 0);
        blk_row_sum<T>(ci, v, rp[i], rp[i + 1], x, c, acc);
        yi = ADD ? cadd(yi, acc) : acc;
    });
}

// y = M b for a dense row-major n x n matrix
template <class T>
__device__ __forceinline__ void blk_dense(int n, const C<T> *M, const C<T> *b, C<T> *y)
{
    const int c = threadIdx.x % kTailBlock;
    blk_rows(0, n, [&](int i) {
        const C<T> *row = M + (size_t)i * n;
        C<T> acc = mk<T>(0, 0);
        int j = 0;
        for (; j + kTailUnroll <= n; j += kTailUnroll) {
            C<T> a[kTailUnroll], xv[kTailUnroll];
#pragma unroll
            for (int u = 0; u < kTailUnroll; ++u) {
                a[u] = row[j + u];
                xv[u] = b[(size_t)(j + u) * kTailBlock + c];
            }
#pragma unroll
            for (int u = 0; u < kTailUnroll; ++u) acc = cadd(acc, cmul(a[u], xv[u]));
        }
        for (; j < n; ++j) acc = cadd(acc, cmul(row[j], b[(size_t)j * kTailBlock + c]));
        y[(size_t)i * kTailBlock + c] = acc;
    });
}

// the first colour with rows at or past row i
template <class T>
__device__ __forceinline__ int blk_colour(const BottomLevel<T> &L, int i)
{
    int k = 0;
    while (L.coff[k + 1] <= i) ++k;
    return k;
}

// b of a level below the one whose columns are formed (null on that level), its
// iterate, e (then s) and residual
template <class T>
struct BlkVec {
    C<T> *b, *x, *e, *r;
};

// The V-cycle over levels D.first .. D.last on kTailBlock identity columns
template <class T, class V>
__device__ __forceinline__ void blk_cycle(const BottomDesc<T> &D, V vec, int bid)
{
    const int c = threadIdx.x % kTailBlock;
    const int kfirst = blk_colour<T>(D.L[D.first], bid);
    for (int l = D.first; l < D.last; ++l) {
        const BottomLevel<T> &L = D.L[l];
        const BlkVec<T> W = vec(l);
        const int k0 = l == D.first ? kfirst : 0;
        blk_rows(0, L.coff[k0], [&](int i) { W.x[(size_t)i * kTailBlock + c] = mk<T>(0, 0); });
        __syncthreads();
        for (int k = k0; k < L.ncolors; ++k) {
            blk_rows(L.coff[k], L.coff[k + 1], [&](int i) {
                C<T> acc = mk<T>(0, 0);
                blk_row_sum<T>(L.ci, L.v, L.rp[i], L.dpos[i], W.x, c, acc);
                W.x[(size_t)i * kTailBlock + c] = cscale(csub(blk_rhs<T>(W.b, bid, i, c), acc), (T)1 / L.diag[i]);
            });
            __syncthreads();
        }
        for (int k = L.ncolors - 1; k >= 0; --k) {
            blk_rows(L.coff[k], L.coff[k + 1], [&](int i) {
                const size_t q = (size_t)i * kTailBlock + c;
                C<T> acc = mk<T>(0, 0);
                blk_row_sum<T>(L.ci, L.v, L.dpos[i] + 1, L.rp[i + 1], W.x, c, acc);
                const C<T> e = cscale(acc, (T)1 / L.diag[i]);
                W.e[q] = e;
                W.x[q] = csub(W.x[q], e);
            });
            __syncthreads();
        }
        blk_rows(0, L.n, [&](int i) {
            C<T> acc = mk<T>(0, 0);
            blk_row_sum<T>(L.ci, L.v, L.rp[i], L.dpos[i], W.e, c, acc);
            W.r[(size_t)i * kTailBlock + c] = acc;
        });
        __syncthreads();
        blk_spmv<T, false>(L.nc, L.rrp, L.rci, L.rv, W.r, vec(l + 1).b);
        __syncthreads();
    }
    blk_dense<T>(D.L[D.last].n, D.cinv, vec(D.last).b, vec(D.last).x);
    __syncthreads();
    for (int l = D.last - 1; l >= D.first; --l) {
        const BottomLevel<T> &L = D.L[l];
        const BlkVec<T> W = vec(l);
        blk_spmv<T, true>(L.n, L.prp, L.pci, L.pv, vec(l + 1).x, W.x);
        __syncthreads();
        for (int k = 0; k < L.ncolors; ++k) {
            blk_rows(L.coff[k], L.coff[k + 1], [&](int i) {
                const size_t q = (size_t)i * kTailBlock + c;
                C<T> lo = mk<T>(0, 0), up = mk<T>(0, 0);
                blk_row_sum<T>(L.ci, L.v, L.rp[i], L.dpos[i], W.x, c, lo);
                blk_row_sum<T>(L.ci, L.v, L.dpos[i] + 1, L.rp[i + 1], W.x, c, up);
                const C<T> sl = csub(blk_rhs<T>(W.b, bid, i, c), lo);
                W.e[q] = sl;
                W.x[q] = cscale(csub(sl, up), (T)1 / L.diag[i]);
            });
            __syncthreads();
        }
        // (the last colour's rows have no U: they stay)
        const int k0 = l == D.first ? kfirst : 0;
        for (int k = L.ncolors - 2; k >= k0; --k) {
            blk_rows(L.coff[k], L.coff[k + 1], [&](int i) {
                const size_t q = (size_t)i * kTailBlock + c;
                C<T> up = mk<T>(0, 0);
                blk_row_sum<T>(L.ci, L.v, L.dpos[i] + 1, L.rp[i + 1], W.x, c, up);
                W.x[q] = cscale(csub(W.e[q], up), (T)1 / L.diag[i]);
            });
            __syncthreads();
        }
    }
}

// vectors of a level in the workspace: the first level needs no b, the coarsest no more
// than b and x
inline __host__ __device__ int tail_vectors(bool first, bool last) { return last ? 2 : first ? 3 : 4; }

// Columns of the explicit sub-cycle of level D.first: work-group g forms
// columns col0 + g kTailBlock .. + kTailBlock - 1 (those below n) with
// blocks of its own (ws + g * ws_blk: each level's vectors in turn) and stores
// them, from the diagonal down, and their mirror into the row-major n x n matrix
// out.
template <class T>
struct TailColumns {
    const BottomDesc<T> *Dp;
    C<T> *ws;
    size_t ws_blk;
    int col0, nblk;
    C<T> *out;
    __device__ void operator()(int bx, int) const
    {
        if (bx >= nblk) return;
        const BottomDesc<T> &D = *Dp;
        const int n = D.L[D.first].n, bid = col0 + bx * kTailBlock;
        C<T> *base = ws + (size_t)bx * ws_blk;
        auto vec = [&](int l) -> BlkVec<T> {
            C<T> *p = base;
            for (int q = D.first; q < l; ++q) p += tail_vectors(q == D.first, false) * (size_t)D.L[q].n * kTailBlock;
            const size_t len = (size_t)D.L[l].n * kTailBlock;
            if (l == D.first) return BlkVec<T>{nullptr, p, p + len, p + 2 * len};
            return BlkVec<T>{p, p + len, p + 2 * len, p + 3 * len};
        };
        blk_cycle<T>(D, vec, bid);
        const C<T> *x = vec(D.first).x;
        for (int t = bid * kTailBlock + threadIdx.x; t < n * kTailBlock; t += kTailThreads) {
            const int i = t / kTailBlock, col = bid + t % kTailBlock;
            if (col > i) continue;
            out[(size_t)i * n + col] = x[t];
            if (col < i) out[(size_t)col * n + i] = mk<T>(x[t].x, -x[t].y);
        }
    }
};

// ---------------------------------------------------------------- host -
template <class T> static C<T> *vec_b(Level &L);
template <class T> static C<T> *vec_x(Level &L);
template <class T> static C<T> *vec_r(Level &L);
template <> double2 *vec_b<double>(Level &L) { return L.b64.get(); }
template <> double2 *vec_x<double>(Level &L) { return L.x64.get(); }
template <> double2 *vec_r<double>(Level &L) { return L.r64.get(); }
template <> float2 *vec_b<float>(Level &L) { return L.b32.get(); }
template <> float2 *vec_x<float>(Level &L) { return L.x32.get(); }
template <> float2 *vec_r<float>(Level &L) { return L.r32.get(); }
template <class T> static C<T> *vec_t(Level &L);
template <> double2 *vec_t<double>(Level &L) { return L.t64.get(); }
template <> float2 *vec_t<float>(Level &L) { return L.t32.get(); }
template <class T> static const C<T> *vals(const Csr &M);
template <> const double2 *vals<double>(const Csr &M) { return M.v64.get(); }
template <> const float2 *vals<float>(const Csr &M) { return M.v32.get(); }
// level-0 diagonal (natural order) and the colour-ordered diagonal of l >= 1
template <class T> static const T *diag(const Level &L);
template <> const double *diag<double>(const Level &L) { return L.diag64.get(); }
template <> const float *diag<float>(const Level &L) { return L.diag32.get(); }
// level-0 diagonal in the colour-split layout of the V-cycle's level-0 vectors
template <class T> static const T *hsplit(const Level &L);
template <> const double *hsplit<double>(const Level &L) { return L.hs64.get(); }
template <> const float *hsplit<float>(const Level &L) { return L.hs32.get(); }
template <class T> static const T *dgn(const Level &L);
template <> const double *dgn<double>(const Level &L) { return L.dg64.get(); }
template <> const float *dgn<float>(const Level &L) { return L.dg32.get(); }

// dense operator of level pre->tail: the coarsest inverse, or the explicit sub-cycle
template <class T> static const C<T> *cinv(const gl_precond *p);
template <> const double2 *cinv<double>(const gl_precond *p)
{
    return p->tail < p->nlev - 1 ? p->tinv64.get() : p->cinv64.get();
}
template <> const float2 *cinv<float>(const gl_precond *p)
{
    return p->tail < p->nlev - 1 ? p->tinv32.get() : p->cinv32.get();
}
template <class T> static int bottom_lds(const gl_precond *p);
template <> int bottom_lds<double>(const gl_precond *p) { return p->lds64; }
template <> int bottom_lds<float>(const gl_precond *p) { return p->lds32; }
template <class T> static const BottomDesc<T> *bdesc(const gl_precond *p);
template <> const BottomDesc<double> *bdesc<double>(const gl_precond *p)
{
    return reinterpret_cast<const BottomDesc<double> *>(p->bdesc64.get());
}
template <> const BottomDesc<float> *bdesc<float>(const gl_precond *p)
{
    return reinterpret_cast<const BottomDesc<float> *>(p->bdesc32.get());
}

// lanes per row: about one lane per 2.5 entries, scaled by 2^shift, in 1 .. 32
static int shifted(int lpr, int shift)
{
    while (shift > 0 && lpr < 32) { lpr *= 2; --shift; }
    while (shift < 0 && lpr > 1) { lpr /= 2; ++shift; }
    return lpr;
}

static int lanes_for(const Csr &M, int shift)
{
    const double avg = M.n ? (double)M.nnz / M.n : 1.0;
    const int lpr = avg <= 2.5 ? 1 : avg <= 5.0 ? 2 : avg <= 10.0 ? 4 : avg <= 20.0 ? 8 : avg <= 40.0 ? 16 : 32;
    return shifted(lpr, shift);
}

// dispatch a CSR kernel over LPR in {1, 2, 4, 8, 16, 32}
#define GLK_LPR_SWITCH(lpr, ...)                              \
    switch (lpr) {                                            \
    case 1: { constexpr int LPR = 1; __VA_ARGS__; } break;    \
    case 2: { constexpr int LPR = 2; __VA_ARGS__; } break;    \
    case 4: { constexpr int LPR = 4; __VA_ARGS__; } break;    \
    case 8: { constexpr int LPR = 8; __VA_ARGS__; } break;    \
    case 16: { constexpr int LPR = 16; __VA_ARGS__; } break;  \
    default: { constexpr int LPR = 32; __VA_ARGS__; } break;  \
    }

template <class T, class TX = T>
static void csr_spmv(const Csr &M, const C<TX> *x, C<T> *y, bool add, int shift, const int *gate,
                     const Launch &L, const FirstColour<T> &fc = {})
{
    const int lpr = lanes_for(M, shift);
    const int nb = blocks_for((int64_t)M.n * lpr);
    GLK_LPR_SWITCH(lpr, {
        if (add) L.run(nb, CsrSpmv<T, LPR, 1, TX>{M.n, M.rp.get(), M.ci.get(), vals<T>(M), x, y, fc, gate});
        else L.run(nb, CsrSpmv<T, LPR, 0, TX>{M.n, M.rp.get(), M.ci.get(), vals<T>(M), x, y, fc, gate});
    });
}

template <class T> static const C<T> *evals(const Level &L);
template <> const double2 *evals<double>(const Level &L) { return L.ev64.get(); }
template <> const float2 *evals<float>(const Level &L) { return L.ev32.get(); }

// lanes per row of a pass whose rows have at most `part` entries in it
// (half or twice as many: 97^3 FP32 953 and 909 us per iteration, 910 with these;
// 161^3 1680 and 1675, 1632)
static int sgs_lanes(int part, int shift) { return shifted(part <= 4 ? 2 : part <= 8 ? 4 : part <= 32 ? 8 : 16, shift); }

// the first colour of level l, when its sweep from zero is csr_pre's
template <class T>
static FirstColour<T> first_colour(gl_precond *pre, int l)
{
    Level &Lv = pre->L[l];
    if (l >= pre->bottom || Lv.patch.np || Lv.ncolors < 2) return {};
    return {Lv.coff[1], dgn<T>(Lv), vec_t<T>(Lv)};
}

// Half a symmetric sweep: the colours in order (forward) or in reverse, those that
// other dispatches form left out (see SgsPass): of the first colour the forward value
// (the writer of b's, sgs_product's), of the last one the backward value
template <class T, int MODE>
static void sgs_half(Level &Lv, int shift, const int *gate, const Launch &L)
{
    constexpr bool fwd = MODE == SGS_FWD0 || MODE == SGS_FWD;
    const int nc = Lv.ncolors;
    const auto rows = [&](int c) { return Lv.coff[c + 1] - Lv.coff[c]; };
    const int k0 = fwd && nc == 1 ? 0 : 1;
    // algorithmic bytes: the entries of the part (index, value, gathered value), and
    // each row's own terms and results; the passes share one event bracket
    const double own = (MODE == SGS_FWD ? 4.0 : MODE == SGS_BWD0 ? 3.0 : 2.0) * sizeof(C<T>) + sizeof(T);
    const int left_out = k0 ? rows(fwd ? 0 : nc - 1) : 0;
    const double bytes = 0.5 * (Lv.Aa.nnz - Lv.n) * (4.0 + 2.0 * sizeof(C<T>)) + (Lv.n - left_out) * own;
    int passes = 0;
    for (int k = k0; k < nc; ++k) passes += rows(fwd ? k : nc - 1 - k) > 0;
    if (passes == 0) return;
    prof_launch(PROF_COARSE_SWEEP, bytes, L, [&] {
        for (int k = k0; k < nc; ++k) {
            const int c = fwd ? k : nc - 1 - k, W = Lv.ewidth[c], cnt = rows(c);
            if (cnt == 0) continue;
            const int lo = fwd ? 0 : std::min(W, Lv.eup[c]), hi = fwd ? Lv.elow[c] : W;
            const int lpr = sgs_lanes(hi - lo, shift);
            GLK_LPR_SWITCH(lpr, {
                L.run(blocks_for((int64_t)cnt * lpr),
                      SgsPass<T, LPR, MODE>{Lv.eci.get() + Lv.eoff[c], evals<T>(Lv) + Lv.eoff[c], W, lo, hi, Lv.coff[c],
                                            cnt, c == nc - 1, dgn<T>(Lv), vec_b<T>(Lv), vec_x<T>(Lv),
                                            vec_r<T>(Lv), vec_t<T>(Lv), gate});
            });
        }
    }, passes);
}

template <class T, int UP>
static void sgs_product(Level &Lv, int shift, const int *gate, const Launch &L)
{
    const int lpr = shifted(lanes_for(Lv.Aa, shift), -1), first = UP && Lv.ncolors > 1 ? Lv.coff[1] : 0;
    GLK_LPR_SWITCH(lpr, {
        L.run(blocks_for((int64_t)Lv.n * lpr),
              SgsProduct<T, LPR, UP>{Lv.n, first, Lv.Aa.rp.get(), Lv.Aa.ci.get(), Lv.dpos.get(), vals<T>(Lv.Aa),
                                     vec_b<T>(Lv), UP ? vec_x<T>(Lv) : vec_r<T>(Lv), dgn<T>(Lv),
                                     UP ? vec_r<T>(Lv) : vec_t<T>(Lv), vec_t<T>(Lv), gate});
    });
}

// x = sweep from zero; the residual in vec_t
template <class T>
static void csr_pre(Level &Lv, int shift, const int *gate, const Launch &L)
{
    sgs_half<T, SGS_FWD0>(Lv, shift, gate, L);
    sgs_half<T, SGS_BWD0>(Lv, shift, gate, L);
    sgs_product<T, 0>(Lv, shift, gate, L);
}

// a sweep of x
template <class T>
static void csr_post(Level &Lv, int shift, const int *gate, const Launch &L)
{
    sgs_product<T, 1>(Lv, shift, gate, L);
    sgs_half<T, SGS_FWD>(Lv, shift, gate, L);
    sgs_half<T, SGS_BWD>(Lv, shift, gate, L);
}

// ---- a level in patches
template <class T> static const C<T> *pvals(const PatchSet &S);
template <> const double2 *pvals<double>(const PatchSet &S) { return S.v64.get(); }
template <> const float2 *pvals<float>(const PatchSet &S) { return S.v32.get(); }

template <class T> static const C<T> *ppvals(const PatchSet &S);
template <> const double2 *ppvals<double>(const PatchSet &S) { return S.pv64.get(); }
template <> const float2 *ppvals<float>(const PatchSet &S) { return S.pv32.get(); }

// calls f with the patch arrays of the level's row width and patch size
template <class T, class F>
static void with_patch(const Level &Lv, F &&f)
{
    const PatchSet &S = Lv.patch;
    auto go = [&](auto w, auto nr) {
        constexpr int W = decltype(w)::value, NR = decltype(nr)::value;
        f(PatchArrays<T, W, NR>{S.size.get(), S.rowid.get(), S.info.get(), S.idx.get(), pvals<T>(S), dgn<T>(Lv),
                                Lv.ncolors, S.W},
          w, nr);
    };
    using std::integral_constant;
    if (S.rows == 512) {
        constexpr integral_constant<int, 512> nr{};
        if (S.W == 8) go(integral_constant<int, 8>{}, nr);
        else if (S.W == 12) go(integral_constant<int, 12>{}, nr);
        else go(integral_constant<int, 16>{}, nr);
    } else {
        constexpr integral_constant<int, 1024> nr{};
        if (S.W == 8) go(integral_constant<int, 8>{}, nr);
        else if (S.W == 12) go(integral_constant<int, 12>{}, nr);
        else go(integral_constant<int, 16>{}, nr);
    }
}

// algorithmic bytes of a sweep: the level's entries, b, the diagonal and x once
template <class T>
static double patch_bytes(const Level &Lv)
{
    return (double)Lv.Aa.nnz * (sizeof(C<T>) + 4.0) + Lv.n * (2.0 * sizeof(C<T>) + sizeof(T));
}

template <class T>
static void patch_pre(Level &Lv, const int *gate, const Launch &L)
{
    prof_launch(PROF_COARSE_SWEEP, patch_bytes<T>(Lv), L, [&] {
        with_patch<T>(Lv, [&](auto A, auto w, auto nr) {
            constexpr int W = decltype(w)::value, NR = decltype(nr)::value;
            L.run<PatchPre<T, W, NR>, NR>(Lv.patch.np,
                                          PatchPre<T, W, NR>{A, vec_b<T>(Lv), vec_x<T>(Lv), vec_r<T>(Lv), gate});
        });
    });
}

// result in vec_r
template <class T, class TX = T>
static void patch_post(Level &Lv, const C<TX> *xc, const int *gate, const Launch &L)
{
    prof_launch(PROF_COARSE_SWEEP, patch_bytes<T>(Lv), L, [&] {
        with_patch<T>(Lv, [&](auto A, auto w, auto nr) {
            constexpr int W = decltype(w)::value, NR = decltype(nr)::value;
            L.run<PatchPost<T, TX, W, NR>, NR>(
                Lv.patch.np, PatchPost<T, TX, W, NR>{A, vec_b<T>(Lv), vec_x<T>(Lv), Lv.patch.PW, Lv.patch.pci.get(),
                                                 ppvals<T>(Lv.patch), xc, vec_r<T>(Lv), gate});
        });
    });
}

// where the cycle leaves the iterate of level l
template <class T>
static C<T> *cycle_result(gl_precond *pre, int l)
{
    Level &Lv = pre->L[l];
    return l < pre->bottom && Lv.patch.np ? vec_r<T>(Lv) : vec_x<T>(Lv);
}

// The form of level 0 of a 2D grid: as gl_precond_set_tiles asked; with
// automatic tiles, tiles of 32 x 16.  Microseconds per MINRES
// iteration, a dispatch per pass / tiles, FP64: 513^2 147 / 136, 769^2 190 /
// 175, 1025^2 291 / 278, 1537^2 578 / 559, 2049^2 1058 / 1048 (smaller grids and
// FP32 gain more).
static int l0_form(const gl_precond *pre) { return pre->auto_tiles ? 2 : pre->l0_tiled; }

// calls f with the tile shape of gl_tiles.l0_tiled (1, 2 or 3)
template <class F>
static void l0_tiled_shape(int which, F &&f)
{
    if (which == 1) f(L0Shape1{});
    else if (which == 2) f(L0Shape2{});
    else f(L0Shape3{});
}

// T: level 0 (stencil sweeps, where the bytes are); TC: levels >= 1 and the
// coarsest solve (latency-bound: their precision costs no bandwidth)
// The V-cycle below level 0, from b of level 1 to x of level 1: the
// multi-kernel levels down (sweep from zero, residual, restriction), the
// small levels and the dense operator of level `tail` (the coarsest inverse
// or the explicit sub-cycle) in one work-group, or that dense product alone
// over many work-groups, then the multi-kernel levels up (prolongation,
// sweep).
template <class TC>
static void coarse_levels(gl_precond *pre, const int *gate, const Launch &L)
{
    const int nb_first = pre->bottom;
    const int sh = pre->lane_shift;
    for (int l = 1; l < nb_first; ++l) {
        Level &Lv = pre->L[l];
        if (Lv.patch.np) {
            patch_pre<TC>(Lv, gate, L);
        } else {
            csr_pre<TC>(Lv, sh, gate, L);
        }
        csr_spmv<TC>(Lv.Ra, Lv.patch.np ? vec_r<TC>(Lv) : vec_t<TC>(Lv), vec_b<TC>(pre->L[l + 1]), false, sh, gate, L,
                     first_colour<TC>(pre, l + 1));
    }
    if (pre->bottom < pre->tail) {
        L.run<Bottom<TC>, kBottomThreads>(1, Bottom<TC>{bdesc<TC>(pre), gate}, bottom_lds<TC>(pre));
    } else {
        Level &Lc = pre->L[pre->tail];
        L.run(blocks_for((int64_t)Lc.n * 64),
              DenseApply<TC>{Lc.n, cinv<TC>(pre), vec_b<TC>(Lc), vec_x<TC>(Lc), gate});
    }
    for (int l = nb_first - 1; l >= 1; --l) {
        Level &Lv = pre->L[l];
        const C<TC> *xc = cycle_result<TC>(pre, l + 1);
        if (Lv.patch.np) {
            patch_post<TC>(Lv, xc, gate, L);
        } else {
            csr_spmv<TC>(Lv.Pa, xc, vec_x<TC>(Lv), true, sh, gate, L);
            csr_post<TC>(Lv, sh, gate, L);
        }
    }
}

// the totals of the output kernel's partials: Re<vdot, z> and, when asked, <u, z>_R
static void finish_dots(RedSlot slot, int nb, int mode, KrylovScalars *ks, double *store, const DeflDot &dd,
                        const int *gate, const Launch &L)
{
    const FinTask a{slot.partials, mode, store};
    launch_finalize2(a, dd.psi ? FinTask{dd.slot.partials, FIN_DEFL_Y, nullptr} : FinTask{}, nb, ks, gate, L);
}

DeflDot defl_dot(const gl_mesh *m, const double2 *psi)
{
    DeflDot d;
    d.psi = psi;
    d.vol = m->g.vol64;
    for (int a = 0; a < 3; ++a) {
        d.N[a] = m->g.N[a];
        d.h[a] = m->g.h[a];
    }
    d.slot = red_slot(m, 3);
    return d;
}

template <int DIM, class T, class TC>
static void vcycle_once_grid(const gl_precond *cpre, const double2 *v, const double2 *vdot, double2 *z,
                        const int *gate, KrylovScalars *ks, int mode, int add, const Launch &L,
                        double *store, const DeflDot &dd)
{
    gl_precond *pre = const_cast<gl_precond *>(cpre);
    const gl_mesh *m = pre->mesh;
    const GeomT<T> g = geom_t<T>(m->g);
    const LinkTab<T> U = link_tab<T>(m);
    const RedSlot slot = red_slot(m, 1);
    Level &L0 = pre->L[0];
    const int n0 = L0.n, nb0 = blocks_for(n0);
    const int nl = pre->nlev;
    const bool f32 = std::is_same<T, float>::value;
    C<T> *b0 = vec_b<T>(L0);
    C<T> *x0 = vec_x<T>(L0);
    // Re<vdot, z> is reduced for the Krylov scalars (ks) or stored (store)
    const int want = ks != nullptr || store != nullptr;
    const int fmode = store ? (int)FIN_STORE : mode;
    if (nl == 1) {
        C<TC> *xc0 = vec_x<TC>(L0);
        L.run(nb0, Narrow<TC>{n0, v, vec_b<TC>(L0), gate});
        L.run(blocks_for((int64_t)n0 * 64), DenseApply<TC>{n0, cinv<TC>(pre), vec_b<TC>(L0), xc0, gate});
        if (add) L.run(nb0, Output<DIM, TC, 1>{n0, xc0, vdot, z, slot, want, dd, gate});
        else L.run(nb0, Output<DIM, TC, 0>{n0, xc0, vdot, z, slot, want, dd, gate});
        if (want) finish_dots(slot, nb0, fmode, ks, store, dd, gate, L);
        return;
    }
    const T *hd = diag<T>(L0), *hs = hsplit<T>(L0);
    Level &L1 = pre->L[1];
    // algorithmic bytes of the level-0 kernels (each array touched once)
    // (the link factor tables are a few KB and stay in cache)
    const double sz = sizeof(C<T>), szr = sizeof(T), nn = n0, mc = 0.5 * nn;
    const double b_pre = nn * 16 + nn * sz + nn * szr + mc * sz;
    const double b_sweep = mc * (sz + szr + sz) + (nn - mc) * sz;
    const double b_resid = b_sweep + (nn - mc) * sz;
    const double szc = sizeof(C<TC>);
    const double b_prol = (g.npair + 1 + L0.Pb.nnz) * 4.0 + L0.Pb.nnz * szc + L0.nc * szc + 2.0 * mc * sz;
    const double b_last = b_sweep - mc * sz + (nn - mc) * sz + nn * 16 * (want ? 2 : 1) + (add ? nn * 16 : 0);
    const double b_restr = (L0.nc + 1 + L0.Rb.nnz) * 4.0 + L0.Rb.nnz * szc + (nn - mc) * sz + L0.nc * szc;
    // level 0 (one thread per red-black pair), down: red (from zero, folded) +
    // black, red, black residual, restriction; in 2D by default the three
    // passes in one LDS-tiled kernel (L0PreTile)
    const int nbp = blocks_for(g.npair);
    const int tiled = DIM == 2 ? l0_form(pre) : 0;
    if (tiled) {
        // each array once (the halo's re-reads come from cache)
        const double b_tile = nn * 16 + nn * szr + 2 * nn * sz + mc * sz;
        prof_launch(PROF_L0_SWEEP, b_tile, L, [&] {
            l0_tiled_shape(tiled, [&](auto sh) {
                using S = decltype(sh);
                const int ntx = (g.N[0] + S::TX - 1) / S::TX, nbt = ntx * ((g.N[1] + S::TY - 1) / S::TY);
                L.run<L0PreTile<T, S>, S::threads>(nbt,
                                                   L0PreTile<T, S>{g, v, hs, U, vec_b<T>(L0), x0, vec_r<T>(L0), ntx, gate});
            });
        });
    } else {
        prof_launch(PROF_L0_SWEEP, b_pre, L, [&] {
            L.run(nbp, L0PreBlack<DIM, T>{g, v, vec_b<T>(L0), x0, U, hd, gate});
        });
        prof_launch(PROF_L0_SWEEP, b_sweep, L, [&] {
            L.run(nbp, L0Sweep<DIM, T>{g, 0, b0, x0, U, hs, gate});
        });
        prof_launch(PROF_L0_RESIDUAL, b_resid, L, [&] {
            L.run(nbp, L0Residual<DIM, T>{g, b0, x0, U, hs, vec_r<T>(L0), gate});
        });
    }
    prof_launch(PROF_L0_TRANSFER, b_restr, L, [&] {
        csr_spmv<TC, T>(L0.Rb, vec_r<T>(L0), vec_b<TC>(L1), false, 0, gate, L, first_colour<TC>(pre, 1));
    });
    // levels >= 1: b of level 1 in, x of level 1 out
    coarse_levels<TC>(pre, gate, L);
    const C<TC> *x1 = cycle_result<TC>(pre, 1);
    // level 0, up: red with the coarse correction, black, red + output
    // black coarse correction, then the red pass (fusing the two reads every
    // black correction four times and was measured slower); in 2D by default
    // all four in one LDS-tiled kernel (L0PostTile), each tile correcting the
    // black nodes of its halo once
    if (tiled) {
        const double b_tile = (g.npair + 1 + L0.Pb.nnz) * 4.0 + L0.Pb.nnz * szc + L0.nc * szc + mc * sz +
                              nn * sz + nn * szr + nn * 16 * (want ? 2 : 1) + (add ? nn * 16 : 0);
        int nbt = 0;
        prof_launch(PROF_L0_SWEEP, b_tile, L, [&] {
            l0_tiled_shape(tiled, [&](auto sh) {
                using S = decltype(sh);
                const int ntx = (g.N[0] + S::TX - 1) / S::TX;
                nbt = ntx * ((g.N[1] + S::TY - 1) / S::TY);
                if (add)
                    L.run<L0PostTile<T, TC, 1, S>, S::threads>(
                        nbt, L0PostTile<T, TC, 1, S>{g, b0, x0, hs, U, L0.Pb.rp.get(), L0.Pb.ci.get(), vals<TC>(L0.Pb),
                                                     x1, z, vdot, slot, want, dd, ntx, gate});
                else
                    L.run<L0PostTile<T, TC, 0, S>, S::threads>(
                        nbt, L0PostTile<T, TC, 0, S>{g, b0, x0, hs, U, L0.Pb.rp.get(), L0.Pb.ci.get(), vals<TC>(L0.Pb),
                                                     x1, z, vdot, slot, want, dd, ntx, gate});
            });
        });
        if (want) finish_dots(slot, nbt, fmode, ks, store, dd, gate, L);
        return;
    }
    prof_launch(PROF_L0_TRANSFER, b_prol, L, [&] {
        L.run(nbp, L0ProlongBlack<DIM, T, TC>{g, x0, L0.Pb.rp.get(), L0.Pb.ci.get(), vals<TC>(L0.Pb), x1, gate});
    });
    prof_launch(PROF_L0_SWEEP, b_sweep, L, [&] {
        L.run(nbp, L0Sweep<DIM, T>{g, 0, b0, x0, U, hs, gate});
    });
    prof_launch(PROF_L0_SWEEP, b_sweep, L, [&] {
        L.run(nbp, L0Sweep<DIM, T>{g, 1, b0, x0, U, hs, gate});
    });
    prof_launch(PROF_L0_SWEEP, b_last, L, [&] {
        if (add) L.run(nbp, L0Last<DIM, T, 1>{g, b0, x0, U, hs, z, vdot, slot, want, dd, gate});
        else L.run(nbp, L0Last<DIM, T, 0>{g, b0, x0, U, hs, z, vdot, slot, want, dd, gate});
    });
    if (want) finish_dots(slot, nbp, fmode, ks, store, dd, gate, L);
}

// Level 0 of a simplicial mesh is a CSR level like the coarse ones: its
// rows in colour order (perm), padded colour blocks for the sweeps, the full
// restriction and prolongation.
template <class T, class TC>
static void vcycle_once_simplicial(const gl_precond *cpre, const double2 *v, const double2 *vdot, double2 *z,
                                   const int *gate, KrylovScalars *ks, int mode, int add, const Launch &L,
                                   double *store, const DeflDot &dd)
{
    gl_precond *pre = const_cast<gl_precond *>(cpre);
    const gl_mesh *m = pre->mesh;
    const RedSlot slot = red_slot(m, 1);
    Level &L0 = pre->L[0];
    const int n0 = L0.n, nb0 = blocks_for(n0);
    const int want = ks != nullptr || store != nullptr;
    const int fmode = store ? (int)FIN_STORE : mode;
    if (pre->nlev == 1) {  // the coarsest inverse in node order
        C<TC> *xc0 = vec_x<TC>(L0);
        L.run(nb0, Narrow<TC>{n0, v, vec_b<TC>(L0), gate});
        L.run(blocks_for((int64_t)n0 * 64), DenseApply<TC>{n0, cinv<TC>(pre), vec_b<TC>(L0), xc0, gate});
        if (add) L.run(nb0, Output<0, TC, 1>{n0, xc0, vdot, z, slot, want, dd, gate});
        else L.run(nb0, Output<0, TC, 0>{n0, xc0, vdot, z, slot, want, dd, gate});
        if (want) finish_dots(slot, nb0, fmode, ks, store, dd, gate, L);
        return;
    }
    Level &L1 = pre->L[1];
    const int sh = pre->lane_shift;
    const int *perm = L0.perm.get();
    C<T> *x0 = vec_x<T>(L0);
    L.run(nb0, NarrowPerm<T>{n0, v, perm, vec_b<T>(L0), first_colour<T>(pre, 0), gate});
    if (L0.patch.np) {
        patch_pre<T>(L0, gate, L);
    } else {
        csr_pre<T>(L0, sh, gate, L);
    }
    csr_spmv<TC, T>(L0.Ra, L0.patch.np ? vec_r<T>(L0) : vec_t<T>(L0), vec_b<TC>(L1), false, sh, gate, L,
                    first_colour<TC>(pre, 1));
    coarse_levels<TC>(pre, gate, L);
    const C<TC> *x1 = cycle_result<TC>(pre, 1);
    if (L0.patch.np) {
        patch_post<T, TC>(L0, x1, gate, L);
        x0 = vec_r<T>(L0);
    } else {
        csr_spmv<T, TC>(L0.Pa, x1, x0, true, sh, gate, L);
        csr_post<T>(L0, sh, gate, L);
    }
    if (add) L.run(nb0, OutputPerm<T, 1>{n0, x0, perm, vdot, z, slot, want, dd, gate});
    else L.run(nb0, OutputPerm<T, 0>{n0, x0, perm, vdot, z, slot, want, dd, gate});
    if (want) finish_dots(slot, nb0, fmode, ks, store, dd, gate, L);
}

// One V-cycle on H x = D v from x = 0 (DIM 0: a simplicial mesh)
template <int DIM, class T, class TC>
static void vcycle_once(const gl_precond *cpre, const double2 *v, const double2 *vdot, double2 *z,
                        const int *gate, KrylovScalars *ks, int mode, int add, const Launch &L,
                        double *store = nullptr, const DeflDot &dd = DeflDot{})
{
    if constexpr (DIM == 0) vcycle_once_simplicial<T, TC>(cpre, v, vdot, z, gate, ks, mode, add, L, store, dd);
    else vcycle_once_grid<DIM, T, TC>(cpre, v, vdot, z, gate, ks, mode, add, L, store, dd);
}

// ------------------------------------------------------------- R_inf ---
// R_inf = H^-1 (eq. prec1; the scaled form of H^-1 D): preconditioned
// conjugate gradients on H x = v from x = 0 with one V-cycle per step, run
// for a fixed number m of steps (chosen at each setup, pcg_calibrate), so
// that the operator is a fixed linear map to the calibration's accuracy and
// the steps can be captured in the MINRES iteration graph.  Scalars of step
// j live at fixed places: rz[j] = <r_j, z_j>, pq[j] = <p_j, H p_j>.

// q = H p (level 0 as the FP64 stencil with its diagonal), partials of Re<p, q>
template <int DIM>
struct PcgHp {
    GeomT<double> g;
    const double2 *p;
    LinkTab<double> U;
    const double *hd;
    double2 *q;
    RedSlot slot;
    const int *gate;
    __device__ void operator()(int bx, int nbx) const
    {
        GATE();
        __shared__ double sm[kBlock / 64];
        const int i = xcd_tile(bx, nbx) * kBlock + threadIdx.x;
        double part = 0.0;
        if (i < g.n) {
            int c[3];
            node_coords<DIM>(g.N, i, c);
            const double2 pi = p[i];
            const double2 qi = cadd(khat_offdiag<DIM, double>(g, i, c, p, U), cscale(pi, hd[i]));
            q[i] = qi;
            part = redot(pi, qi);
        }
        block_reduce_store(part, slot, sm, bx);
    }
};

// x += alpha p (x = alpha p at the first step), r -= alpha q, alpha = rz / pq
// (0 when pq is not positive: nothing left to reduce); partials of |r|^2
// when asked (calibration)
struct PcgStep {
    int n;
    const double2 *p, *q;
    double2 *x, *r;
    const double *rz, *pq;
    int first;
    RedSlot slot;
    int want_rr;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE();
        __shared__ double sm[kBlock / 64];
        const double den = *pq;
        const double alpha = den > 0.0 ? *rz / den : 0.0;
        const int i = bx * kBlock + threadIdx.x;
        double part = 0.0;
        if (i < n) {
            const double2 pi = p[i], qi = q[i];
            x[i] = first ? cscale(pi, alpha) : cadd(x[i], cscale(pi, alpha));
            const double2 ri = csub(r[i], cscale(qi, alpha));
            r[i] = ri;
            part = cabs2(ri);
        }
        if (want_rr) block_reduce_store(part, slot, sm, bx);
    }
};

// p = z + beta p, beta = rz_new / rz (0 when rz is not positive)
struct PcgDir {
    int n;
    const double2 *z;
    double2 *p;
    const double *rz, *rz_new;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE();
        const double den = *rz;
        const double beta = den > 0.0 ? *rz_new / den : 0.0;
        const int i = bx * kBlock + threadIdx.x;
        if (i < n) p[i] = cadd(z[i], cscale(p[i], beta));
    }
};

// partials of |r|^2 (calibration)
struct PcgNorm {
    int n;
    const double2 *r;
    RedSlot slot;
    __device__ void operator()(int bx, int) const
    {
        __shared__ double sm[kBlock / 64];
        const int i = bx * kBlock + threadIdx.x;
        block_reduce_store(i < n ? cabs2(r[i]) : 0.0, slot, sm, bx);
    }
};

// r = v (the first residual, x = 0)
struct PcgInit {
    int n;
    const double2 *v;
    double2 *r;
    const int *gate;
    __device__ void operator()(int bx, int) const
    {
        GATE();
        const int i = bx * kBlock + threadIdx.x;
        if (i < n) r[i] = v[i];
    }
};

struct PcgBufs {
    double2 *x, *r, *p, *q, *z;
    double *rz, *pq;
};

static PcgBufs pcg_bufs(const gl_precond *pre)
{
    gl_precond *p = const_cast<gl_precond *>(pre);
    const size_t n = (size_t)pre->L[0].n;
    double2 *b = p->pcg.get();
    double *sc = p->pcg_sc.get();
    return PcgBufs{b, b + n, b + 2 * n, b + 3 * n, b + 4 * n, sc, sc + kPcgMaxSteps + 1};
}

// m steps of CG; z = x with the Krylov partials of Re<vdot, z> when ks is set
template <int DIM, class T, class TC>
static void vcycle_pcg(const gl_precond *pre, const double2 *v, double2 *z, const int *gate, KrylovScalars *ks,
                       int mode, const Launch &L, const DeflDot &dd)
{
    const gl_mesh *m = pre->mesh;
    const GeomT<double> g = geom_t<double>(m->g);
    const int n = pre->L[0].n, nb = blocks_for(n);
    const PcgBufs B = pcg_bufs(pre);
    const int steps = std::max(1, pre->pcg_m);
    const RedSlot hslot = red_slot(m, 0);
    L.run(nb, PcgInit{n, v, B.r, gate});
    // z_0 = V(r_0) straight into p_0
    vcycle_once<DIM, T, TC>(pre, B.r, B.r, B.p, gate, nullptr, 0, 0, L, B.rz);
    for (int j = 0; j < steps; ++j) {
        L.run(nb, PcgHp<DIM>{g, B.p, link_tab<double>(m), pre->L[0].diag64.get(), B.q, hslot, gate});
        launch_finalize(hslot.partials, nb, FIN_STORE, nullptr, B.pq + j, gate, L);
        L.run(nb, PcgStep{n, B.p, B.q, B.x, B.r, B.rz + j, B.pq + j, j == 0, hslot, 0, gate});
        if (j + 1 < steps) {
            vcycle_once<DIM, T, TC>(pre, B.r, B.r, B.z, gate, nullptr, 0, 0, L, B.rz + j + 1);
            L.run(nb, PcgDir{n, B.z, B.p, B.rz + j, B.rz + j + 1, gate});
        }
    }
    const RedSlot slot = red_slot(m, 1);
    L.run(nb, Output<DIM, double, 0>{n, B.x, v, z, slot, ks != nullptr, dd, gate});
    if (ks) finish_dots(slot, nb, mode, ks, nullptr, dd, gate, L);
}

template <int DIM>
static void pcg_calibrate_dim(gl_precond *pre, hipStream_t s)
{
    // CG from a seeded counter-hash right-hand side with the norm of the
    // residual read after every step: m = the steps to 1e-12, plus 2
    const gl_mesh *m = pre->mesh;
    const GeomT<double> g = geom_t<double>(m->g);
    const int n = pre->L[0].n, nb = blocks_for(n);
    const PcgBufs B = pcg_bufs(pre);
    const RedSlot hslot = red_slot(m, 0), rslot = red_slot(m, 2);
    double2 *v = pre->vin.get();
    k_hash_rhs<<<nb, kBlock, 0, s>>>(n, v);
    GLK_CHECK_LAUNCH();
    const Launch L{s};
    double *rr = m->dscal.get() + 8;
    auto host_rr = [&]() {
        double h = 0.0;
        GLK_HIP(hipMemcpyAsync(&h, rr, sizeof(double), hipMemcpyDeviceToHost, s));
        GLK_HIP(hipStreamSynchronize(s));
        return h;
    };
    L.run(nb, PcgInit{n, v, B.r, nullptr});
    L.run(nb, PcgNorm{n, B.r, rslot});
    launch_finalize(rslot.partials, nb, FIN_STORE, nullptr, rr, nullptr, L);
    const double rr0 = host_rr();
    vcycle_once<DIM, double, double>(pre, B.r, B.r, B.p, nullptr, nullptr, 0, 0, L, B.rz);
    int steps = kPcgMaxSteps;
    for (int j = 0; j < kPcgMaxSteps; ++j) {
        L.run(nb, PcgHp<DIM>{g, B.p, link_tab<double>(m), pre->L[0].diag64.get(), B.q, hslot, nullptr});
        launch_finalize(hslot.partials, nb, FIN_STORE, nullptr, B.pq + j, nullptr, L);
        L.run(nb, PcgStep{n, B.p, B.q, B.x, B.r, B.rz + j, B.pq + j, j == 0, rslot, 1, nullptr});
        launch_finalize(rslot.partials, nb, FIN_STORE, nullptr, rr, nullptr, L);
        if (!(host_rr() > 1e-24 * rr0)) {
            steps = std::min(kPcgMaxSteps, j + 1 + 2);
            break;
        }
        if (j + 1 < kPcgMaxSteps) {
            vcycle_once<DIM, double, double>(pre, B.r, B.r, B.z, nullptr, nullptr, 0, 0, L, B.rz + j + 1);
            L.run(nb, PcgDir{n, B.z, B.p, B.rz + j, B.rz + j + 1, nullptr});
        }
    }
    pre->pcg_m = steps;
}

void pcg_calibrate(gl_precond *pre, hipStream_t s)
{
    const size_t n = (size_t)pre->L[0].n;
    if (pre->pcg.count < 5 * n) pre->pcg.alloc(5 * n);
    if (pre->pcg_sc.count < 2 * kPcgMaxSteps + 2) pre->pcg_sc.alloc(2 * kPcgMaxSteps + 2);
    with_dim(pre->mesh->g, [&](auto D) { pcg_calibrate_dim<decltype(D)::value>(pre, s); });
}

template <int DIM, class T, class TC>
static void vcycle_k(const gl_precond *pre, const double2 *v, double2 *z, const int *gate,
                     KrylovScalars *ks, int mode, const Launch &L, const DeflDot &dd)
{
    const int k = pre->opts.cycles;
    if (k == 0) {
        vcycle_pcg<DIM, T, TC>(pre, v, z, gate, ks, mode, L, dd);
        return;
    }
    if (k <= 1) {
        vcycle_once<DIM, T, TC>(pre, v, v, z, gate, ks, mode, 0, L, nullptr, dd);
        return;
    }
    // x <- x + V(v - H x), k times from x = 0
    const gl_mesh *m = pre->mesh;
    const GeomT<double> g = geom_t<double>(m->g);
    const int nb0 = blocks_for(pre->L[0].n);
    vcycle_once<DIM, T, TC>(pre, v, v, z, gate, nullptr, 0, 0, L);
    for (int c = 1; c < k; ++c) {
        L.run(nb0, L0ResidualFull<DIM>{g, v, z, link_tab<double>(m), pre->L[0].diag64.get(), pre->cyc_r.get(),
                                       gate});
        const bool lastc = (c == k - 1);
        vcycle_once<DIM, T, TC>(pre, pre->cyc_r.get(), v, z, gate, lastc ? ks : nullptr, mode, 1, L, nullptr,
                                lastc ? dd : DeflDot{});
    }
}

// The split of the levels while a solve's V-cycles are enqueued
struct SolverSplit {
    gl_precond *p;
    const int bottom, tail;
    SolverSplit(const gl_precond *pre, bool solver)
        : p(const_cast<gl_precond *>(pre)), bottom(pre->bottom), tail(pre->tail)
    {
        if (solver && pre->stail) p->bottom = p->tail = pre->stail;
    }
    ~SolverSplit()
    {
        p->bottom = bottom;
        p->tail = tail;
    }
};

void vcycle_enqueue(const gl_precond *pre, const double2 *v, double2 *z, const int *gate,
                    KrylovScalars *ks, int mode, const Launch &L, gl_precision p, const DeflDot &dd, bool solver)
{
    const SolverSplit split(pre, solver);
    with_dim(pre->mesh->g, [&](auto D) {
        constexpr int K = decltype(D)::value;
        if (p == GL_FP32) vcycle_k<K, float, float>(pre, v, z, gate, ks, mode, L, dd);
        else if (p == GL_MIXED) vcycle_k<K, float, double>(pre, v, z, gate, ks, mode, L, dd);
        else vcycle_k<K, double, double>(pre, v, z, gate, ks, mode, L, dd);
    });
}

void vcycle_enqueue(const gl_precond *pre, const double2 *v, double2 *z, const int *gate,
                    KrylovScalars *ks, int mode, const Launch &L)
{
    vcycle_enqueue(pre, v, z, gate, ks, mode, L, pre->opts.precision, DeflDot{}, false);
}

// The level whose sub-cycle a solve applies as an explicit matrix with
// automatic tiles (0: none): the one that saves most over
// kSolverCycles V-cycles, its formation counted.  Microseconds, from
// measurements: a level in patches 30, else 3.2 per dispatch of its 4 C, or 1.4
// per step inside the bottom kernel; a dense product 4 and its bytes at 4 TB/s;
// the formation 3 per step of the cycle, and its gathers, about 46 bytes per
// column and stored entry, at 7 TB/s (545 rows: 0.17 ms for 29 us a cycle; 195
// rows: 0.04 for 16; 5 592 rows of 31 colours: 12 ms for 270 us, not taken).
// The choice hardly depends on the cycles assumed: 12 to 200 give the same levels on
// all of 15 grids and domains measured (65^2-1025^2, 17x4001, 49^3-129^3, discs,
// tetrahedra), 6 gives up the sub-cycles of 1247, 1540 and 1387 rows (257^2, 8 / 24 /
// 152 iterations 1.47 / 2.41 / 10.22 ms with 24, 1.44 / 2.54 / 11.89 with 6).  2048
// rows keep matrix and workspace under 0.35 GB a handle; the sub-cycle of 2561 rows
// (97^3) would take 0.55 GB and 18.7 ms for 24 iterations, 26.0 without.
constexpr int kSolverCycles = 24, kSolverTail = 2048;

static int solver_tail(const gl_precond *pre)
{
    const int last = pre->nlev - 1;
    if (!pre->auto_tiles || pre->tail < last) return 0;
    int best = 0;
    double best_gain = 0.0;
    double saved = 4.0, steps = 3.0, nnz = (double)pre->L[last].n * pre->L[last].n;
    for (int l = last - 1; l >= 1; --l) {
        const Level &L = pre->L[l];
        if (L.n > kSolverTail || L.ncolors > kMaxColors) break;
        saved += l >= pre->bottom ? 1.4 * (4 * L.ncolors + 1) : L.patch.np ? 30.0 : 3.2 * 4 * L.ncolors;
        steps += 4 * L.ncolors + 3;
        nnz += L.A.nnz;
        const double dense = 4.0 + 16.0 * L.n * (double)L.n / 4e6;
        const double form = 3.0 * steps + 46.0 * L.n * nnz / 7e6;
        const double gain = kSolverCycles * (saved - dense) - form;
        if (gain > best_gain) {
            best = l;
            best_gain = gain;
        }
    }
    return best;
}

// Device descriptors of the bottom levels (pointers fixed after setup).
template <class T>
static void fill_bottom(gl_precond *pre, BottomDesc<T> &D)
{
    std::memset(&D, 0, sizeof(D));
    D.first = pre->bottom;
    D.last = pre->tail;
    D.cinv = cinv<T>(pre);
    for (int l = 1; l < pre->nlev; ++l) {
        Level &L = pre->L[l];
        BottomLevel<T> &B = D.L[l];
        B.n = L.n;
        B.nc = L.nc;
        B.ncolors = L.ncolors;
        B.rp = L.Aa.rp.get();
        B.ci = L.Aa.ci.get();
        B.dpos = L.dpos.get();
        B.v = vals<T>(L.Aa);
        B.diag = dgn<T>(L);
        for (int c = 0; c <= L.ncolors && c <= kMaxColors && c < (int)L.coff.size(); ++c) B.coff[c] = L.coff[c];
        if (l + 1 < pre->nlev) {
            B.prp = L.Pa.rp.get();
            B.pci = L.Pa.ci.get();
            B.pv = vals<T>(L.Pa);
            B.rrp = L.Ra.rp.get();
            B.rci = L.Ra.ci.get();
            B.rv = vals<T>(L.Ra);
        }
        B.b = vec_b<T>(L);
        B.x = vec_x<T>(L);
        B.r = vec_r<T>(L);
        B.eci = L.eci.get();
        B.ev = evals<T>(L);
        for (int c = 0; c < L.ncolors && c < kMaxColors && c < (int)L.ewidth.size(); ++c) {
            B.ewidth[c] = L.ewidth[c];
            B.eoff[c] = L.eoff[c];
        }
    }
    // the first bottom level keeps its iterate in LDS when it fits
    D.lds_level = -1;
    if (D.first < D.last) {
        int dev = 0, lmax = 0;
        GLK_HIP(hipGetDevice(&dev));
        GLK_HIP(hipDeviceGetAttribute(&lmax, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
        const size_t need = (size_t)pre->L[D.first].n * sizeof(C<T>);
        if (need + 1024 <= (size_t)lmax) D.lds_level = D.first;
    }
}

// memory of the explicit sub-cycle of level ex
static void tail_matrix(gl_precond *pre, int ex)
{
    const size_t nt = (size_t)pre->L[ex].n;
    if (pre->tinv64.count < nt * nt) pre->tinv64.alloc(nt * nt);
    if (pre->tinv32.count < nt * nt) pre->tinv32.alloc(nt * nt);
}

static int tail_blocks(const gl_precond *pre, int ex) { return (pre->L[ex].n + kTailBlock - 1) / kTailBlock; }

// blocks of columns that one launch forms at most: as many as the workspace bound allows
static int tail_fit(const gl_precond *pre, int ex)
{
    const size_t fit = kTailWorkspace / (pre->tws_col * sizeof(double2));
    return (int)std::max<size_t>(1, std::min<size_t>(tail_blocks(pre, ex), fit));
}

// the handle's own workspace for forming it
static TailSpace tail_workspace(gl_precond *pre, int ex)
{
    const int blocks = tail_fit(pre, ex);
    if (pre->tws.count < pre->tws_col * blocks) pre->tws.alloc(pre->tws_col * blocks);
    return TailSpace{pre->tws.get(), blocks};
}

void bottom_descriptors(gl_precond *pre, hipStream_t s)
{
    const int last = pre->nlev - 1;
    // level with an explicit sub-cycle: the first l >= 1 with at most
    // dense_rows rows and a bottom-kernel colouring (the coarsest if none)
    int tail = last;
    if (pre->dense_rows > 0)
        for (int l = 1; l < last; ++l) {
            const Level &L = pre->L[l];
            if (L.n <= pre->dense_rows) {
                bool fits = true;
                for (int q = l; q < last; ++q) fits = fits && pre->L[q].ncolors <= kMaxColors;
                if (fits) tail = l;
                break;
            }
        }
    pre->tail = tail;
    // first level of the bottom kernel: the smallest l >= 1 from which every
    // level above the tail fits (size and colour count); a single-level
    // hierarchy is just the dense solve on level 0.  One work-group applies
    // an explicit sub-cycle only up to kBottomDenseRows rows: a larger one is
    // a product for many work-groups, so no level goes to the bottom kernel.
    int first = tail;
    if (tail == last || pre->L[tail].n <= kBottomDenseRows)
        for (int l = tail - 1; l >= 1; --l) {
            const Level &L = pre->L[l];
            if (L.n > pre->bottom_rows || L.ncolors > kMaxColors) break;
            first = l;
        }
    // a level in patches takes two dispatches whatever its size and stays out
    // of the bottom kernel (106 rows of 9 colours above a dense one of 8: 17 us
    // with its transfers and the dense product; 49 us in the bottom kernel)
    while (first < tail && pre->L[first].patch.np) ++first;
    pre->bottom = first;
    pre->stail = solver_tail(pre);
    pre->stail_current = false;
    pre->tinv64.release();
    pre->tinv32.release();
    pre->tws.release();
    pre->tws_col = 0;
    if (const int ex = tail < last ? tail : pre->stail) {  // the level with an explicit sub-cycle
        size_t col = 0;
        for (int l = ex; l <= last; ++l) col += tail_vectors(l == ex, l == last) * (size_t)pre->L[l].n;
        pre->tws_col = col * kTailBlock;  // elements per block of columns
        if (ex == tail) {
            // (a solve's is allocated by the first solve: a handle may serve applications only)
            tail_matrix(pre, ex);
            tail_workspace(pre, ex);
        }
        // formation: levels ex .. coarsest with the coarsest inverse
        BottomDesc<double> dt;
        const int keep = pre->tail;
        pre->tail = last;
        const int keep_b = pre->bottom;
        pre->bottom = ex;
        fill_bottom<double>(pre, dt);
        pre->tail = keep;
        pre->bottom = keep_b;
        dt.lds_level = -1;
        pre->tdesc64.alloc(sizeof(dt));
        GLK_HIP(hipMemcpyAsync(pre->tdesc64.get(), &dt, sizeof(dt), hipMemcpyHostToDevice, s));
    } else {
        pre->tdesc64.release();
    }
    BottomDesc<double> d64;
    BottomDesc<float> d32;
    fill_bottom<double>(pre, d64);
    fill_bottom<float>(pre, d32);
    pre->lds64 = d64.lds_level >= 0 ? (int)(pre->L[d64.lds_level].n * sizeof(double2)) : 0;
    pre->lds32 = d32.lds_level >= 0 ? (int)(pre->L[d32.lds_level].n * sizeof(float2)) : 0;
    pre->bdesc64.alloc(sizeof(d64));
    pre->bdesc32.alloc(sizeof(d32));
    GLK_HIP(hipMemcpyAsync(pre->bdesc64.get(), &d64, sizeof(d64), hipMemcpyHostToDevice, s));
    GLK_HIP(hipMemcpyAsync(pre->bdesc32.get(), &d32, sizeof(d32), hipMemcpyHostToDevice, s));
    GLK_HIP(hipStreamSynchronize(s));
}

// The explicit sub-cycle of level `tail` from the current values: FP64
// columns, kTailBlock per work-group and as many work-groups per launch as
// the workspace holds, then the FP32 copy.
static void tail_columns(gl_precond *pre, int ex, const TailSpace &ws, const Launch &L)
{
    const int nt = pre->L[ex].n;
    const auto *D = reinterpret_cast<const BottomDesc<double> *>(pre->tdesc64.get());
    const int nblk = tail_blocks(pre, ex);
    for (int b0 = 0; b0 < nblk; b0 += ws.blocks) {
        const int nb = std::min(ws.blocks, nblk - b0);
        L.run<TailColumns<double>, kTailThreads>(
            nb, TailColumns<double>{D, ws.p, pre->tws_col, b0 * kTailBlock, nb, pre->tinv64.get()});
    }
    const int64_t nn = (int64_t)nt * nt;
    L.run(blocks_for(nn), Narrow<float>{(int)nn, pre->tinv64.get(), pre->tinv32.get(), nullptr});
}

void form_tail(gl_precond *pre, hipStream_t s)
{
    if (pre->has_values && pre->tail < pre->nlev - 1)
        tail_columns(pre, pre->tail, tail_workspace(pre, pre->tail), Launch{s});
}

// f, which allocates for the explicit sub-cycle of solves on pre: where there is no
// memory for it, solves on the handle do without
template <class F>
static bool tail_allocates(gl_precond *pre, F &&f)
{
    try {
        f();
        return true;
    } catch (const Error &e) {
        if (e.status != GL_ERR_OUT_OF_MEMORY) throw;
    }
    (void)hipGetLastError();
    pre->tinv64.release();
    pre->tinv32.release();
    pre->tws.release();
    pre->stail = 0;
    pre->uid = new_precond_uid();
    return false;
}

size_t solver_tail_space(const gl_precond *cpre, size_t most, int *blocks)
{
    gl_precond *pre = const_cast<gl_precond *>(cpre);
    if (!pre->stail || pre->stail_current) return 0;
    if (!tail_allocates(pre, [&] { tail_matrix(pre, pre->stail); })) return 0;
    *blocks = (int)std::max<size_t>(1, std::min<size_t>(tail_fit(pre, pre->stail), most / pre->tws_col));
    return pre->tws_col * *blocks;
}

void solver_tail_enqueue(const gl_precond *cpre, const Launch &L, const TailSpace &shared)
{
    gl_precond *pre = const_cast<gl_precond *>(cpre);
    if (!pre->stail || pre->stail_current) return;
    TailSpace ws = shared;
    if (!ws.p && !tail_allocates(pre, [&] {
            tail_matrix(pre, pre->stail);
            ws = tail_workspace(pre, pre->stail);
        }))
        return;
    tail_columns(pre, pre->stail, ws, L);
    pre->stail_current = true;
}

void solver_tail_drop(const gl_precond *cpre)
{
    gl_precond *pre = const_cast<gl_precond *>(cpre);
    tail_allocates(pre, [] { fail(GL_ERR_OUT_OF_MEMORY, ""); });
}

}  // namespace glk

using namespace glk;

extern "C" gl_status gl_precond_apply(const gl_precond *pre, const void *r, void *z, gl_stream stream)
{
    return guarded([&] {
        if (!pre || !r || !z) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_apply: NULL argument");
        if (r == z) fail(GL_ERR_INVALID_ARGUMENT, "gl_precond_apply: r and z alias");
        hipStream_t s = as_stream(stream);
        // R_k r = AMG_k(H, D r)
        double2 *vin = const_cast<gl_precond *>(pre)->vin.get();
        scale_by_volume(pre->mesh, (const double2 *)r, vin, s);
        vcycle_enqueue(pre, vin, (double2 *)z, nullptr, nullptr, 0, Launch{s});
    });
}
