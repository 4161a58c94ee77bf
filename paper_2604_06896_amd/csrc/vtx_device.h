// Device functions shared by the grid kernels and the persistent batch
// kernel of libvtx.  Formulas follow VertAX (arXiv 2604.06896), Methods,
// "Vertex model formulation": E = sum_c K_A (A-A0)^2 + K_P (P-P0)^2 +
// sum_e lambda l, with the force derived per vertex from the three cells
// and three edges around it.
#pragma once

#include "vtx_internal.h"

namespace vtx {

// ---------------------------------------------------------------- cells
// Area and perimeter of one cell from its corner row.  Corner k is packed
// as vertex id + image (W_k) relative to corner 0; positions are taken
// relative to corner 0 (r_0 = 0) so the shoelace sum never sees absolute
// coordinates:  A = 1/2 sum_k r_{k-1} x r_k,  P = sum_k |r_k - r_{k-1}|.
// When `det` is set, edges shorter than sqrt(lmin2) whose source id is below
// the target id (one half-edge of each edge) are appended to `list` as the
// global index of their source corner.  NOIMG: every corner is known to
// carry the zero image, and the periodic differences reduce to plain
// subtractions (the same values).
template <typename PosT, typename M, bool NOIMG = false, typename CornerAt>
__device__ __forceinline__ void cell_geom(const DevTissue &t, const PosT *__restrict__ X,
                                          int n, CornerAt corner_at, int row_base, M &A, M &P,
                                          bool det, M lmin2, int32_t *list,
                                          unsigned int *count) {
    const PosT Lx = (PosT)t.Lx, Ly = (PosT)t.Ly;
    // The first U corners: ids, then all their positions in flight at once
    // (rows beyond U sides take the loop below).
    constexpr int U = 8;
    int32_t w[U];
    typename Vec2<PosT>::type q[U];
#pragma unroll
    for (int k = 0; k < U; ++k) w[k] = corner_at(k < n ? k : 0);
#pragma unroll
    for (int k = 0; k < U; ++k) q[k] = ld2(X, id_of(w[k]));
    const auto p0 = q[0];
    const int v0 = id_of(w[0]);
    M px = 0, py = 0, a = 0, per = 0;
    int vprev = v0;
    auto step = [&](int k, int32_t wk, typename Vec2<PosT>::type qk) {
        const int v = id_of(wk);
        const M rx = (M)pdiff<PosT>(qk.x, p0.x, NOIMG ? 0 : ox_of(wk), Lx);
        const M ry = (M)pdiff<PosT>(qk.y, p0.y, NOIMG ? 0 : oy_of(wk), Ly);
        const M dx = rx - px, dy = ry - py;
        const M l2 = dx * dx + dy * dy;
        a += px * ry - py * rx;
        per += len_of(l2);
        if (det && l2 < lmin2 && vprev < v) {
            unsigned int s = atomicAdd(count, 1u);
            list[s] = row_base + k - 1;
        }
        px = rx;
        py = ry;
        vprev = v;
    };
#pragma unroll
    for (int k = 1; k < U; ++k)
        if (k < n) step(k, w[k], q[k]);
    for (int k = U; k < n; ++k) {
        const int32_t wk = corner_at(k);
        step(k, wk, ld2(X, id_of(wk)));
    }
    const M l2 = px * px + py * py;  // closing edge, corner n-1 -> corner 0
    per += len_of(l2);
    if (det && l2 < lmin2 && vprev < v0) {
        unsigned int s = atomicAdd(count, 1u);
        list[s] = row_base + n - 1;
    }
    A = (M)0.5 * a;
    P = per;
}

// The same area, perimeter and short-edge list, without a branch per corner:
// a row is read as if it went on with copies of its corner 0, so the step
// after the last corner is the closing edge and the ones after it add zero
// to both sums (exactly).  The branches of cell_geom keep the square roots of
// successive corners in separate basic blocks, one dependent chain after
// another; here six of them are in flight at once.  For kernels with one or
// two waves per SIMD, where that latency is the time of the cell pass; the
// evaluation of large tissues, with many waves to hide it, keeps cell_geom
// and does not compute the copies.
// `head(k)` returns corner k for a constant k <= 6, `tail(k)` for any k > 6;
// both return corner 0 for k >= n.
template <typename PosT, bool NOIMG = false, typename Head, typename Tail>
__device__ __forceinline__ void cell_geom_flat(const DevTissue &t, const PosT *__restrict__ X,
                                               int n, Head head, Tail tail, int row_base, PosT &A,
                                               PosT &P, bool det, PosT lmin2, int32_t *list,
                                               unsigned int *count) {
    const PosT Lx = (PosT)t.Lx, Ly = (PosT)t.Ly;
    const int32_t w0 = head(0);
    const auto p0 = ld2(X, id_of(w0));
    const int v0 = id_of(w0);
    PosT px = 0, py = 0, a = 0, per = 0;
    int vprev = v0;
    uint32_t shorts = 0;
    auto step = [&](int k, int32_t wk, typename Vec2<PosT>::type qk) {
        const PosT rx = pdiff<PosT>(qk.x, p0.x, NOIMG ? 0 : ox_of(wk), Lx);
        const PosT ry = pdiff<PosT>(qk.y, p0.y, NOIMG ? 0 : oy_of(wk), Ly);
        const PosT dx = rx - px, dy = ry - py;
        const PosT l2 = dx * dx + dy * dy;
        a += px * ry - py * rx;
        per += len_of(l2);
        if (det) {
            const int v = id_of(wk);
            if (k < 32) shorts |= (l2 < lmin2 && vprev < v ? 1u : 0u) << k;
            else if (l2 < lmin2 && vprev < v) list[atomicAdd(count, 1u)] = row_base + k - 1;
            vprev = v;
        }
        px = rx;
        py = ry;
    };
    constexpr int U = 6;
    int32_t w[U];
    typename Vec2<PosT>::type q[U];
#pragma unroll
    for (int k = 1; k <= U; ++k) w[k - 1] = head(k);
#pragma unroll
    for (int k = 1; k <= U; ++k) q[k - 1] = ld2(X, id_of(w[k - 1]));
#pragma unroll
    for (int k = 1; k <= U; ++k) step(k, w[k - 1], q[k - 1]);
    for (int k = U + 1; k <= n; ++k) {
        const int32_t wk = tail(k);
        step(k, wk, ld2(X, id_of(wk)));
    }
    if (det)
        for (; shorts; shorts &= shorts - 1)
            list[atomicAdd(count, 1u)] = row_base + __builtin_ctz(shorts) - 1;
    A = (PosT)0.5 * a;
    P = per;
}

// ---------------------------------------------------------------- vertex
// Force on vertex i from its star (outgoing half-edges h_k = i -> j_k,
// sector cell a_k = face(h_k), edge e_k).  With d_k = x_{j_k} - x_i,
// u_k = d_k / l_k and R(a) = (a_y, -a_x):
//   F_i = sum_k [ u_k (lambda_k + cP(a_k) + cP(a_{k-1}))
//                 - 1/2 R(d_k) (cA(a_k) - cA(a_{k-1})) ],
// cA = 2 K_A (A - A0), cP = 2 K_P (P - P0), indices mod 3.  This is
// -grad_i of the energy: the perimeter and line-tension terms pull along
// each edge, the area terms push across it by the pressure difference.
template <typename PosT, typename M>
struct Star {
    M dx[3], dy[3], ux[3], uy[3], l[3], inv[3];
    M cA[3], cP[3], lam[3];
    int nb[3];
};

// A star is loaded in three stages: (1) the star entries (two 16-byte and
// one 4-byte coalesced load) and the own position, (2) every gather they
// index, issued before any is used, (3) the arithmetic.
template <typename PosT, typename M>
struct StarLoad {
    int32_t w[3], c[3], e[3];
    typename Vec2<PosT>::type pi, q[3];
    typename Vec2<M>::type cc[3];
    PosT lam[3];
};

template <typename PosT, typename M>
__device__ __forceinline__ void star_ids(const DevTissue &t, const PosT *__restrict__ X, int v,
                                         StarLoad<PosT, M> &L) {
    const int nv = t.n_vert;
    const int4 a = reinterpret_cast<const int4 *>(t.star)[v];
    const int4 b = reinterpret_cast<const int4 *>(t.star + 4 * (int64_t)nv)[v];
    L.e[2] = t.star[8 * (int64_t)nv + v];
    L.w[0] = a.x;
    L.w[1] = a.y;
    L.w[2] = a.z;
    L.c[0] = a.w;
    L.c[1] = b.x;
    L.c[2] = b.y;
    L.e[0] = b.z;
    L.e[1] = b.w;
    L.pi = ld2(X, v);
}

template <typename PosT, typename M>
__device__ __forceinline__ void star_gather(const PosT *__restrict__ X, const DevParams<PosT> &p,
                                            const M *__restrict__ cap, StarLoad<PosT, M> &L) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        L.q[k] = ld2(X, id_of(L.w[k]));
        L.cc[k] = ld2(cap, L.c[k]);
    }
    if (p.lam) {
#pragma unroll
        for (int k = 0; k < 3; ++k) L.lam[k] = p.lam[L.e[k]];
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) L.lam[k] = p.lam_s;
    }
}

// NOIMG: the three neighbours are known to carry the zero image.  HVP: the
// inverse lengths of the Hessian-vector product (len_inv_hvp).
template <typename PosT, typename M, bool NOIMG = false, bool HVP = false>
__device__ __forceinline__ void star_math(const DevTissue &t, const StarLoad<PosT, M> &L,
                                          Star<PosT, M> &s, PosT &xi, PosT &yi) {
    const PosT Lx = (PosT)t.Lx, Ly = (PosT)t.Ly;
    xi = L.pi.x;
    yi = L.pi.y;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        s.nb[k] = id_of(L.w[k]);
        s.dx[k] = (M)pdiff<PosT>(L.q[k].x, L.pi.x, NOIMG ? 0 : ox_of(L.w[k]), Lx);
        s.dy[k] = (M)pdiff<PosT>(L.q[k].y, L.pi.y, NOIMG ? 0 : oy_of(L.w[k]), Ly);
        s.cA[k] = L.cc[k].x;
        s.cP[k] = L.cc[k].y;
        s.lam[k] = (M)L.lam[k];
        // a zero-length edge contributes its minimum-norm subgradient, 0
        M l, inv;
        if (HVP) len_inv_hvp(s.dx[k] * s.dx[k] + s.dy[k] * s.dy[k], l, inv);
        else len_inv(s.dx[k] * s.dx[k] + s.dy[k] * s.dy[k], l, inv);
        s.l[k] = l;
        s.inv[k] = inv;
        s.ux[k] = s.dx[k] * inv;
        s.uy[k] = s.dy[k] * inv;
    }
}

template <typename PosT, typename M>
__device__ __forceinline__ void load_star(const DevTissue &t, const PosT *__restrict__ X,
                                          const DevParams<PosT> &p, const M *__restrict__ cap,
                                          int v, Star<PosT, M> &s, PosT &xi, PosT &yi) {
    StarLoad<PosT, M> L;
    star_ids<PosT, M>(t, X, v, L);
    star_gather<PosT, M>(X, p, cap, L);
    star_math<PosT, M>(t, L, s, xi, yi);
}

template <typename PosT, typename M>
__device__ __forceinline__ void star_force(const Star<PosT, M> &s, M &fx, M &fy) {
    fx = 0;
    fy = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int km = (k + 2) % 3;
        const M T = s.lam[k] + s.cP[k] + s.cP[km];
        const M dA = (M)0.5 * (s.cA[k] - s.cA[km]);
        fx += T * s.ux[k] - dA * s.dy[k];
        fy += T * s.uy[k] + dA * s.dx[k];
    }
}

// ---------------------------------------------------------- T1 helpers
// Exact (double) helpers used by the sequential T1 pass.  Positions of the
// two vertices of the edge under test can be overridden.
template <typename PosT>
struct PosOverride {
    int vi, vj;
    double xi, yi, xj, yj;
    __device__ __forceinline__ void get(const PosT *X, int v, double &x, double &y) const {
        if (v == vi) { x = xi; y = yi; }
        else if (v == vj) { x = xj; y = yj; }
        else { x = (double)X[2 * (int64_t)v]; y = (double)X[2 * (int64_t)v + 1]; }
    }
};

template <typename PosT>
__device__ __forceinline__ void he_vec(const DevTissue &t, const PosT *X, int h,
                                       const PosOverride<PosT> &ov, double &dx, double &dy) {
    const int32_t *r = t.he + 8 * (int64_t)h;
    double xs, ys, xg, yg;
    ov.get(X, r[HS], xs, ys);
    ov.get(X, r[HG], xg, yg);
    dx = pdiff<double>(xg, xs, r[HOX], t.Lx);
    dy = pdiff<double>(yg, ys, r[HOY], t.Ly);
}

template <typename PosT>
__device__ __forceinline__ void cell_walk(const DevTissue &t, const PosT *X, int h0,
                                          const PosOverride<PosT> &ov, double &A, double &P) {
    double rx = 0.0, ry = 0.0, a = 0.0, per = 0.0;
    int h = h0;
    int guard = 0;
    do {
        double dx, dy;
        he_vec<PosT>(t, X, h, ov, dx, dy);
        a += rx * dy - ry * dx;
        per += sqrt(dx * dx + dy * dy);
        rx += dx;
        ry += dy;
        h = t.he[8 * (int64_t)h + HN];
    } while (h != h0 && ++guard < 4096);
    A = 0.5 * a;
    P = per;
}

// ------------------------------------------------------------------- T1
// One half-edge record loaded as two 16-byte vectors.
struct HeRec {
    int prev, next, twin, src, tgt, face, ox, oy;
};
__device__ __forceinline__ HeRec he_rec(const DevTissue &t, int h) {
    const int4 *r = reinterpret_cast<const int4 *>(t.he + 8 * (int64_t)h);
    const int4 a = r[0], b = r[1];
    return HeRec{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
}

// Area and perimeter (FP64) of cell c read from its corner row, with the
// two vertices of the edge under test at overridden positions and one
// optional edit of the corner sequence:
//   edit 1: drop vertex va;
//   edit 2: put vertex vb, at the image of va plus (sx, sy), right before va.
// Coordinates are unwrapped x + W L; the first corner is the origin.  One
// lane walks the row; the T1 pass uses it for rows longer than kRowLanes.
template <typename PosT>
__device__ __forceinline__ void row_geom(const DevTissue &t, const PosT *X, int c,
                                         const PosOverride<PosT> &ov, int edit, int va, int vb,
                                         int sx, int sy, double &A, double &P) {
    const int rb = t.row_ptr[c], n = t.nsides[c];
    double x0 = 0.0, y0 = 0.0, px = 0.0, py = 0.0, a = 0.0, per = 0.0;
    bool first = true;
    for (int k = 0, ins = 0; k < n;) {
        const int32_t wk = t.corner[rb + k];
        int v = id_of(wk), wx = ox_of(wk), wy = oy_of(wk);
        if (edit == 1 && v == va) {
            ++k;
            continue;
        }
        if (edit == 2 && v == va && !ins) {  // vb first, then va on the next turn
            ins = 1;
            v = vb;
            wx += sx;
            wy += sy;
        } else {
            ++k;
        }
        double x, y;
        ov.get(X, v, x, y);
        const double rx = x + wx * t.Lx, ry = y + wy * t.Ly;
        if (first) {
            x0 = rx;
            y0 = ry;
            first = false;
            continue;
        }
        const double ux = rx - x0, uy = ry - y0;
        const double dx = ux - px, dy = uy - py;
        a += px * uy - py * ux;
        per += len_of(dx * dx + dy * dy);
        px = ux;
        py = uy;
    }
    per += len_of(px * px + py * py);  // closing edge back to the first corner
    A = 0.5 * a;
    P = per;
}

template <typename PosT>
__device__ __forceinline__ double cell_energy(const DevParams<PosT> &p, int c, double A,
                                              double P) {
    const double da = A - (double)p.a0(c), dp = P - (double)p.p0(c);
    return (double)p.ka(c) * da * da + (double)p.kp(c) * dp * dp;
}

// In-place edit of cell c's corner row after an exchange.
//   edit 1: drop vertex va; the corner before it now leaves by half-edge nh.
//   edit 2: insert vertex vb, leaving by half-edge nh, right before va, at
//           the image of va plus (sx, sy).
// Images are re-based so that the first corner has image 0.  A row without
// a spare slot is first moved to the free pool at the end of the corner
// arrays (*relocated is set; rows are compacted again after the pass).
// Returns false on an inconsistency or when the pool is exhausted.
__device__ __forceinline__ bool row_edit(const DevTissue &t, int c, int edit, int va, int vb,
                                         int nh, int sx, int sy, int *relocated) {
    int rb = t.row_ptr[c];
    const int n = t.nsides[c];
    if (edit == 2 && n + 1 > t.row_cap[c]) {
        const int nb = *t.pool_top;
        const int cap = n + 1 + kRowExtra;
        if (nb + cap > t.corner_cap) return false;
        for (int q = 0; q < n; ++q) {
            t.corner[nb + q] = t.corner[rb + q];
            t.corner_he[nb + q] = t.corner_he[rb + q];
        }
        *t.pool_top = nb + cap;
        t.row_ptr[c] = nb;
        t.row_cap[c] = cap;
        rb = nb;
        *relocated = 1;
    }
    int32_t *cw = t.corner + rb;
    int32_t *ch = t.corner_he + rb;
    int k = 0;
    while (k < n && id_of(cw[k]) != va) ++k;
    if (k == n) return false;
    if (edit == 1) {
        const int kp = (k + n - 1) % n;
        ch[kp] = nh;
        for (int q = k; q + 1 < n; ++q) {
            cw[q] = cw[q + 1];
            ch[q] = ch[q + 1];
        }
        t.nsides[c] = n - 1;
    } else {
        for (int q = n; q > k; --q) {
            cw[q] = cw[q - 1];
            ch[q] = ch[q - 1];
        }
        cw[k] = pack_id(vb, ox_of(cw[k + 1]) + sx, oy_of(cw[k + 1]) + sy);
        ch[k] = nh;
        t.nsides[c] = n + 1;
    }
    const int m = t.nsides[c];
    const int bx = ox_of(cw[0]), by = oy_of(cw[0]);
    if (bx || by)
        for (int q = 0; q < m; ++q) cw[q] = pack_id(id_of(cw[q]), ox_of(cw[q]) - bx, oy_of(cw[q]) - by);
    for (int q = 0; q < m; ++q)
        if (ox_of(cw[q]) < -1 || ox_of(cw[q]) > 1 || oy_of(cw[q]) < -1 || oy_of(cw[q]) > 1)
            return false;
    return true;
}

// Result of one sequential T1 pass.
struct T1Counts {
    int64_t swaps, stretches;
    int changed;    // topology changed
    int relocated;  // a row moved to the pool: compact all rows after the pass
    int overflow;   // 1: too many pending re-checks; 2: row edit failed
};

// Rows of up to this many corners are evaluated and edited by 16 lanes (an
// exchange adds one corner, and the closing edge takes one more lane).
constexpr int kRowLanes = 14;

__device__ __forceinline__ int lane_int(int x, int lane) {
    return __builtin_amdgcn_readlane(x, lane);
}
constexpr int kDppRowShl1 = 0x101;  // lane i of a row of 16 reads lane i + 1
constexpr int kDppRowShr1 = 0x111;  // lane i of a row of 16 reads lane i - 1

// Area and perimeter of four polygons, one per row of 16 lanes: lane s < m
// holds corner s (unwrapped), m + 1 <= 16.  Valid in lane 0 of each row.  The
// terms are added in corner order, as one lane walking the row adds them.
__device__ __forceinline__ void quad_rows_geom(double rx, double ry, int s, int m, int m_max,
                                               double &A, double &P) {
    const int first = (threadIdx.x & 63) & 48;
    const double x0 = __shfl(rx, first, 64), y0 = __shfl(ry, first, 64);
    const double ux = s < m ? rx - x0 : 0.0, uy = s < m ? ry - y0 : 0.0;
    // (lane 0 of a row has no lane before it and reads the 0 of `old`)
    const double px = dpp_f64<kDppRowShr1>(ux), py = dpp_f64<kDppRowShr1>(uy);
    const double dx = ux - px, dy = uy - py;
    double cross = px * uy - py * ux;
    double len = len_of(dx * dx + dy * dy);
    double a = 0.0, per = 0.0;
    for (int k = 1; k <= m_max; ++k) {
        cross = dpp_f64<kDppRowShl1>(cross);
        len = dpp_f64<kDppRowShl1>(len);
        a += cross;
        per += len;
    }
    A = 0.5 * a;
    P = per;
}

// Sequential T1 pass over the ascending candidate list `list[0..n)` (edge
// ids, sorted, may hold duplicates and INT_MAX padding), run by the 64
// lanes of ONE wave with wave-uniform control flow.  Each candidate is
// re-checked with the current positions; edges next to a processed edge
// that become short are visited in turn as well, so the result equals
// visiting every edge in ascending id order.
//
// A candidate is a chain of dependent loads, so the pass is arranged to make
// it short: the half-edge of the edge, then the stars of its ends i and j
// (which name the other four half-edges, vertices, edges and cells around
// the edge), then the four cells' rows, their corners and the positions,
// each level loaded by as many lanes as it has entries.  With h: i -> j in
// C1 and its twin in C2, the star of i holds h, twin(prev(h)) = i -> a (in
// C3) and next(twin) = i -> b (in C2) counter-clockwise, the star of j holds
// the twin, j -> d (in C4) and next(h) = j -> c (in C1).  Both outcomes are
// evaluated on the rows C1..C4 (16 lanes each, the exchange as an edit of the
// row) and the five edges at the ends (a lane each).  An exchange is then
// stored from values in registers, the rows by their lanes: C1 drops j, C2
// drops i, C3 gains j before i and C4 gains i before j, and the moved
// half-edges change image offset by the offset of h so that every edge
// vector is kept.  A walk by single lanes with a load per step (the form
// before) took about 45 us per exchange and 15 us per stretch.
template <typename PosT, typename M>
__device__ __forceinline__ T1Counts t1_sequential(const DevTissue &t, PosT *X,
                                                  const DevParams<PosT> &p, M *cap,
                                                  const int32_t *list, int n, int32_t *extra,
                                                  double l_min, double l_new) {
    const int lane = threadIdx.x & 63, q = lane >> 4, s = lane & 15;
    const int nv = t.n_vert;
    T1Counts out{0, 0, 0, 0, 0};
    int pos = 0, n_extra = 0;
    int last = -1;
    const double hl = 0.5 * l_new;
    for (;;) {
        // next edge: min of list[pos] and the pending set.  Every lane keeps
        // the same bookkeeping (the LDS set is written by all lanes with the
        // same values), so no lane depends on another's writes.
        int e = 0x7fffffff;
        while (pos < n && list[pos] <= last) ++pos;
        if (pos < n) e = list[pos];
        for (int a = 0; a < n_extra; ++a)
            if (extra[a] < e) e = extra[a];
        e = __builtin_amdgcn_readfirstlane(e);
        if (e == 0x7fffffff) break;
        if (pos < n && list[pos] == e) ++pos;
        {   // drop e (and anything below it) from the pending set
            int m = 0;
            for (int a = 0; a < n_extra; ++a) {
                const int v = extra[a];
                if (v > e) extra[m++] = v;
            }
            n_extra = m;
        }
        last = e;

        const int h = __builtin_amdgcn_readfirstlane(t.edge_he[e]);
        const HeRec rh = he_rec(t, h);
        const int i = __builtin_amdgcn_readfirstlane(rh.src);
        const int j = __builtin_amdgcn_readfirstlane(rh.tgt);
        const int tw = __builtin_amdgcn_readfirstlane(rh.twin);
        const int p1 = __builtin_amdgcn_readfirstlane(rh.prev);
        const int n1 = __builtin_amdgcn_readfirstlane(rh.next);
        const int hox = __builtin_amdgcn_readfirstlane(rh.ox);
        const int hoy = __builtin_amdgcn_readfirstlane(rh.oy);
        // star slots: lanes 0-2 those of i, lanes 4-6 those of j
        const int sl = (lane & 3) < 3 ? (lane & 3) : 0;
        const int sv = (lane & 4) ? j : i;
        const int32_t st_w = t.star[star_nb_at(nv, sl, sv)];
        const int32_t st_c = t.star[star_cell_at(nv, sl, sv)];
        const int32_t st_e = t.star[star_edge_at(nv, sl, sv)];
        const int32_t st_h = t.star_he[sl * nv + sv];
        const int p2_v = t.he[8 * (int64_t)tw + HP];
        const int tn1_v = t.he[8 * (int64_t)n1 + HT];
        const double xi = (double)X[2 * (int64_t)i], yi = (double)X[2 * (int64_t)i + 1];
        const double xj = (double)X[2 * (int64_t)j], yj = (double)X[2 * (int64_t)j + 1];
        const double dx = pdiff<double>(xj, xi, hox, t.Lx), dy = pdiff<double>(yj, yi, hoy, t.Ly);
        const double l = len_of(dx * dx + dy * dy);
        if (__builtin_amdgcn_readfirstlane(l < l_min ? 0 : 1)) continue;
        double ux = 1.0, uy = 0.0;
        if (l > 0.0) { ux = dx / l; uy = dy / l; }
        const double mx = xi + 0.5 * dx, my = yi + 0.5 * dy;
        const double sxL = hox * t.Lx, syL = hoy * t.Ly;
        const PosOverride<PosT> S{i, j, mx - hl * ux, my - hl * uy, mx + hl * ux - sxL, my + hl * uy - syL};
        const double nx = -uy, ny = ux;
        const PosOverride<PosT> T{i, j, mx + hl * nx, my + hl * ny, mx - hl * nx - sxL, my - hl * ny - syL};

        // slots after that of h (at i) and of the twin (at j)
        const uint64_t at_i = __builtin_amdgcn_ballot_w64(lane < 3 && st_h == h);
        const uint64_t at_j = __builtin_amdgcn_ballot_w64(lane >= 4 && lane < 7 && st_h == tw);
        const int s0 = at_i ? __builtin_ctzll(at_i) : 0, s4 = at_j ? __builtin_ctzll(at_j) - 4 : 0;
        const int la = (s0 + 1) % 3, lb = (s0 + 2) % 3, ld = 4 + (s4 + 1) % 3, lc = 4 + (s4 + 2) % 3;
        const int wa = lane_int(st_w, la), wb = lane_int(st_w, lb), wc = lane_int(st_w, lc),
                  wd = lane_int(st_w, ld);
        const int ea = lane_int(st_e, la), eb = lane_int(st_e, lb), ec = lane_int(st_e, lc),
                  ed = lane_int(st_e, ld);
        const int tp1 = lane_int(st_h, la), n2 = lane_int(st_h, lb), tp2 = lane_int(st_h, ld);
        const int C1 = lane_int(st_c, s0), C2 = lane_int(st_c, 4 + s4), C3 = lane_int(st_c, la),
                  C4 = lane_int(st_c, ld);
        const int p2 = __builtin_amdgcn_readfirstlane(p2_v);
        const int tn1 = __builtin_amdgcn_readfirstlane(tn1_v);
        // half-edges the kept offsets refer to: a -> i, j -> c, d -> j, i -> b
        const int p1x = -ox_of(wa), p1y = -oy_of(wa), n1x = ox_of(wc), n1y = oy_of(wc);
        const int p2x = -ox_of(wd), p2y = -oy_of(wd), n2x = ox_of(wb), n2y = oy_of(wb);
        const int va_ = id_of(wa), vb_ = id_of(wb), vc_ = id_of(wc), vd_ = id_of(wd);

        // the cells: row q of lanes has C1..C4
        const int cq = q == 0 ? C1 : q == 1 ? C2 : q == 2 ? C3 : C4;
        const int rb = t.row_ptr[cq], nq = t.nsides[cq], rc = t.row_cap[cq];
        const double ka = (double)p.ka(cq), a0 = (double)p.a0(cq), kp = (double)p.kp(cq),
                     p0 = (double)p.p0(cq);
        const int tn2_v = t.he[8 * (int64_t)n2 + HT];
        // stars of c (lanes 0-2) and b (lanes 4-6), which change neighbour
        const int cv = (lane & 4) ? vb_ : vc_;
        const int32_t cb_w = t.star[star_nb_at(nv, sl, cv)];
        const int32_t cb_c = t.star[star_cell_at(nv, sl, cv)];
        const int32_t cb_e = t.star[star_edge_at(nv, sl, cv)];
        const int32_t cb_h = t.star_he[sl * nv + cv];
        // (a, b, c and d are neither i nor j where C1..C4 are distinct)
        // the five edges at i and j: lanes 0-4 for the stretch, 8-12 for the
        // exchange (i -> c and j -> b replace j -> c and i -> b)
        const int er = lane & 7;
        const int ev = er == 1 ? va_ : er == 2 ? vc_ : er == 3 ? vd_ : vb_;
        const int ee = er == 0 ? e : er == 1 ? ea : er == 2 ? ec : er == 3 ? ed : eb;
        const double xf = (double)X[2 * (int64_t)ev], yf = (double)X[2 * (int64_t)ev + 1];
        const double el = (double)p.lm(ee);

        const bool distinct = C1 != C2 && C1 != C3 && C1 != C4 && C2 != C3 && C2 != C4 && C3 != C4;
        const int nC1 = lane_int(nq, 0), nC2 = lane_int(nq, 16), nC3 = lane_int(nq, 32),
                  nC4 = lane_int(nq, 48);
        const bool admissible = distinct && nC1 > 3 && nC2 > 3;
        const int n_max = max(max(nC1, nC2), max(nC3, nC4));
        const bool wide = n_max <= kRowLanes;
        // the exchange as an edit of row q: C1 drops j, C2 drops i, C3 gains j
        // before i, C4 gains i before j
        const int ed_q = q < 2 ? 1 : 2;
        const int ev_a = (q == 0 || q == 3) ? j : i;
        const int ev_b = q == 2 ? j : i;
        const int esx = q == 2 ? hox : -hox, esy = q == 2 ? hoy : -hoy;

        int32_t cw = 0, ch = 0, xw = 0, xh = 0;  // the lane's corner now and after the exchange
        int xox = 0, xoy = 0, xm = 0;            // its image, and the corners after the exchange
        bool ok = true;                          // the row holds the vertex to edit at
        double AS = 0.0, PS = 0.0, AT = 0.0, PT = 0.0;
        if (wide) {
            const int at = rb + (s < nq ? s : 0);
            cw = t.corner[at];
            ch = t.corner_he[at];
            const int v = id_of(cw);
            double x = (double)X[2 * (int64_t)v], y = (double)X[2 * (int64_t)v + 1];
            double xs = v == i ? S.xi : v == j ? S.xj : x, ys = v == i ? S.yi : v == j ? S.yj : y;
            quad_rows_geom(xs + ox_of(cw) * t.Lx, ys + oy_of(cw) * t.Ly, s, nq, n_max, AS, PS);
            if (admissible) {
                const uint64_t hit = __builtin_amdgcn_ballot_w64(s < nq && v == ev_a);
                const int hits = (int)((hit >> (16 * q)) & 0xffffu);
                ok = hits != 0;
                const int k = ok ? __builtin_ctz(hits) : 0;
                // corner s of the edited row: one of the old row, or the new one
                xm = ed_q == 1 ? nq - 1 : nq + 1;
                const bool ins = ed_q == 2 && s == k;
                const int from = (lane & 48) + (ed_q == 1 ? (s < k ? s : min(s + 1, 15))
                                                          : (s <= k ? s : s - 1));
                xw = __shfl(cw, from, 64);
                xh = __shfl(ch, from, 64);
                const double fx = __shfl(x, from, 64), fy = __shfl(y, from, 64);
                const int xv = ins ? ev_b : id_of(xw);
                xox = ox_of(xw) + (ins ? esx : 0);
                xoy = oy_of(xw) + (ins ? esy : 0);
                // the corner before a dropped vertex leaves by a new half-edge
                const int kp_new = k > 0 ? k - 1 : nq - 2;
                if (ed_q == 1 && s == kp_new) xh = q == 0 ? n1 : n2;
                if (ins) xh = q == 2 ? tw : h;
                xw = xv;  // the id; the image is added when it is stored
                const double xt = xv == i ? T.xi : xv == j ? T.xj : fx;
                const double yt = xv == i ? T.yi : xv == j ? T.yj : fy;
                quad_rows_geom(xt + xox * t.Lx, yt + xoy * t.Ly, s, xm, n_max + 1, AT, PT);
            }
        } else if (s == 0) {
            row_geom<PosT>(t, X, cq, S, 0, -1, -1, 0, 0, AS, PS);
            if (admissible) row_geom<PosT>(t, X, cq, T, ed_q, ev_a, ev_b, esx, esy, AT, PT);
        }
        bool take_T = false;
        if (admissible) {
            auto energy = [&](double A, double P) {
                const double da = A - a0, dp = P - p0;
                return ka * da * da + kp * dp * dp;
            };
            const double eS = energy(AS, PS), eT = energy(AT, PT);
            const double ES = ((readlane_f64(eS, 0) + readlane_f64(eS, 16)) + readlane_f64(eS, 32)) +
                              readlane_f64(eS, 48);
            const double ET0 = ((readlane_f64(eT, 0) + readlane_f64(eT, 16)) + readlane_f64(eT, 32)) +
                               readlane_f64(eT, 48);
            const bool exch = (lane & 8) != 0;
            const double ix = exch ? T.xi : S.xi, iy = exch ? T.yi : S.yi;
            const double jx = exch ? T.xj : S.xj, jy = exch ? T.yj : S.yj;
            // source and target of the edge, its image offset
            const bool c_at_i = er == 2 && exch, b_at_j = er == 4 && exch;
            const double gx = er == 0 ? jx : er == 1 ? ix : er == 3 ? jx : xf;
            const double gy = er == 0 ? jy : er == 1 ? iy : er == 3 ? jy : yf;
            const double sx = er == 0 ? ix : er == 2 ? (c_at_i ? ix : jx)
                                                     : er == 4 ? (b_at_j ? jx : ix) : xf;
            const double sy = er == 0 ? iy : er == 2 ? (c_at_i ? iy : jy)
                                                     : er == 4 ? (b_at_j ? jy : iy) : yf;
            const int ox = er == 0 ? hox : er == 1 ? p1x : er == 2 ? n1x + (c_at_i ? hox : 0)
                         : er == 3 ? p2x : n2x - (b_at_j ? hox : 0);
            const int oy = er == 0 ? hoy : er == 1 ? p1y : er == 2 ? n1y + (c_at_i ? hoy : 0)
                         : er == 3 ? p2y : n2y - (b_at_j ? hoy : 0);
            const double ddx = gx + ox * t.Lx - sx, ddy = gy + oy * t.Ly - sy;
            const double le = el * len_of(ddx * ddx + ddy * ddy);
            auto edges = [&](int o) {
                return (((readlane_f64(le, o) + readlane_f64(le, o + 1)) + readlane_f64(le, o + 2)) +
                        readlane_f64(le, o + 3)) + readlane_f64(le, o + 4);
            };
            take_T = ET0 + edges(8) < ES + edges(0);
        }
        take_T = __builtin_amdgcn_readfirstlane(take_T ? 1 : 0) != 0;
        const double Wxi = take_T ? T.xi : S.xi, Wyi = take_T ? T.yi : S.yi;
        const double Wxj = take_T ? T.xj : S.xj, Wyj = take_T ? T.yj : S.yj;
        // coefficients of C1..C4 from the kept outcome's geometry
        if (s == 0) {
            cap[2 * (int64_t)cq] = (M)(2.0 * ka * ((take_T ? AT : AS) - a0));
            cap[2 * (int64_t)cq + 1] = (M)(2.0 * kp * ((take_T ? PT : PS) - p0));
        }
        if (lane == 0) {
            X[2 * (int64_t)i] = (PosT)Wxi;
            X[2 * (int64_t)i + 1] = (PosT)Wyi;
            X[2 * (int64_t)j] = (PosT)Wxj;
            X[2 * (int64_t)j + 1] = (PosT)Wyj;
        }
        if (take_T) {
            const int tn2 = __builtin_amdgcn_readfirstlane(tn2_v);
            const int c1x = n1x + hox, c1y = n1y + hoy;  // i -> c
            const int b2x = n2x - hox, b2y = n2y - hoy;  // j -> b
            if (lane == 0) {
                auto R = [&](int x) { return t.he + 8 * (int64_t)x; };
                // C1: a->i -> i->c
                R(p1)[HN] = n1;
                R(n1)[HP] = p1;
                R(n1)[HS] = i;
                R(tn1)[HG] = i;
                R(n1)[HOX] = c1x;
                R(n1)[HOY] = c1y;
                R(tn1)[HOX] = -c1x;
                R(tn1)[HOY] = -c1y;
                // C2: d->j -> j->b
                R(p2)[HN] = n2;
                R(n2)[HP] = p2;
                R(n2)[HS] = j;
                R(tn2)[HG] = j;
                R(n2)[HOX] = b2x;
                R(n2)[HOY] = b2y;
                R(tn2)[HOX] = -b2x;
                R(tn2)[HOY] = -b2y;
                // C4: c->i -> i->j -> j->d
                R(tn1)[HN] = h;
                R(h)[HP] = tn1;
                R(h)[HN] = tp2;
                R(tp2)[HP] = h;
                R(h)[HF] = C4;
                // C3: b->j -> j->i -> i->a
                R(tn2)[HN] = tw;
                R(tw)[HP] = tn2;
                R(tw)[HN] = tp1;
                R(tp1)[HP] = tw;
                R(tw)[HF] = C3;
                if (t.cell_he[C1] == h) t.cell_he[C1] = n1;
                if (t.cell_he[C2] == tw) t.cell_he[C2] = n2;
            }
            // stars: i from h (i->j, i->c, i->a), j from the twin (j->i, j->b,
            // j->d); c and b turned so that the changed half-edge comes first
            if ((lane & 3) < 3 && lane < 7) {
                const int k = lane & 3;
                const bool at_j2 = (lane & 4) != 0;
                const int v = at_j2 ? j : i;
                int32_t w, c, ed2, he2;
                if (!at_j2) {
                    w = k == 0 ? pack_id(j, hox, hoy) : k == 1 ? pack_id(vc_, c1x, c1y) : wa;
                    c = k == 0 ? C4 : k == 1 ? C1 : C3;
                    ed2 = k == 0 ? e : k == 1 ? ec : ea;
                    he2 = k == 0 ? h : k == 1 ? n1 : tp1;
                } else {
                    w = k == 0 ? pack_id(i, -hox, -hoy) : k == 1 ? pack_id(vb_, b2x, b2y) : wd;
                    c = k == 0 ? C3 : k == 1 ? C2 : C4;
                    ed2 = k == 0 ? e : k == 1 ? eb : ed;
                    he2 = k == 0 ? tw : k == 1 ? n2 : tp2;
                }
                t.star[star_nb_at(nv, k, v)] = w;
                t.star[star_cell_at(nv, k, v)] = c;
                t.star[star_edge_at(nv, k, v)] = ed2;
                t.star_he[k * nv + v] = he2;
            }
            {
                const int moved = (lane & 4) ? tn2 : tn1;
                const bool slot = (lane & 3) < 3 && lane < 7;
                const uint64_t first = __builtin_amdgcn_ballot_w64(slot && cb_h == moved);
                const int f0 = (int)(first & 7u), f1 = (int)((first >> 4) & 7u);
                const int f = (lane & 4) ? (f1 ? __builtin_ctz(f1) : 0) : (f0 ? __builtin_ctz(f0) : 0);
                if (slot) {
                    const int k = ((lane & 3) + 3 - f) % 3;
                    const int32_t w = k != 0 ? cb_w
                                             : (lane & 4) ? pack_id(j, -b2x, -b2y)
                                                          : pack_id(i, -c1x, -c1y);
                    t.star[star_nb_at(nv, k, cv)] = w;
                    t.star[star_cell_at(nv, k, cv)] = cb_c;
                    t.star[star_edge_at(nv, k, cv)] = cb_e;
                    t.star_he[k * nv + cv] = cb_h;
                }
            }
            // rows
            if (wide) {
                // a row without a spare slot moves to the pool (C3 first)
                const bool grow = ed_q == 2 && xm > rc;
                const uint64_t grows = __builtin_amdgcn_ballot_w64(grow);
                const bool g3 = ((grows >> 32) & 1u) != 0, g4 = ((grows >> 48) & 1u) != 0;
                int rb2 = rb;
                if (g3 || g4) {
                    const int top = __builtin_amdgcn_readfirstlane(*t.pool_top);
                    const int cap3 = g3 ? nC3 + 1 + kRowExtra : 0, cap4 = g4 ? nC4 + 1 + kRowExtra : 0;
                    if (top + cap3 + cap4 > t.corner_cap) ok = false;
                    if (grow) rb2 = q == 2 ? top : top + cap3;
                    if (lane == 0) *t.pool_top = top + cap3 + cap4;
                    out.relocated = 1;
                }
                // images relative to the (new) first corner
                xox -= lane_int(xox, 0) * (q == 0) + lane_int(xox, 16) * (q == 1) +
                       lane_int(xox, 32) * (q == 2) + lane_int(xox, 48) * (q == 3);
                xoy -= lane_int(xoy, 0) * (q == 0) + lane_int(xoy, 16) * (q == 1) +
                       lane_int(xoy, 32) * (q == 2) + lane_int(xoy, 48) * (q == 3);
                if (s < xm && (xox < -1 || xox > 1 || xoy < -1 || xoy > 1)) ok = false;
                if (__builtin_amdgcn_ballot_w64(!ok) != 0) {
                    out.overflow = 2;
                } else {
                    if (s < xm) {
                        t.corner[rb2 + s] = pack_id(xw, xox, xoy);
                        t.corner_he[rb2 + s] = xh;
                    }
                    if (s == 0) {
                        t.nsides[cq] = xm;
                        if (grow) {
                            t.row_ptr[cq] = rb2;
                            t.row_cap[cq] = xm + kRowExtra;
                        }
                    }
                }
            } else {
                int bad = 0, moved = 0;
                if (lane == 0) {
                    bool good = row_edit(t, C1, 1, j, -1, n1, 0, 0, &moved);
                    good = row_edit(t, C2, 1, i, -1, n2, 0, 0, &moved) && good;
                    good = row_edit(t, C3, 2, i, j, tw, hox, hoy, &moved) && good;
                    good = row_edit(t, C4, 2, j, i, h, -hox, -hoy, &moved) && good;
                    bad = good ? 0 : 1;
                }
                if (lane_int(bad, 0)) out.overflow = 2;
                if (lane_int(moved, 0)) out.relocated = 1;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        if (out.overflow == 2) return out;
        if (take_T) {
            ++out.swaps;
            out.changed = 1;
        } else {
            ++out.stretches;
        }
        // the four other edges at i and j may have become short: a->i, and
        // i->c, d->j, j->b after an exchange (j->c, i->b after a stretch);
        // lanes 0-3 in the order a, c, d, b
        {
            const double far_x = __shfl(xf, (lane & 3) + 1, 64), far_y = __shfl(yf, (lane & 3) + 1, 64);
            const int r = lane & 3;
            const bool near_i = r == 0 || (r == 1 && take_T) || (r == 3 && !take_T);
            const double wx = near_i ? Wxi : Wxj, wy = near_i ? Wyi : Wyj;
            // (the far end is i or j itself only in tilings of a few cells)
            const int fv = r == 0 ? va_ : r == 1 ? vc_ : r == 2 ? vd_ : vb_;
            const double farx = fv == i ? Wxi : fv == j ? Wxj : far_x;
            const double fary = fv == i ? Wyi : fv == j ? Wyj : far_y;
            const bool out_going = (r & 1) != 0;  // from i or j to the far vertex
            const int ox = r == 0 ? p1x : r == 1 ? n1x + (take_T ? hox : 0)
                         : r == 2 ? p2x : n2x - (take_T ? hox : 0);
            const int oy = r == 0 ? p1y : r == 1 ? n1y + (take_T ? hoy : 0)
                         : r == 2 ? p2y : n2y - (take_T ? hoy : 0);
            const double gx = out_going ? farx : wx, gy = out_going ? fary : wy;
            const double fx = out_going ? wx : farx, fy = out_going ? wy : fary;
            const double ddx = gx + ox * t.Lx - fx, ddy = gy + oy * t.Ly - fy;
            const uint64_t shorts = __builtin_amdgcn_ballot_w64(
                lane < 4 && len_of(ddx * ddx + ddy * ddy) < l_min);
            for (int a = 0; a < 4; ++a) {
                const int e2 = a == 0 ? ea : a == 1 ? ec : a == 2 ? ed : eb;
                if (e2 <= e || !((shorts >> a) & 1u)) continue;
                bool present = false;
                for (int b = 0; b < n_extra; ++b) present |= extra[b] == e2;
                if (!present) {
                    if (n_extra >= kT1Extra) out.overflow = 1;
                    else extra[n_extra++] = e2;
                }
            }
        }
    }
    return out;
}

// Block-wide bitonic sort (ascending) of `a[0..n)`, n a power of two, one
// compare-exchange pair per thread and round.  Pairs at a distance of at
// most 64 stay inside the 128 elements their wave works on, so between two
// such rounds the wave only waits for its own accesses; the block meets at a
// barrier for the longer distances and at the end.  The rounds are a chain
// of dependent LDS accesses: the sort of 4096 keys takes 78 of them, and
// with a barrier each and both elements of a pair read by both threads it
// was half of the tile build's 200 us.
__device__ __forceinline__ void block_bitonic(int32_t *a, int n) {
    const int np = n >> 1;
    for (int k = 2; k <= n; k <<= 1)
        for (int jj = k >> 1; jj > 0; jj >>= 1) {
            for (int p = threadIdx.x; p < np; p += blockDim.x) {
                const int i = ((p & ~(jj - 1)) << 1) | (p & (jj - 1));
                const int32_t x = a[i], y = a[i + jj];
                if ((x > y) == ((i & k) == 0)) {
                    a[i] = y;
                    a[i + jj] = x;
                }
            }
            const int next = jj > 1 ? jj >> 1 : k;  // distance of the next round
            if (jj > 64 || next > 64 || (jj == 1 && k == n)) {
                __syncthreads();
            } else {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                __builtin_amdgcn_wave_barrier();
            }
        }
}

// Rebuild the cell -> corner rows from the half-edge table (block-wide):
// row_ptr is the exclusive scan of nsides, each row is walked from
// cell_he[c] with the cumulative image of each corner.  Returns nonzero
// (in thread 0) if a cell spans more than one periodic image.
__device__ __forceinline__ int rebuild_rows_block(const DevTissue &t, int32_t *sh_scan) {
    __shared__ int32_t carry;
    __shared__ int bad;
    if (threadIdx.x == 0) { carry = 0; bad = 0; }
    __syncthreads();
    const int nc = t.n_cell;
    for (int base = 0; base < nc; base += blockDim.x) {
        const int c = base + threadIdx.x;
        const int v = c < nc ? t.nsides[c] + kRowSlack : 0;
        sh_scan[threadIdx.x] = v;
        __syncthreads();
        for (int off = 1; off < (int)blockDim.x; off <<= 1) {
            int add = threadIdx.x >= (unsigned)off ? sh_scan[threadIdx.x - off] : 0;
            __syncthreads();
            sh_scan[threadIdx.x] += add;
            __syncthreads();
        }
        if (c < nc) t.row_ptr[c] = carry + sh_scan[threadIdx.x] - v;
        __syncthreads();
        if (threadIdx.x == blockDim.x - 1) carry += sh_scan[threadIdx.x];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        t.row_ptr[nc] = carry;
        *t.pool_top = t.pool_start;
        if (carry > t.pool_start) bad = 1;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < nc; c += blockDim.x) {
        const int h0 = t.cell_he[c];
        int base = t.row_ptr[c];
        t.row_cap[c] = t.nsides[c] + kRowSlack;
        int wx = 0, wy = 0, h = h0, k = 0;
        do {
            const int32_t *r = t.he + 8 * (int64_t)h;
            if (wx < -1 || wx > 1 || wy < -1 || wy > 1) bad = 1;
            t.corner[base + k] = pack_id(r[HS], wx, wy);
            t.corner_he[base + k] = h;
            wx += r[HOX];
            wy += r[HOY];
            h = r[HN];
            ++k;
        } while (h != h0 && k < 4096);
    }
    __syncthreads();
    return bad;
}

// ------------------------------------------------------------------- HVP
// Directional derivatives of one cell's area and perimeter along v, in the
// precision of the positions:
//   dA = sum_k grad_k A . v_k,  grad_k A = 1/2 R(r_{k+1} - r_{k-1});
//   dP = sum_k u_k . (v_{k+1} - v_k)  (zero-length edges contribute 0).
// Stored as (G, B) = (2 K_A dA, 2 K_P dP).  `corner_at(k)` returns the
// packed corner k of the cell's row, which has n corners.
template <typename PosT, typename M, typename CornerAt>
__device__ __forceinline__ void hvp_cell_row(const DevTissue &t, const PosT *__restrict__ X,
                                             const double *__restrict__ v, int n,
                                             CornerAt corner_at, PosT ka, PosT kp,
                                             M *__restrict__ aux, int c) {
    using C = PosT;
    const PosT Lx = (PosT)t.Lx, Ly = (PosT)t.Ly;
    const int32_t w0 = corner_at(0);
    const auto p0 = ld2(X, id_of(w0));
    auto rel = [&](int k, C &rx, C &ry, C &vx, C &vy) {
        const int32_t w = corner_at(k);
        const int vv = id_of(w);
        if (k == 0) {
            rx = 0;
            ry = 0;
        } else {
            const auto q = ld2(X, vv);
            rx = (C)pdiff<PosT>(q.x, p0.x, ox_of(w), Lx);
            ry = (C)pdiff<PosT>(q.y, p0.y, oy_of(w), Ly);
        }
        const auto vq = ld2(v, vv);
        vx = (C)vq.x;
        vy = (C)vq.y;
    };
    C rpx, rpy, vd0, vd1;
    rel(n - 1, rpx, rpy, vd0, vd1);
    C rcx, rcy, vcx, vcy;
    rel(0, rcx, rcy, vcx, vcy);
    C dA = 0, dP = 0;
    for (int k = 0; k < n; ++k) {
        const int kn = (k + 1 == n) ? 0 : k + 1;
        C rnx, rny, vnx, vny;
        rel(kn, rnx, rny, vnx, vny);
        const C gx = (C)0.5 * (rny - rpy), gy = (C)-0.5 * (rnx - rpx);
        dA += gx * vcx + gy * vcy;
        const C dx = rnx - rcx, dy = rny - rcy;
        const C l2 = dx * dx + dy * dy;
        if (l2 > (C)0) dP += over_len_hvp(dx * (vnx - vcx) + dy * (vny - vcy), l2);
        rpx = rcx;
        rpy = rcy;
        rcx = rnx;
        rcy = rny;
        vcx = vnx;
        vcy = vny;
    }
    st2(aux, c, (M)((C)2 * (C)ka * dA), (M)((C)2 * (C)kp * dP));
}

template <typename PosT, typename M>
__device__ __forceinline__ void hvp_cell_one(const DevTissue &t, const PosT *__restrict__ X,
                                             const DevParams<PosT> &p,
                                             const double *__restrict__ v, M *__restrict__ aux,
                                             int c) {
    const int rb = t.row_ptr[c], n = t.nsides[c];
    hvp_cell_row<PosT, M>(
        t, X, v, n, [&](int k) { return t.corner[rb + k]; }, p.ka(c), p.kp(c), aux, c);
}

// (H v)_i = sum_k [ T_k w_k - u_k (B_k + B_{k-1}) + 1/2 R(d_k)(G_k - G_{k-1})
//                   + 1/2 R(v_{j_k} - v_i)(cA_k - cA_{k-1}) ]
// with w_k = (I - u_k u_k^T)(v_i - v_{j_k}) / l_k, T_k the edge tension
// (lambda_k + cP_k + cP_{k-1}), G = 2K_A dA and B = 2K_P dP of the sector
// cells.  From a star whose entries and gathers are in `L`: returns
// (Hv)_i in (hx, hy) and v_i . (Hv)_i.
template <typename PosT, typename M>
__device__ __forceinline__ double hvp_vertex_star(const DevTissue &t,
                                                  const StarLoad<PosT, M> &L,
                                                  const M *__restrict__ aux,
                                                  const double *__restrict__ v, int i,
                                                  double &hx_out, double &hy_out) {
    Star<PosT, M> s;
    PosT xi, yi;
    star_math<PosT, M, false, true>(t, L, s, xi, yi);
    const auto vi = ld2(v, i);
    M G[3], B[3], vx[3], vy[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const auto g = ld2(aux, L.c[k]);
        G[k] = g.x;
        B[k] = g.y;
        const auto vj = ld2(v, s.nb[k]);
        vx[k] = (M)(vj.x - vi.x);  // v_{j_k} - v_i
        vy[k] = (M)(vj.y - vi.y);
    }
    M hx = 0, hy = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int km = (k + 2) % 3;
        const M T = s.lam[k] + s.cP[k] + s.cP[km];
        const M du = -(vx[k] * s.ux[k] + vy[k] * s.uy[k]);  // (v_i - v_j) . u
        const M wx = (-vx[k] - du * s.ux[k]) * s.inv[k];
        const M wy = (-vy[k] - du * s.uy[k]) * s.inv[k];
        const M Bs = B[k] + B[km];
        const M dG = (M)0.5 * (G[k] - G[km]);
        const M dC = (M)0.5 * (s.cA[k] - s.cA[km]);
        hx += T * wx - s.ux[k] * Bs + dG * s.dy[k] + dC * vy[k];
        hy += T * wy - s.uy[k] * Bs - dG * s.dx[k] - dC * vx[k];
    }
    hx_out = (double)hx;
    hy_out = (double)hy;
    return vi.x * (double)hx + vi.y * (double)hy;
}

// Writes (Hv)_i and returns v_i . (Hv)_i.
template <typename PosT, typename M>
__device__ __forceinline__ double hvp_vertex_one(const DevTissue &t, const PosT *__restrict__ X,
                                                 const DevParams<PosT> &p,
                                                 const M *__restrict__ cap,
                                                 const M *__restrict__ aux,
                                                 const double *__restrict__ v,
                                                 double *__restrict__ Hv, int i) {
    StarLoad<PosT, M> L;
    star_ids<PosT, M>(t, X, i, L);
    star_gather<PosT, M>(X, p, cap, L);
    double hx, hy;
    const double d = hvp_vertex_star<PosT, M>(t, L, aux, v, i, hx, hy);
    st2(Hv, i, hx, hy);
    return d;
}

// ------------------------------------------------------------ contractions
// theta = lambda:  g_e = -(d2E/dX dlambda_e) . mu = -u_e . (mu_tgt - mu_src)
template <typename PosT>
__device__ __forceinline__ double contract_lambda_one(const DevTissue &t, const PosT *X,
                                                      const double *mu, int e) {
    const int32_t *r = t.he + 8 * (int64_t)t.edge_he[e];
    const int s = r[HS], q = r[HG];
    const double dx = pdiff<double>((double)X[2 * (int64_t)q], (double)X[2 * (int64_t)s], r[HOX], t.Lx);
    const double dy = pdiff<double>((double)X[2 * (int64_t)q + 1], (double)X[2 * (int64_t)s + 1], r[HOY], t.Ly);
    const double l = sqrt(dx * dx + dy * dy);
    return l > 0.0 ? -(dx * (mu[2 * (int64_t)q] - mu[2 * (int64_t)s]) +
                       dy * (mu[2 * (int64_t)q + 1] - mu[2 * (int64_t)s + 1])) / l
                   : 0.0;
}

// theta = P0:  g_c = -(d2E/dX dP0_c) . mu = 2 K_P grad P_c . mu
template <typename PosT>
__device__ __forceinline__ double contract_p0_one(const DevTissue &t, const PosT *X,
                                                  const DevParams<PosT> &p, const double *mu,
                                                  int c) {
    const int rb = t.row_ptr[c], n = t.nsides[c];
    double dP = 0.0;
    for (int k = 0; k < n; ++k) {
        const int h = t.corner_he[rb + k];
        const int32_t *r = t.he + 8 * (int64_t)h;
        const int s = r[HS], q = r[HG];
        const double dx = pdiff<double>((double)X[2 * (int64_t)q], (double)X[2 * (int64_t)s], r[HOX], t.Lx);
        const double dy = pdiff<double>((double)X[2 * (int64_t)q + 1], (double)X[2 * (int64_t)s + 1], r[HOY], t.Ly);
        const double l = sqrt(dx * dx + dy * dy);
        if (l > 0.0)
            dP += (dx * (mu[2 * (int64_t)q] - mu[2 * (int64_t)s]) +
                   dy * (mu[2 * (int64_t)q + 1] - mu[2 * (int64_t)s + 1])) / l;
    }
    return 2.0 * (double)p.kp(c) * dP;
}

// Edge length in double from positions of any precision.
template <typename PosT>
__device__ __forceinline__ double edge_len_one(const DevTissue &t, const PosT *X, int e) {
    const int32_t *r = t.he + 8 * (int64_t)t.edge_he[e];
    const int s = r[HS], q = r[HG];
    const double dx = pdiff<double>((double)X[2 * (int64_t)q], (double)X[2 * (int64_t)s], r[HOX], t.Lx);
    const double dy = pdiff<double>((double)X[2 * (int64_t)q + 1], (double)X[2 * (int64_t)s + 1], r[HOY], t.Ly);
    return sqrt(dx * dx + dy * dy);
}

}  // namespace vtx
