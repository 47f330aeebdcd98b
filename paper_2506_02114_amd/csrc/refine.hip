// Cell refinement and the network that predicts it.
//
// The paper apportions each ray-grid cell as two triangles (sec. 3.2); where
// the mapping is strongly curved (next to a star, across a caustic) that
// linear interpolation is coarse.  Plain refinement: a (sub)cell is refined
// if its mapped ears disagree in orientation (a critical curve crosses it) or
// if splitting it 2 x 2 changes its in-map deposits by more than tau times
// its image area (L1 over pixels); a refined cell is replaced by its four
// children, which are tested again down to `max_depth` levels; cells whose
// triangles span more than `window` pixels are left alone.  The map changes
// by (deposits of the leaves - deposits of the cell).
//
// The learned variant runs the test only on the cells a small network
// (12 -> 64 -> 64 -> 1, BF16 weights, FP32 accumulation on the matrix cores)
// flags from each cell's mapped corners and ear signs, plus every folded cell.
#include <algorithm>
#include <cstddef>
#include <vector>

#include "cellfeat.hpp"
#include "colarea.hpp"
#include "shoot_dev.hpp"

namespace mlm {

namespace {

constexpr int RBLK = 64;

// A triangle of the refinement in coordinates local to (ou, ov), an integer
// point at or below its box (so the subtraction is exact): vertices, edge
// slopes and its deposit per unit of covered area, w / S (S its signed
// area; f = 0 for a degenerate or non-finite one, which deposits nothing).
// Its pixel areas are column sums (colarea.hpp): in pixel column i the area
// between rows j and j + 1 is H(j + 1 - ov) - H(j - ov), signed like S.
struct RTri {
    P2 T[3];
    double sv[3], su[3];
    double f;
};

__device__ inline RTri rtri(double u0, double v0, double u1, double v1, double u2, double v2, double ou, double ov,
                            double w)
{
    RTri t;
    const double S = 0.5 * area2(u0, v0, u1, v1, u2, v2);
    t.f = (S != 0.0 && isfinite(S)) ? w / S : 0.0;
    if (t.f == 0.0) return t;
    t.T[0] = P2{u0 - ou, v0 - ov};
    t.T[1] = P2{u1 - ou, v1 - ov};
    t.T[2] = P2{u2 - ou, v2 - ov};
    tri_slopes(t.T, t.sv, t.su);
    return t;
}

// rows per pass of a column's sums (registers hold one pass)
constexpr int RCH = 10;

// adds the deposits of triangle t in pixel column i, rows jc .. jc + nr - 1,
// to acc[0 .. nr)
__device__ inline void column_deposits(const RTri &t, int64_t i, int64_t jc, int nr, double ou, double ov,
                                       double (&acc)[RCH])
{
    if (t.f == 0.0) return;
    ColSegs<double> S;
    const double cl = (double)i - ou;
    col_segments(t.T, t.sv, t.su, cl, cl + 1.0, S);
    double h0 = col_cumulative(S, (double)jc - ov);
#pragma unroll
    for (int k = 0; k < RCH; ++k) {
        if (k < nr) {
            const double h1 = col_cumulative(S, (double)(jc + k + 1) - ov);
            acc[k] += t.f * (h1 - h0);
            h0 = h1;
        }
    }
}

struct RefineArgs {
    double x0, y0, d1, d2;
    LensConst lc;
    MapGeom g;
    int nlevels, L0_exp, p;
    double L0;
    const int32_t *child0, *leaf, *node_leaf;
    const LeafInfo *leaves;
    const double4 *near;
    const double2 *deriv;
    double tau;
    int max_depth, window;
};

// image point (x0 + A d1, y0 + B d2), evaluated as written
__device__ inline void image_point(const RefineArgs &ra, double A, double B, double &x, double &y)
{
#pragma clang fp contract(off)
    x = ra.x0 + A * ra.d1;
    y = ra.y0 + B * ra.d2;
}

// source position (pixel units) of an image point
__device__ inline void shoot_uv(const RefineArgs &ra, double A, double B, double &u, double &v)
{
    double x, y;
    image_point(ra, A, B, x, y);
    const int64_t lf = find_leaf(x, y, ra.nlevels, ra.L0, ra.L0_exp, ra.child0, ra.leaf, ra.node_leaf);
    if (lf < 0) {
        u = v = nan("");
        return;
    }
    const LeafInfo li = ra.leaves[lf];
    double ax, ay;
    leaf_alpha<double>(x - li.cx, y - li.cy, li, ra.near + li.near_off, ra.deriv + lf * ra.p, ra.p, ax, ay);
    double w1, w2;
    double2 uv;
    finish_vertex(ra.lc, ra.g, x, y, ax, ay, w1, w2, uv);
    u = uv.x;
    v = uv.y;
}

struct SubCell {
    double A0, B0, h;
    int d;
    double u[4], v[4];
};

// ray k of the five new ones of a subcell's 3 x 3 grid, in halves of its side:
// (1, 0), (0, 1), (1, 1), (2, 1), (1, 2)
__device__ inline double ray_a(const SubCell &c, int k) { return c.A0 + (k == 1 ? 0.0 : (k == 3 ? c.h : 0.5 * c.h)); }
__device__ inline double ray_b(const SubCell &c, int k) { return c.B0 + (k == 0 ? 0.0 : (k == 4 ? c.h : 0.5 * c.h)); }

// The five rays of a subcell.  They nearly always lie in one leaf, and a
// wavefront's subcells do too: then the leaf's stars and coefficients are read
// once for all of them, as scalars (the lanes of each leaf in turn), and the
// tree is descended once.  The arithmetic is shoot_uv's, in its order: the
// refinement's decisions compare these rays with the grid's.  (Ray by ray, each
// lane loading its own stars, a wavefront's tests took some 13000 instruction
// slots, with this and test_line 3400.)
__device__ inline void shoot_five(const RefineArgs &ra, const SubCell &c, double (&u)[5], double (&v)[5])
{
    double x[5], y[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) image_point(ra, ray_a(c, k), ray_b(c, k), x[k], y[k]);
    int lf = (int)find_leaf(x[2], y[2], ra.nlevels, ra.L0, ra.L0_exp, ra.child0, ra.leaf, ra.node_leaf);
    bool one = lf >= 0;
    if (one) {   // the leaf's square holds the others: the same cell index at its level
        const double cx = ra.leaves[lf].cx, cy = ra.leaves[lf].cy, sc = 0.5 * ra.leaves[lf].invL;
        const double i = floor((cx + ra.L0) * sc), j = floor((cy + ra.L0) * sc);
#pragma unroll
        for (int k = 0; k < 5; ++k)
            one = one && floor((x[k] + ra.L0) * sc) == i && floor((y[k] + ra.L0) * sc) == j;
    }
    bool todo = one;
    double ax[5], ay[5];
    while (__any(todo)) {
        const uint64_t m = __ballot(todo);
        if (!(todo && lf == __builtin_amdgcn_readlane(lf, __ffsll((unsigned long long)m) - 1))) continue;
        // wavefront-uniform to the compiler too (the lanes here share lf, and it
        // would put that, a vector, in the place of the lane read above)
        const int ul = __builtin_amdgcn_readfirstlane(lf);
        // (read as constant memory, so that the wavefront's loads are scalar ones)
        using CD = const __attribute__((address_space(4))) double;
        using CI = const __attribute__((address_space(4))) int32_t;
        CD *lp = (CD *)(ra.leaves + ul);
        const struct {
            double cx, cy, invL;
            int32_t near_cnt;
        } li{lp[offsetof(LeafInfo, cx) / 8], lp[offsetof(LeafInfo, cy) / 8], lp[offsetof(LeafInfo, invL) / 8],
             ((CI *)lp)[offsetof(LeafInfo, near_cnt) / 4]};
        CD *ns = (CD *)(ra.near + ((CI *)lp)[offsetof(LeafInfo, near_off) / 4]);
        CD *dv = (CD *)(ra.deriv + (int64_t)ul * ra.p);
#pragma unroll
        for (int k = 0; k < 5; ++k) ax[k] = ay[k] = 0.0;
#pragma unroll 2
        for (int32_t s = 0; s < li.near_cnt; ++s) {
            const double4 st = make_double4(ns[4 * s], ns[4 * s + 1], ns[4 * s + 2], 0.0);
#pragma unroll
            for (int k = 0; k < 5; ++k) near_star<double>(x[k] - li.cx, y[k] - li.cy, st, ax[k], ay[k]);
        }
        double sr[5], si[5];
        double zr[5], zi[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            sr[k] = dv[2 * ra.p - 2];
            si[k] = dv[2 * ra.p - 1];
            zr[k] = (x[k] - li.cx) * li.invL;
            zi[k] = (y[k] - li.cy) * li.invL;
        }
#pragma unroll 2
        for (int l = ra.p - 2; l >= 0; --l) {
            const double2 cf = make_double2(dv[2 * l], dv[2 * l + 1]);
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                const double nr = sr[k] * zr[k] - si[k] * zi[k] + cf.x;
                const double ni = sr[k] * zi[k] + si[k] * zr[k] + cf.y;
                sr[k] = nr;
                si[k] = ni;
            }
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            ax[k] += sr[k];
            ay[k] -= si[k];
        }
        todo = false;
    }
    // (behind the loop: inside it the compiler lifts the rectangular sheet's
    // logarithms, which need no leaf, out of their branch)
    if (one) {
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            double w1, w2;
            double2 uv;
            finish_vertex(ra.lc, ra.g, x[k], y[k], ax[k], ay[k], w1, w2, uv);
            u[k] = uv.x;
            v[k] = uv.y;
        }
    } else {
#pragma unroll 1
        for (int k = 0; k < 5; ++k) {
            double uk, vk;
            shoot_uv(ra, ray_a(c, k), ray_b(c, k), uk, vk);
#pragma unroll
            for (int m = 0; m < 5; ++m)
                if (m == k) {
                    u[m] = uk;
                    v[m] = vk;
                }
        }
    }
}

// the subcell's 3 x 3 grid of source points: its corners and five new rays
__device__ inline void fill_grid(const RefineArgs &ra, const SubCell &c, double (&gu)[3][3], double (&gv)[3][3])
{
    double u[5], v[5];
    shoot_five(ra, c, u, v);
    gu[0][0] = c.u[0]; gv[0][0] = c.v[0];
    gu[0][2] = c.u[1]; gv[0][2] = c.v[1];
    gu[2][2] = c.u[2]; gv[2][2] = c.v[2];
    gu[2][0] = c.u[3]; gv[2][0] = c.v[3];
    gu[0][1] = u[0]; gv[0][1] = v[0];
    gu[1][0] = u[1]; gv[1][0] = v[1];
    gu[1][1] = u[2]; gv[1][1] = v[2];
    gu[1][2] = u[3]; gv[1][2] = v[3];
    gu[2][1] = u[4]; gv[2][1] = v[4];
}

// triangle t of a refinement test: t = 0, 1 the (sub)cell's two, t = 2 ..
// 9 its four children's two each (child (r, s) of the 3 x 3 grid, t = 2 +
// 2 (2 r + s) + k), corners in the cell pass's order
__device__ inline void test_triangle(int t, const SubCell &c, const double (&gu)[3][3], const double (&gv)[3][3],
                                     double &a0, double &b0, double &a1, double &b1, double &a2, double &b2)
{
    switch (t) {
#define MLM_TRI(T, U0, V0, U1, V1, U2, V2) \
    case T: a0 = U0; b0 = V0; a1 = U1; b1 = V1; a2 = U2; b2 = V2; return;
        MLM_TRI(0, c.u[0], c.v[0], c.u[1], c.v[1], c.u[2], c.v[2])
        MLM_TRI(1, c.u[0], c.v[0], c.u[2], c.v[2], c.u[3], c.v[3])
        MLM_TRI(2, gu[0][0], gv[0][0], gu[0][1], gv[0][1], gu[1][1], gv[1][1])
        MLM_TRI(3, gu[0][0], gv[0][0], gu[1][1], gv[1][1], gu[1][0], gv[1][0])
        MLM_TRI(4, gu[0][1], gv[0][1], gu[0][2], gv[0][2], gu[1][2], gv[1][2])
        MLM_TRI(5, gu[0][1], gv[0][1], gu[1][2], gv[1][2], gu[1][1], gv[1][1])
        MLM_TRI(6, gu[1][0], gv[1][0], gu[1][1], gv[1][1], gu[2][1], gv[2][1])
        MLM_TRI(7, gu[1][0], gv[1][0], gu[2][1], gv[2][1], gu[2][0], gv[2][0])
        MLM_TRI(8, gu[1][1], gv[1][1], gu[1][2], gv[1][2], gu[2][2], gv[2][2])
        default: MLM_TRI(9, gu[1][1], gv[1][1], gu[2][2], gv[2][2], gu[2][1], gv[2][1])
#undef MLM_TRI
    }
}

// What the test by one line says: refined or not, or that another test has to
// decide, for a grid within 2 x 2 pixels or for a wider one
enum Verdict { KEEP = 0, REFINE = 1, NEEDS_BOX = 2, NEEDS_COLUMNS = 3 };

// the box of the 3 x 3 grid: whether it is finite and within the window
__device__ inline bool grid_box(const RefineArgs &ra, const double (&gu)[3][3], const double (&gv)[3][3], double &umin,
                                double &umax, double &vmin, double &vmax)
{
    umin = vmin = 1e300;
    umax = vmax = -1e300;
    bool finite = true;
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            finite = finite && isfinite(gu[r][s]) && isfinite(gv[r][s]);
            umin = fmin(umin, gu[r][s]);
            umax = fmax(umax, gu[r][s]);
            vmin = fmin(vmin, gv[r][s]);
            vmax = fmax(vmax, gv[r][s]);
        }
    return finite && umax - umin <= ra.window && vmax - vmin <= ra.window;
}

__device__ inline bool cell_folded(const SubCell &c)
{
    float f[12];
    cell_features(c.u, c.v, f);
    return folded(f);
}

// Calls f(i, j, d) with what splitting the (sub)cell changes in every in-map
// pixel of the grid's box (its children's deposits less its own), for a grid in
// any box: pixel column by column, a pass of RCH rows at a time, one triangle
// after the other (t uniform across the wavefront, so the vertex choice is a
// scalar branch and only one triangle's column state is live)
template <class F>
__device__ inline void split_columns(const RefineArgs &ra, const SubCell &c, const double (&gu)[3][3],
                                     const double (&gv)[3][3], double umin, double umax, double vmin, double vmax, F &&f)
{
    const double w = ra.g.tri_weight * c.h * c.h;   // parent triangle weight
    const double ou = floor(umin), ov = floor(vmin);
    const int64_t i0 = max((int64_t)ou, (int64_t)0), i1 = min((int64_t)floor(umax), (int64_t)ra.g.n1 - 1);
    const int64_t j0 = max((int64_t)ov, (int64_t)0), j1 = min((int64_t)floor(vmax), (int64_t)ra.g.n2 - 1);
    for (int64_t jc = j0; jc <= j1; jc += RCH) {
        const int nr = (int)min((int64_t)RCH, j1 - jc + 1);
        for (int64_t i = i0; i <= i1; ++i) {
            double diff[RCH];
#pragma unroll
            for (int k = 0; k < RCH; ++k) diff[k] = 0.0;
#pragma unroll 1
            for (int t = 0; t < 10; ++t) {
                double a0, b0, a1, b1, a2, b2;
                test_triangle(t, c, gu, gv, a0, b0, a1, b1, a2, b2);
                column_deposits(rtri(a0, b0, a1, b1, a2, b2, ou, ov, t < 2 ? -w : 0.25 * w), i, jc, nr, ou, ov,
                                diff);
            }
#pragma unroll
            for (int k = 0; k < RCH; ++k)
                if (k < nr) f(i, jc + k, diff[k]);
        }
    }
}

// share of a triangle's area where x < 1 (x: its vertices' coordinates relative
// to the box): the line cuts the corner at the lone vertex, (1 - x0)^2 / ((x1 -
// x0) (x2 - x0)) of the area
__device__ inline double line_share(double a, double b, double c)
{
    const double lo = lesser(a, b), hi = greater(a, b);
    const double mn = lesser(lo, c), mx = greater(hi, c), md = greater(lo, lesser(hi, c));
    const bool low = md < 1.0;
    const double e = low ? mx - 1.0 : 1.0 - mn, h = low ? mx - md : md - mn;
    const double q = fdiv(e * e, (mx - mn) * h);
    return mx < 1.0 ? 1.0 : (mn >= 1.0 ? 0.0 : (low ? 1.0 - q : q));
}

// The test of a grid within two pixels: one pixel line at most crosses it, so a
// triangle's deposits are its shares on either side.  Five of six tests are of
// this kind, and their ten triangles cost 30 instructions each instead of 220 a
// pixel column.
__device__ inline Verdict test_line(const RefineArgs &ra, const SubCell &c, const double (&gu)[3][3],
                                    const double (&gv)[3][3], double umin, double umax, double vmin, double vmax)
{
    const double fu = floor(umin), fv = floor(vmin);
    const bool two_u = umax - fu >= 1.0, two_v = vmax - fv >= 1.0;
    if (!(umax - fu < 2.0 && vmax - fv < 2.0)) return NEEDS_COLUMNS;
    if (two_u && two_v) return NEEDS_BOX;
    // the first pixel and, where a line crosses the grid, the one beyond
    const double i = fu, j = fv, i2 = fu + (two_u ? 1.0 : 0.0), j2 = fv + (two_v ? 1.0 : 0.0);
    const double n1 = ra.g.n1, n2 = ra.g.n2;
    const bool in1 = i >= 0.0 && j >= 0.0 && i < n1 && j < n2;
    const bool in2 = (two_u || two_v) && i2 >= 0.0 && j2 >= 0.0 && i2 < n1 && j2 < n2;
    const double o = two_v ? fv : fu;
    double d1 = 0.0, d2 = 0.0;   // (children's deposits - the cell's) in units of its triangle weight
#pragma unroll
    for (int t = 0; t < 10; ++t) {
        double a0, b0, a1, b1, a2, b2;
        test_triangle(t, c, gu, gv, a0, b0, a1, b1, a2, b2);
        const double S = area2(a0, b0, a1, b1, a2, b2);
        const double x0 = (two_v ? b0 : a0) - o, x1 = (two_v ? b1 : a1) - o, x2 = (two_v ? b2 : a2) - o;
        const double f = S != 0.0 ? (t < 2 ? -1.0 : 0.25) : 0.0, q = line_share(x0, x1, x2);
        d1 += f * q;
        d2 += f * (1.0 - q);
    }
    const double l1 = (in1 ? fabs(d1) : 0.0) + (in2 ? fabs(d2) : 0.0);
    return l1 > ra.tau * 2.0 ? REFINE : KEEP;
}

// The same for a grid within the 2 x 2 pixels from (fu, fv): d[0 .. 4) what
// splitting changes in the pixels (0, 0), (1, 0), (0, 1), (1, 1) of the box, in
// units of the cell's triangle weight.  A triangle's share left of u = 1 and
// below v = 1 is that of the corner u = 1 cuts off, clipped at v = 1 (or, the
// corner lying right of it, the share below v = 1 less that).
__device__ inline void split_box(const SubCell &c, const double (&gu)[3][3], const double (&gv)[3][3], double fu,
                                 double fv, double (&d)[4])
{
    d[0] = d[1] = d[2] = d[3] = 0.0;
#pragma unroll 1
    for (int t = 0; t < 10; ++t) {
        double a0, b0, a1, b1, a2, b2;
        test_triangle(t, c, gu, gv, a0, b0, a1, b1, a2, b2);
        const double f = area2(a0, b0, a1, b1, a2, b2) != 0.0 ? (t < 2 ? -1.0 : 0.25) : 0.0;
        a0 -= fu; a1 -= fu; a2 -= fu;
        b0 -= fv; b1 -= fv; b2 -= fv;
        const double l = line_share(a0, a1, a2), h = line_share(b0, b1, b2);
        double q = l * h;   // one of them 0 or 1
        if (l > 0.0 && l < 1.0 && h > 0.0 && h < 1.0) {
            const bool la = a0 < 1.0, lb = a1 < 1.0, lc = a2 < 1.0;
            const double p0 = lb == lc ? a0 : (la == lc ? a1 : a2), r0 = lb == lc ? b0 : (la == lc ? b1 : b2);
            const double p1 = lb == lc ? a1 : (la == lc ? a2 : a0), r1 = lb == lc ? b1 : (la == lc ? b2 : b0);
            const double p2 = lb == lc ? a2 : (la == lc ? a0 : a1), r2 = lb == lc ? b2 : (la == lc ? b0 : b1);
            const double t1 = fdiv(1.0 - p0, p1 - p0), t2 = fdiv(1.0 - p0, p2 - p0);
            const double k = t1 * t2 * line_share(r0, r0 + t1 * (r1 - r0), r0 + t2 * (r2 - r0));
            q = p0 < 1.0 ? k : h - k;
        }
        d[0] += f * q;
        d[1] += f * (h - q);
        d[2] += f * (l - q);
        d[3] += f * ((1.0 - l) - (h - q));
    }
}

// the test by the 2 x 2 pixels of the box
__device__ inline bool test_box(const RefineArgs &ra, const SubCell &c, const double (&gu)[3][3],
                                const double (&gv)[3][3], double umin, double vmin)
{
    const double fu = floor(umin), fv = floor(vmin), n1 = ra.g.n1, n2 = ra.g.n2;
    double d[4], l1 = 0.0;
    split_box(c, gu, gv, fu, fv, d);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double i = fu + (k & 1), j = fv + (k >> 1);
        if (i >= 0.0 && j >= 0.0 && i < n1 && j < n2) l1 += fabs(d[k]);
    }
    return l1 > ra.tau * 2.0;
}

// the test of a grid of any width
__device__ inline bool test_columns(const RefineArgs &ra, const SubCell &c, const double (&gu)[3][3],
                                    const double (&gv)[3][3], double umin, double umax, double vmin, double vmax)
{
    double l1 = 0.0;
    split_columns(ra, c, gu, gv, umin, umax, vmin, vmax, [&](int64_t, int64_t, double d) { l1 += fabs(d); });
    return l1 > ra.tau * 2.0 * (ra.g.tri_weight * c.h * c.h);
}

// The test of one subcell by its 3 x 3 grid of source points (corners from the
// subcell, five new rays): whether it is refined.  (The tests of grids in a 2 x 2 box
// and of wider ones in launches of their own, on gathered items whose rays had to be
// shot again, were the faster way only while a lane loaded its own stars: one-level
// refinement of 200 x 200 pixels at 8, 256 and 4096 cells a pixel takes 1.26, 6.1 and
// 39 ms so and 0.80, 5.2 and 33 here, the learned refinement of a 400 x 400 map 89
// and 83.)
__device__ inline bool refine_test(const RefineArgs &ra, const SubCell &c, int &too_large)
{
    double gu[3][3], gv[3][3], umin, umax, vmin, vmax;
    fill_grid(ra, c, gu, gv);
    if (!grid_box(ra, gu, gv, umin, umax, vmin, vmax)) {
        too_large = 1;
        return false;
    }
    if (cell_folded(c)) return true;
    const Verdict v = test_line(ra, c, gu, gv, umin, umax, vmin, vmax);
    if (v == NEEDS_BOX) return test_box(ra, c, gu, gv, umin, vmin);
    if (v == NEEDS_COLUMNS) return test_columns(ra, c, gu, gv, umin, umax, vmin, vmax);
    return v == REFINE;
}

// Refinement level by level (breadth first): every (sub)cell of a level is
// one thread of k_refine_test, which only decides; the few refined ones are
// numbered by a scan and expanded by k_refine_expand, which moves their
// deposits to their four children and lists the children for the next
// level.  Lanes of a wavefront so do equal work, where one thread walking a
// cell's whole subtree kept the other lanes waiting.
//
// A level's items are either candidate cells (cand: a + (nr1 - 1) b, corners
// from the strip's vertices) or a list of subcells.
__device__ inline SubCell level_item(int64_t t, const int64_t *__restrict__ cand, const SubCell *__restrict__ list,
                                     int64_t nr1, int64_t vb0, const double2 *__restrict__ verts)
{
    if (list) return list[t];
    SubCell c;
    // (a strip's cells number fewer than 2^32: its first row is vb0)
    const uint32_t cell = (uint32_t)(cand[t] - (nr1 - 1) * vb0), ncol = (uint32_t)(nr1 - 1);
    const int64_t a = cell % ncol, b = vb0 + cell / ncol;
    c.A0 = (double)a;
    c.B0 = (double)b;
    c.h = 1.0;
    c.d = 0;
    const double2 *r0 = verts + (b - vb0) * nr1, *r1 = r0 + nr1;
    const double2 q[4] = {r0[a], r0[a + 1], r1[a + 1], r1[a]};
    for (int m = 0; m < 4; ++m) {
        c.u[m] = q[m].x;
        c.v[m] = q[m].y;
    }
    return c;
}

// counts of a wavefront's items added to its workgroup's slot of stats: [0]
// tested, [1] refined, [2] too large (one atomic per wavefront each; at one
// address for all, some 5 ns each, they took two thirds of the test's time)
__device__ inline void add_stats(unsigned long long *__restrict__ stats, int tested, int refined, int large)
{
    int v[3] = {tested, refined, large};
    stats += (size_t)(blockIdx.x % REFINE_SLOTS) * REFINE_STRIDE;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
        if ((threadIdx.x & 63) == 0 && v[k]) atomicAdd(stats + k, (unsigned long long)v[k]);
    }
}

// The refined items of a level, 64 items a mask (a workgroup's), with their number
// (a scan of these, and not of a flag per item, numbers them: with 4-byte flags and
// 8-byte places of every item, numbering the cells and subcells of the learned
// refinement of a 400 x 400 map moved 17 GB).  Bound by instruction issue.
static_assert(RBLK == 64, "a workgroup is a mask");
__global__ __launch_bounds__(RBLK) __attribute__((amdgpu_waves_per_eu(3))) void k_refine_test(RefineArgs ra, int64_t n, const int64_t *__restrict__ cand,
                                                      const SubCell *__restrict__ list, int64_t nr1, int64_t vb0,
                                                      const double2 *__restrict__ verts, uint64_t *__restrict__ mask,
                                                      int32_t *__restrict__ cnt, unsigned long long *__restrict__ stats)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int large = 0;
    bool yes = false;
    if (t < n) yes = refine_test(ra, level_item(t, cand, list, nr1, vb0, verts), large);
    const uint64_t m = __ballot(yes);
    if (threadIdx.x == 0) {
        mask[blockIdx.x] = m;
        cnt[blockIdx.x] = __popcll(m);
    }
    add_stats(stats, t < n ? 1 : 0, yes ? 1 : 0, large);
}

// item[..] = base + t for the flagged t in order (pos: exclusive scan of the
// masks' counts); with mask == NULL for every t
__global__ __launch_bounds__(256) void k_list_flagged(int64_t n, const uint64_t *__restrict__ mask,
                                                      const int64_t *__restrict__ pos, int64_t base,
                                                      int64_t *__restrict__ item)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    if (!mask) {
        item[t] = base + t;
        return;
    }
    const uint64_t m = mask[t >> 6], bit = 1ull << (t & 63);
    if (m & bit) item[pos[t >> 6] + __popcll(m & (bit - 1ull))] = base + t;
}

// the k-th refined item, k < n: the map loses its deposits and gains its four
// children's, and the children are written to out[4 k .. 4 k + 3].  (Over all
// the items of a level, a refined one in thirty, this took as long as 0.6 of
// the tests.)
__global__ __launch_bounds__(RBLK) void k_refine_expand(RefineArgs ra, int64_t n, const int64_t *__restrict__ item,
                                                        const int64_t *__restrict__ cand,
                                                        const SubCell *__restrict__ list, int64_t nr1, int64_t vb0,
                                                        const double2 *__restrict__ verts, double *__restrict__ map,
                                                        SubCell *__restrict__ out)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const SubCell c = level_item(item[k], cand, list, nr1, vb0, verts);
    double gu[3][3], gv[3][3];
    fill_grid(ra, c, gu, gv);
    const double hh = 0.5 * c.h;
    SubCell *dst = out + 4 * k;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            SubCell ch;
            ch.A0 = c.A0 + s * hh;
            ch.B0 = c.B0 + r * hh;
            ch.h = hh;
            ch.d = c.d + 1;
            const double cu[4] = {gu[r][s], gu[r][s + 1], gu[r + 1][s + 1], gu[r + 1][s]};
            const double cv[4] = {gv[r][s], gv[r][s + 1], gv[r + 1][s + 1], gv[r + 1][s]};
            for (int m = 0; m < 4; ++m) {
                ch.u[m] = cu[m];
                ch.v[m] = cv[m];
            }
            dst[2 * r + s] = ch;
        }
    // the change per pixel (a refined child takes its own back), summed over the
    // ten triangles before it goes to the map: neighbouring cells meet at a few
    // pixels, and their atomics there were what the pass waited for
    double umin, umax, vmin, vmax;
    (void)grid_box(ra, gu, gv, umin, umax, vmin, vmax);
    const double fu = floor(umin), fv = floor(vmin), n1 = ra.g.n1, n2 = ra.g.n2;
    if (umax - fu < 2.0 && vmax - fv < 2.0) {
        const double w = ra.g.tri_weight * c.h * c.h;
        double d[4];
        split_box(c, gu, gv, fu, fv, d);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const double i = fu + (m & 1), j = fv + (m >> 1);
            if (d[m] != 0.0 && i >= 0.0 && j >= 0.0 && i < n1 && j < n2)
                unsafeAtomicAdd(map + (int64_t)j * ra.g.n1 + (int64_t)i, d[m] * w);
        }
    } else {
        split_columns(ra, c, gu, gv, umin, umax, vmin, vmax, [&](int64_t i, int64_t j, double d) {
            if (d != 0.0) unsafeAtomicAdd(map + j * (int64_t)ra.g.n1 + i, d);
        });
    }
}

// features of arbitrary cells, corners shot on the spot
__global__ __launch_bounds__(RBLK) void k_sample_features(RefineArgs ra, int64_t n, const int64_t *__restrict__ ab,
                                                          float *__restrict__ feats)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const double A = (double)ab[2 * t], B = (double)ab[2 * t + 1];
    double u4[4], v4[4];
    shoot_uv(ra, A, B, u4[0], v4[0]);
    shoot_uv(ra, A + 1.0, B, u4[1], v4[1]);
    shoot_uv(ra, A + 1.0, B + 1.0, u4[2], v4[2]);
    shoot_uv(ra, A, B + 1.0, u4[3], v4[3]);
    float f[12];
    cell_features(u4, v4, f);
    for (int m = 0; m < 12; ++m) feats[t * 12 + m] = isfinite(f[m]) ? f[m] : 0.0f;
}

// the refinement test at depth 0 of arbitrary cells (labels only)
__global__ __launch_bounds__(RBLK) __attribute__((amdgpu_waves_per_eu(3))) void k_sample_labels(RefineArgs ra, int64_t n, const int64_t *__restrict__ ab,
                                                        uint8_t *__restrict__ label)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    SubCell c;
    c.A0 = (double)ab[2 * t];
    c.B0 = (double)ab[2 * t + 1];
    c.h = 1.0;
    c.d = 0;
    shoot_uv(ra, c.A0, c.B0, c.u[0], c.v[0]);
    shoot_uv(ra, c.A0 + 1.0, c.B0, c.u[1], c.v[1]);
    shoot_uv(ra, c.A0 + 1.0, c.B0 + 1.0, c.u[2], c.v[2]);
    shoot_uv(ra, c.A0, c.B0 + 1.0, c.u[3], c.v[3]);
    int large = 0;
    label[t] = refine_test(ra, c, large) ? 1 : 0;
}

}  // namespace

RefineArgs make_refine_args(const Tree &T, const Region &R, const LensConst &lc, const MapGeom &g, double tau,
                            int max_depth, int window)
{
    RefineArgs ra{};
    ra.x0 = R.x0;
    ra.y0 = R.y0;
    ra.d1 = R.d1;
    ra.d2 = R.d2;
    ra.lc = lc;
    ra.g = g;
    ra.nlevels = T.nlevels;
    ra.L0_exp = T.L0_exp;
    ra.p = T.p;
    ra.L0 = T.L0;
    ra.child0 = T.child0;
    ra.leaf = T.leaf;
    ra.node_leaf = T.node_leaf;
    ra.leaves = T.leaves;
    ra.near = T.near;
    ra.deriv = T.deriv;
    ra.tau = tau;
    ra.max_depth = max_depth;
    ra.window = window;
    return ra;
}

size_t refine_subcell_bytes() { return sizeof(SubCell); }

void launch_refine_test(const Tree &T, const Region &R, const LensConst &lc, const MapGeom &g, double tau, int depth,
                        int window, int64_t n, const int64_t *cand, const void *list, int64_t nr1, int64_t vb0,
                        const double2 *verts, uint64_t *mask, int32_t *cnt, unsigned long long *stats, hipStream_t st)
{
    if (n <= 0) return;
    const RefineArgs ra = make_refine_args(T, R, lc, g, tau, depth, window);
    hipLaunchKernelGGL(k_refine_test, dim3((unsigned)((n + RBLK - 1) / RBLK)), dim3(RBLK), 0, st, ra, n, cand,
                       static_cast<const SubCell *>(list), nr1, vb0, verts, mask, cnt, stats);
}

void launch_refine_expand(const Tree &T, const Region &R, const LensConst &lc, const MapGeom &g, double tau, int depth,
                          int window, int64_t nref, const int64_t *cand, const void *list, int64_t nr1, int64_t vb0,
                          const double2 *verts, const int64_t *item, double *map, void *out, hipStream_t st)
{
    if (nref <= 0) return;
    const RefineArgs ra = make_refine_args(T, R, lc, g, tau, depth, window);
    hipLaunchKernelGGL(k_refine_expand, dim3((unsigned)((nref + RBLK - 1) / RBLK)), dim3(RBLK), 0, st, ra, nref, item,
                       cand, static_cast<const SubCell *>(list), nr1, vb0, verts, map, static_cast<SubCell *>(out));
}

void launch_sample_features(const Tree &T, const Region &R, const LensConst &lc, const MapGeom &g, int64_t n,
                            const int64_t *ab, float *feats, hipStream_t st)
{
    if (n <= 0) return;
    const RefineArgs ra = make_refine_args(T, R, lc, g, 0.0, 1, 1);
    hipLaunchKernelGGL(k_sample_features, dim3((unsigned)((n + RBLK - 1) / RBLK)), dim3(RBLK), 0, st, ra, n, ab,
                       feats);
}

void launch_sample_labels(const Tree &T, const Region &R, const LensConst &lc, const MapGeom &g, double tau,
                          int window, int64_t n, const int64_t *ab, uint8_t *label, hipStream_t st)
{
    if (n <= 0) return;
    const RefineArgs ra = make_refine_args(T, R, lc, g, tau, 1, window);
    hipLaunchKernelGGL(k_sample_labels, dim3((unsigned)((n + RBLK - 1) / RBLK)), dim3(RBLK), 0, st, ra, n, ab, label);
}

void launch_list_flagged(int64_t n, const uint64_t *mask, const int64_t *pos, int64_t base, int64_t *item, hipStream_t st)
{
    if (n > 0)
        hipLaunchKernelGGL(k_list_flagged, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, mask, pos, base, item);
}

}  // namespace mlm
