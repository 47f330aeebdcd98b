// Ray shooting by patches, for grids whose rays lie far closer together than
// the stars.  A ray of k_shoot sums its leaf's ~14 near stars and ~20 Taylor
// terms; where a leaf holds thousands of rays, the field over a PATCH of P x P
// neighbouring rays is one power series of few terms about the patch's centre:
// the leaf's Taylor series re-expanded there, plus each near star's
// m / (z - z_i) = (m / w0) sum_k (-t / w0)^k, w0 the centre's offset from the
// star, t the ray's from the centre.  k_patch_coef forms each patch's
// coefficients once for its P^2 rays; k_shoot_patch and k_irs_patch evaluate
// them.  Stars too close to the patch for that are summed directly, ray by
// ray, and patches that a smooth sheet's edge crosses (or that any other limit
// excludes) go ray by ray altogether, as k_shoot does.
//
// Every series is cut where its remainder is below half a unit in the last
// place of the rays' own positions, so the result differs from k_shoot's by
// rounding only.
//
// Rays come in pairs +t, -t about the patch's centre: with E and O the even
// and odd parts of the series, f(+-t) = E(t^2) +- t O(t^2), so a ray costs two
// multiply-adds a term instead of four.  The coefficients are
// wavefront-uniform and reach the vector units as scalars.
#include <algorithm>
#include <cmath>

#include "shoot_dev.hpp"

namespace mlm {

namespace {

// rays per leaf from which patches pay: few rays, many rays
constexpr double PATCH_RAYS_PER_LEAF[2] = {32768.0, 10000.0}, PATCH_MANY_RAYS = 3.2e7;
constexpr double LARGE_PATCH_RAYS_PER_LEAF = 262144.0;   // (many rays alone)
constexpr double SMALL_PATCH_RAYS_PER_LEAF[2] = {8192.0, 3000.0}, SMALL_PATCH_MANY_RAYS = 1.6e7;
constexpr int PC_MAX = 24;    // most coefficients of a patch
constexpr int PC_DIRECT = 8;  // most stars summed directly
constexpr int PC_STARS = 64;  // most near stars of a leaf in this path
// A patch begins at a leaf's first rays and may reach far beyond a leaf that is
// smaller (next to a tight group of stars).  The leaf's series, good within the
// leaf, is there a sum of huge terms that cancel, and so are the patch's
// coefficients: over 16 x 16 rays a leaf 2 rays wide came out 2e-3 off, one of 1
// ray worthless.  Their rounding grows with the sum of the terms' magnitudes at the
// patch's far end; where that passes PC_REACH times the same sum at the leaf's
// corner plus the size of the positions, the rays' own rounding, the patch goes ray
// by ray.  (Over 1.2e7 patches among evenly spread stars the quotient was below 0.5
// everywhere, so none of them does.  It is not formed for a patch within two
// half-lengths: the stars of a leaf's series lie three away at least, so its terms
// are at most a few times those at the corner there.)
constexpr double PC_REACH = 2.0;
// cost in vector instructions of one more coefficient and of a direct star,
// per ray: what the number of coefficients is chosen by
constexpr int COST_COEF = 2, COST_STAR = 18;

struct PatchHead {
    int32_t lf, a0, b0, nanb;      // leaf, first column and row, columns | rows << 16 inside the leaf
    int32_t n, ndir, lin, pad;     // coefficients (0: ray by ray), direct stars, sheet's linear part (PatchLin)
};
struct PatchInfo : PatchHead {
    int32_t dir[PC_DIRECT];        // direct stars (indices into the leaf's near stars)
};
enum PatchLin { LIN_NONE = 0, LIN_DISC = 1, LIN_RECT = 2 };

// the tree as find_leaf goes down it
struct LeafFinder {
    int nlevels, L0_exp;
    double L0;
    const int32_t *child0, *leaf, *node_leaf;
};

struct PatchArgs {
    double r, ir;          // a patch's half diagonal (the largest |t|) and its inverse
    double hx, hy;         // half sides
    double span;           // extent of the source-plane map: the scale of the positions' rounding
    double sure;           // inverse ray shooting: largest distance from a pixel's middle (pixels) at which a ray's pixel is certain
};

// coefficients needed for a star (m > 0) at distance |w0| = w from the centre
// so that the remainder m / w eps^n / (1 - eps), eps = r / w, stays below tol
__device__ inline int star_terms(double r, double r2, double m, double tol)
{
    const float iw = (float)(1.0 / sqrt(r2)), eps = (float)r * iw;
    if (!(eps < 0.7f)) return 99;
    const float need = __log2f((float)tol * (1.0f - eps) / ((float)m * iw)) / __log2f(eps);
    return need < 1.0f ? 1 : (need > 90.0f ? 99 : (int)need + 1);
}

// the coefficients of four patches per wavefront, sixteen lanes each: lane j
// of a patch holds coefficients j and 16 + j, and takes near stars j, 16 + j, ...
template <int P>
__global__ __launch_bounds__(64) void k_patch_coef(ShootArgs sa, LensConst lc, PatchArgs pa, int64_t npatch,
                                                   const int32_t *__restrict__ tile_leaf,
                                                   const int32_t *__restrict__ tile_off,
                                                   const LeafInfo *__restrict__ leaves,
                                                   const double4 *__restrict__ near,
                                                   const double2 *__restrict__ deriv,
                                                   const double *__restrict__ binom, PatchInfo *__restrict__ info,
                                                   double2 *__restrict__ coef)
{
    __shared__ double2 pw[8][65];   // powers of eight orders, one column per lane
    const int lane = threadIdx.x, g = lane >> 4, j = lane & 15;
    const int64_t t = (int64_t)blockIdx.x * 4 + g, tt = t < npatch ? t : npatch - 1;
    const int32_t lf = tile_leaf[tt];
    const LeafInfo li = leaves[lf];
    const int32_t local = (int32_t)tt - tile_off[lf];
    const int32_t ty = local / li.ntx, tx = local - ty * li.ntx;
    const int32_t a0 = li.a_lo + tx * P, b0 = li.b_lo + ty * P;
    const double px = grid_pos(sa.x0, sa.d1, a0, sa.h + 0.5 * (P - 1));
    const double py = grid_pos(sa.y0, sa.d2, b0, sa.h + 0.5 * (P - 1));
    const double sx = px - li.cx, sy = py - li.cy;
    const double r = pa.r;
    // half a unit in the last place of the positions, over what may share it
    const double tol = 0x1p-53 * (fabs(px) + fabs(py) + pa.span) * (1.0 / 16.0);
    const uint64_t sub = 0xffffull << (16 * g);

    // the leaf's Taylor series about the patch's centre:
    // D_j = rho^j sum_{l >= j} C(l, j) d_l s^(l - j), Horner in s
    const int p = sa.p;
    double2 D0 = make_double2(0, 0), D1 = make_double2(0, 0);
    bool general = li.near_cnt > PC_STARS;   // whether the patch goes ray by ray
    {
        const double sr = sx * li.invL, si = sy * li.invL, rho = r * li.invL;
        const double2 *dv = deriv + (int64_t)lf * p;
        const double s2 = sr * sr + si * si, room = 2.0 - rho;
        if (__any(room < 0.0 || s2 > room * room)) {
            const double reach = sqrt(s2) + rho;
            // the terms' magnitudes at the patch's far end and at the leaf's corner
            double far_end = 0.0, corner = 0.0;
            for (int l = p - 1; l >= 0; --l) {
                const double2 d = dv[l];
                const double a = fabs(d.x) + fabs(d.y);
                far_end = fma(far_end, reach, a);
                corner = fma(corner, M_SQRT2, a);
            }
            general = general || !(far_end <= PC_REACH * (corner + fabs(px) + fabs(py) + pa.span));   // (true for NaN)
        }
        for (int l = p - 1; l >= 0; --l) {
            const double2 d = dv[l];
            if (l >= j) {
                const double c = binom[l * 32 + j];
                const double nr = D0.x * sr - D0.y * si + c * d.x;
                D0.y = D0.x * si + D0.y * sr + c * d.y;
                D0.x = nr;
            }
            if (l >= j + 16) {
                const double c = binom[l * 32 + 16 + j];
                const double nr = D1.x * sr - D1.y * si + c * d.x;
                D1.y = D1.x * si + D1.y * sr + c * d.y;
                D1.x = nr;
            }
        }
        double f = 1.0, b = rho;
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            if (k == 4) D1 = cscale(D1, f * b);
            else if (j >> k & 1) f *= b;
            b *= b;
        }
        D0 = cscale(D0, f);
    }
    const uint64_t h0 = (__ballot(fabs(D0.x) + fabs(D0.y) > tol) & sub) >> (16 * g);
    const uint64_t h1 = (__ballot(fabs(D1.x) + fabs(D1.y) > tol) & sub) >> (16 * g);
    int nmin = h1 ? 16 + 64 - __clzll(h1) : (h0 ? 64 - __clzll(h0) : 0);   // coefficients the far field needs

    // the smooth sheet: inside it a linear term (and, for the rectangle, the
    // corners' logarithms); outside the disc the field of its whole mass at
    // the origin; a patch its edge crosses goes ray by ray
    int lin = LIN_NONE;
    double xx = 0, xy = 0, xm = 0, xs = 0;   // this lane's extra pole: offset, mass (disc) or sign (corner)
    if (lc.sheet == 1) {
        const double d = sqrt(px * px + py * py), R = sqrt(lc.r_star2);
        if (d + r < R) {
            lin = LIN_DISC;
        } else if (d - r > R) {
            if (j == 0) {
                xx = px;
                xy = py;
                xm = -lc.kappa_star * lc.r_star2;
            }
        } else {
            general = true;
        }
    } else if (lc.sheet == 2) {
        if (fabs(px) + pa.hx < lc.c1 && fabs(py) + pa.hy < lc.c2) {
            lin = LIN_RECT;
            if (j < 4) {   // t = conj(c) - z, c - z, -conj(c) - z, -c - z
                xx = (j < 2 ? lc.c1 : -lc.c1) - px;
                xy = (j == 1 || j == 2 ? lc.c2 : -lc.c2) - py;
                xs = j & 1 ? -1.0 : 1.0;
            }
        } else {
            general = true;
        }
    }
    const double xr2 = xx * xx + xy * xy;
    int xneed = 0;
    if (xm != 0.0) xneed = star_terms(r, xr2, -xm, tol);
    else if (xs != 0.0) xneed = star_terms(r, xr2, lc.kappa_star * xr2, tol);
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) xneed = max(xneed, __shfl_xor(xneed, o, 64));
    nmin = max(nmin, xneed);

    // terms each near star needs; the cheapest number of coefficients
    const double4 *ns = near + li.near_off;
    int need[PC_STARS / 16];
    int cnt[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < PC_STARS / 16; ++c) {
        need[c] = 0;
        const int i = 16 * c + j;
        if (!general && i < li.near_cnt) {
            const double4 s = ns[i];
            const double wx = sx - s.x, wy = sy - s.y;
            need[c] = star_terms(r, wx * wx + wy * wy, s.z, tol);
        }
#pragma unroll
        for (int k = 0; k < 5; ++k) cnt[k] += __popcll(__ballot(need[c] > 8 + 4 * k) & sub);
    }
    int n = 0, best = 1 << 30, ndir = 0;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int nk = 8 + 4 * k, cost = COST_COEF * nk + COST_STAR * cnt[k];
        if (nk >= nmin && cnt[k] <= PC_DIRECT && cost < best) {
            best = cost;
            n = nk;
            ndir = cnt[k];
        }
    }
    if (general) n = 0;

    // the near stars' series, eight orders at a time: each lane writes its
    // star's terms to LDS, then lane j adds up half of its patch's sixteen
    // lanes for order (j & 7)
    int nmax = n;
    nmax = max(nmax, __shfl_xor(nmax, 16, 64));
    nmax = max(nmax, __shfl_xor(nmax, 32, 64));
    int chunks = n > 0 ? (li.near_cnt + 15) / 16 : 0;
    chunks = max(chunks, __shfl_xor(chunks, 16, 64));
    chunks = max(chunks, __shfl_xor(chunks, 32, 64));
    auto add_block = [&](int b) {   // pw holds orders 8 b .. 8 b + 7
        __syncthreads();
        double2 s = make_double2(0, 0);
        const int col = 16 * g + (j & 8);
#pragma unroll
        for (int i = 0; i < 8; ++i) s = cadd(s, pw[j & 7][col + i]);
        s.x += __shfl_xor(s.x, 8, 64);
        s.y += __shfl_xor(s.y, 8, 64);
        if (b == 2) {
            if (j < 8) D1 = cadd(D1, s);
        } else if (j >> 3 == b) {
            D0 = cadd(D0, s);
        }
        __syncthreads();
    };
#pragma unroll
    for (int c = 0; c < PC_STARS / 16; ++c) {
        if (c >= chunks) break;
        double2 term = make_double2(0, 0), u = make_double2(0, 0);
        const int i = 16 * c + j;
        if (i < li.near_cnt && need[c] <= n) {
            const double4 s = ns[i];
            const double wx = sx - s.x, wy = sy - s.y, inv = 1.0 / (wx * wx + wy * wy);
            term = make_double2(s.z * wx * inv, -s.z * wy * inv);   // m / w0
            u = make_double2(-r * wx * inv, r * wy * inv);          // -r / w0
        }
        for (int b = 0; 8 * b < nmax; ++b) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                pw[k][lane] = term;
                term = cmul(term, u);
            }
            add_block(b);
        }
    }
    if (__any(n > 0 && (xm != 0.0 || xs != 0.0))) {
        // the sheet's poles: f = xm / z outside the disc; inside the rectangle
        // f = (i kappa_* / pi) sum_c +-T(t_c), T(t) = t log t, whose series in
        // t = t0 - r tau is T(t0), -(1 + log t0) r, r (r / t0)^(k - 1) / (k (k - 1))
        double2 term = make_double2(0, 0), u = make_double2(0, 0), lead0 = term, lead1 = term;
        const bool use = n > 0 && (xm != 0.0 || xs != 0.0);
        double fac = 0.0;
        if (use) {
            const double inv = 1.0 / xr2;
            if (xs == 0.0) {
                term = make_double2(xm * xx * inv, -xm * xy * inv);
                u = make_double2(-r * xx * inv, r * xy * inv);
            } else {
                fac = xs * lc.kappa_star * (1.0 / M_PI);
                u = make_double2(r * xx * inv, -r * xy * inv);   // r / t0
                const double2 T = t_log_t(xx, xy);
                const double2 L = make_double2(0.5 * log(xr2), atan2(xy, xx));
                lead0 = make_double2(-fac * T.y, fac * T.x);
                lead1 = make_double2(fac * r * L.y, -fac * r * (1.0 + L.x));
                term = make_double2(-fac * r * u.y, fac * r * u.x);   // i fac r (r / t0), order 2 times 2
            }
        }
        for (int b = 0; 8 * b < nmax; ++b) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int o = 8 * b + k;
                if (fac == 0.0) {
                    pw[k][lane] = term;
                    term = cmul(term, u);
                } else if (o < 2) {
                    pw[k][lane] = o == 0 ? lead0 : lead1;
                } else {
                    pw[k][lane] = cscale(term, 1.0 / (double)(o * (o - 1)));
                    term = cmul(term, u);
                }
            }
            add_block(b);
        }
    }
    if (t >= npatch) return;
    double2 *out = coef + t * PC_MAX;
    if (j < n) out[j] = D0;
    if (16 + j < n) out[16 + j] = D1;
    PatchInfo *pi = info + t;
    if (j == 0) {
        pi->lf = lf;
        pi->a0 = a0;
        pi->b0 = b0;
        pi->nanb = min(P, li.na - tx * P) | min(P, li.nb - ty * P) << 16;
        pi->n = n;
        pi->ndir = ndir;
        pi->lin = lin;
        pi->pad = 0;
    }
    if (n > 0) {
        int at = 0;
#pragma unroll
        for (int c = 0; c < PC_STARS / 16; ++c) {
            const uint64_t m = (__ballot(need[c] > n) & sub) >> (16 * g);
            if (need[c] > n) pi->dir[at + __popcll(m & ((1ull << j) - 1ull))] = 16 * c + j;
            at += __popcll(m);
        }
    }
}

// What a wavefront evaluates a patch with: lane (column, row group); a group's
// rows of the patch's upper half, each ray with its mirror image in the lower
template <int P> struct PatchLane {
    static constexpr int GROUPS = 64 / P;              // row groups
    static constexpr int ROWS = P / 2 / GROUPS;        // row pairs of a lane
    static constexpr int SW = ROWS < 2 ? ROWS : 2;     // evaluated together
};

// from a ray's deflection (u, v) to its pixel coordinates: the macro model with
// the sheet's linear part
struct Finish {
    double l1, l2, k1, k2, ip1, ip2;
    __device__ Finish(const LensConst &lc, const MapGeom &g, int lin)
        : l1(lc.lam1), l2(lc.lam2), k1(-g.ylo1), k2(-g.ylo2), ip1(1.0 / g.pix1), ip2(1.0 / g.pix2)
    {
        if (lin == LIN_DISC) {
            l1 += lc.kappa_star;
            l2 += lc.kappa_star;
        } else if (lin == LIN_RECT) {
            l1 += 2.0 * lc.kappa_star;
            k1 += 2.0 * lc.kappa_star * lc.c1;
        }
    }
    __device__ void operator()(const LensConst &lc, double x, double y, double &u, double &v) const
    {
        double w1 = fma(l1, x, k1) - u, w2 = fma(l2, y, k2) - v;
        if (lc.cubic) {
            const double a = lc.psi3[0], b = lc.psi3[1], c = lc.psi3[2], d = lc.psi3[3];
            w1 -= 0.5 * (a * x * x + 2.0 * b * x * y + c * y * y);
            w2 -= 0.5 * (b * x * x + 2.0 * c * x * y + d * y * y);
        }
        u = w1 * ip1;
        v = w2 * ip2;
    }
};

// The pixel coordinates of the rays of a sweep: SW pairs, [2 s] the upper ray
// (row P/2 + row of the patch) and [2 s + 1] its mirror image
template <int P>
__device__ inline void eval_sweep(const ShootArgs &sa, const LensConst &lc, const MapGeom &g, const PatchArgs &pa,
                                  const PatchHead &pi, const int32_t *__restrict__ dir, const LeafInfo &li,
                                  const double4 *__restrict__ ns, const double2 *__restrict__ cf, int col, int row0,
                                  double (&u)[2 * PatchLane<P>::SW], double (&v)[2 * PatchLane<P>::SW])
{
    constexpr int SW = PatchLane<P>::SW;
    const double zr = ((double)col - 0.5 * (P - 1)) * sa.d1 * pa.ir;
    double zi[SW], wr[SW], wi[SW], er[SW], ei[SW], orr[SW], oi[SW];
#pragma unroll
    for (int s = 0; s < SW; ++s) {
        zi[s] = ((double)(row0 + s) + 0.5) * sa.d2 * pa.ir;
        wr[s] = zr * zr - zi[s] * zi[s];
        wi[s] = 2.0 * zr * zi[s];
        er[s] = ei[s] = orr[s] = oi[s] = 0.0;
    }
    for (int k = pi.n - 4; k >= 0; k -= 4) {   // n is a multiple of 4
        const double2 c0 = cf[k], c1 = cf[k + 1], c2 = cf[k + 2], c3 = cf[k + 3];
#pragma unroll
        for (int s = 0; s < SW; ++s) {
            double tr = fma(er[s], wr[s], fma(-ei[s], wi[s], c2.x));
            double ti = fma(er[s], wi[s], fma(ei[s], wr[s], c2.y));
            er[s] = fma(tr, wr[s], fma(-ti, wi[s], c0.x));
            ei[s] = fma(tr, wi[s], fma(ti, wr[s], c0.y));
            tr = fma(orr[s], wr[s], fma(-oi[s], wi[s], c3.x));
            ti = fma(orr[s], wi[s], fma(oi[s], wr[s], c3.y));
            orr[s] = fma(tr, wr[s], fma(-ti, wi[s], c1.x));
            oi[s] = fma(tr, wi[s], fma(ti, wr[s], c1.y));
        }
    }
    // deflections (u, v hold them until the end): the conjugate of f
#pragma unroll
    for (int s = 0; s < SW; ++s) {
        const double tr = fma(orr[s], zr, -(oi[s] * zi[s])), ti = fma(orr[s], zi[s], oi[s] * zr);
        u[2 * s] = er[s] + tr;
        v[2 * s] = -(ei[s] + ti);
        u[2 * s + 1] = er[s] - tr;
        v[2 * s + 1] = ti - ei[s];
    }
    const double xp = grid_pos(sa.x0, sa.d1, pi.a0 + col, sa.h), xm = grid_pos(sa.x0, sa.d1, pi.a0 + P - 1 - col, sa.h);
    double y[2 * SW];
#pragma unroll
    for (int s = 0; s < SW; ++s) {
        y[2 * s] = grid_pos(sa.y0, sa.d2, pi.b0 + P / 2 + row0 + s, sa.h);
        y[2 * s + 1] = grid_pos(sa.y0, sa.d2, pi.b0 + P / 2 - 1 - row0 - s, sa.h);
    }
    for (int k = 0; k < pi.ndir; ++k) {
        const double4 st = ns[dir[k]];
#pragma unroll
        for (int s = 0; s < 2 * SW; ++s)
            near_star<double>((s & 1 ? xm : xp) - li.cx, y[s] - li.cy, st, u[s], v[s]);
    }
    const Finish f(lc, g, pi.lin);
#pragma unroll
    for (int s = 0; s < 2 * SW; ++s) f(lc, s & 1 ? xm : xp, y[s], u[s], v[s]);
}

// pixel coordinates of one ray, ray by ray: the arithmetic of k_shoot in its
// order (leaf_alpha), the loops not unrolled, as few rays take it and its
// registers would cost the patches' occupancy
__device__ inline double2 exact_ray(const ShootArgs &sa, const LensConst &lc, const MapGeom &g, const LeafInfo &li,
                                    const double4 *__restrict__ ns, const double2 *__restrict__ dv, int64_t a, int64_t b)
{
    const double x = grid_pos(sa.x0, sa.d1, a, sa.h), y = grid_pos(sa.y0, sa.d2, b, sa.h);
    const double dx = x - li.cx, dy = y - li.cy;
    double ax = 0, ay = 0;
#pragma unroll 1
    for (int32_t s = 0; s < li.near_cnt; ++s) near_star<double>(dx, dy, ns[s], ax, ay);
    const double zr = dx * li.invL, zi = dy * li.invL;
    double sr = dv[sa.p - 1].x, si = dv[sa.p - 1].y;
#pragma unroll 1
    for (int l = sa.p - 2; l >= 0; --l) {
        const double2 c = dv[l];
        const double nr = sr * zr - si * zi + c.x;
        const double ni = sr * zi + si * zr + c.y;
        sr = nr;
        si = ni;
    }
    double w1, w2;
    double2 uv;
    finish_vertex(lc, g, x, y, ax + sr, ay - si, w1, w2, uv);
    return uv;
}

// The corners of the cells that the cell pass found too thin for patches
// (ThinList), ray by ray.  (A map lists tens of cells.)
__global__ __launch_bounds__(64) void k_shoot_thin(ShootArgs sa, LensConst lc, MapGeom g, LeafFinder find, int64_t cb0,
                                                   const LeafInfo *__restrict__ leaves,
                                                   const double4 *__restrict__ near,
                                                   const double2 *__restrict__ deriv, ThinList thin,
                                                   const double2 *__restrict__ verts)
{
    const int64_t n = 4 * (int64_t)min(*thin.count, THIN_CELLS);
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = thin.cell[t >> 2];
        const int64_t a = c % (sa.nr1 - 1) + (t & 1), b = cb0 + c / (sa.nr1 - 1) + ((t >> 1) & 1);
        const double x = grid_pos(sa.x0, sa.d1, a), y = grid_pos(sa.y0, sa.d2, b);
        const int64_t lf = find_leaf(x, y, find.nlevels, find.L0, find.L0_exp, find.child0, find.leaf, find.node_leaf);
        if (lf < 0) {
            thin.corner[t] = verts[(b - sa.vb0) * sa.nr1 + a];
            continue;
        }
        const LeafInfo li = leaves[lf];
        double ax, ay, w1, w2;
        leaf_alpha<double>(x - li.cx, y - li.cy, li, near + li.near_off, deriv + lf * sa.p, sa.p, ax, ay);
        finish_vertex(lc, g, x, y, ax, ay, w1, w2, thin.corner[t]);
    }
}

// patch column and row of ray s of a sweep
template <int P> __device__ inline int ray_col(int col, int s) { return s & 1 ? P - 1 - col : col; }
template <int P> __device__ inline int ray_row(int row0, int s)
{
    const int r = row0 + (s >> 1);
    return s & 1 ? P / 2 - 1 - r : P / 2 + r;
}

// the grid vertices of patch blockIdx.x (one wavefront)
template <int P>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_shoot_patch(ShootArgs sa, LensConst lc, MapGeom g, PatchArgs pa,
                                                    const PatchInfo *__restrict__ info,
                                                    const double2 *__restrict__ coef,
                                                    const LeafInfo *__restrict__ leaves,
                                                    const double4 *__restrict__ near,
                                                    const double2 *__restrict__ deriv, double2 *__restrict__ verts)
{
    using L = PatchLane<P>;
    const int64_t t = blockIdx.x;
    const PatchHead pi = info[t];
    const LeafInfo li = leaves[pi.lf];
    const double4 *ns = near + li.near_off;
    const int col = threadIdx.x & (P - 1), grp = threadIdx.x / P;
    const int na = pi.nanb & 0xffff, nb = pi.nanb >> 16;
    double2 *out = verts + (pi.b0 - sa.vb0) * sa.nr1 + pi.a0;
    if (pi.n == 0) {
        const double2 *dv = deriv + (int64_t)pi.lf * sa.p;
        for (int row = grp; row < nb; row += L::GROUPS)
            if (col < na) out[row * sa.nr1 + col] = exact_ray(sa, lc, g, li, ns, dv, pi.a0 + col, pi.b0 + row);
        return;
    }
#pragma unroll 1
    for (int sw = 0; sw < L::ROWS; sw += L::SW) {
        const int row0 = grp * L::ROWS + sw;
        double u[2 * L::SW], v[2 * L::SW];
        eval_sweep<P>(sa, lc, g, pa, pi, info[t].dir, li, ns, coef + t * PC_MAX, col, row0, u, v);
#pragma unroll
        for (int s = 0; s < 2 * L::SW; ++s) {
            const int c = ray_col<P>(col, s), rw = ray_row<P>(row0, s);
            if (c < na && rw < nb) out[rw * sa.nr1 + c] = make_double2(u[s], v[s]);
        }
    }
}

// Rays whose pixel coordinate lies close to a pixel's edge are shot again ray by
// ray, so that every ray counts in the pixel that k_shoot_irs counts it in: closer
// than EDGE, or, where pixels are small against the positions, than EDGE_UNITS
// units in the last place of what a position is the sum of (patch_edge), of which
// the series' and the rounding's error is a few.
constexpr double EDGE = 1e-6, EDGE_UNITS = 256.0;
constexpr double EDGE_MOST = 1.0 / 64.0;   // (beyond this every sixteenth ray or more would be shot again)

// inverse ray shooting of patch blockIdx.x: the patch's counts are summed in an
// LDS window of W x W pixels about its centre's image (a lane adds a run of
// rays in one pixel at once), the rest go to the map's counts.  (WIDE: the edges are
// wider than EDGE; as an argument for every map the width costs scalar registers that
// the loop is short of: 0.4 % of the 2.4e10-ray map.)
template <int P, int W, bool WIDE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_irs_patch(ShootArgs sa, LensConst lc, MapGeom g, PatchArgs pa,
                                                  const PatchInfo *__restrict__ info,
                                                  const double2 *__restrict__ coef,
                                                  const LeafInfo *__restrict__ leaves,
                                                  const double4 *__restrict__ near,
                                                  const double2 *__restrict__ deriv,
                                                  unsigned long long *__restrict__ counts)
{
    using L = PatchLane<P>;
    __shared__ unsigned win[W * W];
    const int64_t t = blockIdx.x;
    const PatchHead pi = info[t];
    const LeafInfo li = leaves[pi.lf];
    const double4 *ns = near + li.near_off;
    const double2 *dv = deriv + (int64_t)pi.lf * sa.p, *cf = coef + t * PC_MAX;
    const int col = threadIdx.x & (P - 1), grp = threadIdx.x / P;
    const int na = pi.nanb & 0xffff, nb = pi.nanb >> 16;
    if (pi.n == 0) {
        for (int row = grp; row - grp < nb; row += L::GROUPS) {
            const bool valid = col < na && row < nb;
            double2 uv = make_double2(0, 0);
            if (valid) uv = exact_ray(sa, lc, g, li, ns, dv, pi.a0 + col, pi.b0 + row);
            irs_count(valid, uv, g, counts);
        }
        return;
    }
    for (int k = threadIdx.x; k < W * W; k += 64) win[k] = 0;
    int i0 = 0, j0 = 0;
    {   // the window about the image of the patch's centre
        const double x = grid_pos(sa.x0, sa.d1, pi.a0, sa.h + 0.5 * (P - 1));
        const double y = grid_pos(sa.y0, sa.d2, pi.b0, sa.h + 0.5 * (P - 1));
        double u = cf[0].x, v = -cf[0].y;
        for (int k = 0; k < pi.ndir; ++k) near_star<double>(x - li.cx, y - li.cy, ns[info[t].dir[k]], u, v);
        Finish(lc, g, pi.lin)(lc, x, y, u, v);
        if (isfinite(u) && isfinite(v)) {
            i0 = (int)fmin(fmax(floor(u), -1e9), 1e9) - W / 2;
            j0 = (int)fmin(fmax(floor(v), -1e9), 1e9) - W / 2;
        }
    }
    __syncthreads();
    int ci[2] = {-1, -1}, cj[2] = {-1, -1};
    unsigned cn[2] = {0, 0};
    auto put = [&](int i, int j, unsigned k) {
        if (k == 0 || i < 0 || j < 0) return;
        const int di = i - i0, dj = j - j0;
        if ((unsigned)di < (unsigned)W && (unsigned)dj < (unsigned)W)
            __hip_atomic_fetch_add(win + dj * W + di, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            atomicAdd(counts + (int64_t)j * g.n1 + i, (unsigned long long)k);
    };
    const double n1 = g.n1, n2 = g.n2, most = WIDE ? pa.sure : 0.5 - EDGE;
    // (the rays to shoot again, four bits a sweep: shot inside the loop below, their
    // constants had a quarter of its instructions move spilled scalars, and the
    // 2.4e10-ray map took 69 ms instead of 58)
    unsigned long long redo = 0;
    static_assert(2 * L::ROWS <= 64 && L::SW <= 2, "a bit per ray of a lane");
#pragma unroll 1
    for (int sw = 0; sw < L::ROWS; sw += L::SW) {
        const int row0 = grp * L::ROWS + sw;
        double u[2 * L::SW], v[2 * L::SW];
        eval_sweep<P>(sa, lc, g, pa, pi, info[t].dir, li, ns, cf, col, row0, u, v);
        unsigned again = 0;
#pragma unroll
        for (int s = 0; s < 2 * L::SW; ++s) {
            const bool valid = ray_col<P>(col, s) < na && ray_row<P>(row0, s) < nb;
            const double fu = floor(u[s]), fv = floor(v[s]);
            // false for NaN
            const bool sure = fabs((u[s] - fu) - 0.5) <= most && fabs((v[s] - fv) - 0.5) <= most;
            if (valid && !sure) again |= 1u << s;
            const int iu = (int)fu, jv = (int)fv;   // (saturating: beyond the map stays beyond)
            const bool in = valid && sure && (unsigned)iu < (unsigned)g.n1 && (unsigned)jv < (unsigned)g.n2;
            const int i = in ? iu : -1, j = in ? jv : -1;
            if (i != ci[s & 1] || j != cj[s & 1]) {
                put(ci[s & 1], cj[s & 1], cn[s & 1]);
                ci[s & 1] = i;
                cj[s & 1] = j;
                cn[s & 1] = 0;
            }
            ++cn[s & 1];
        }
        redo |= (unsigned long long)again << (2 * sw);
    }
    while (__any(redo != 0)) {
        if (redo) {
            const int k = __ffsll(redo) - 1, sw = k / (2 * L::SW) * L::SW, s = k % (2 * L::SW);
            const int row0 = grp * L::ROWS + sw;
            const double2 uv = exact_ray(sa, lc, g, li, ns, dv, pi.a0 + ray_col<P>(col, s), pi.b0 + ray_row<P>(row0, s));
            const double fu = floor(uv.x), fv = floor(uv.y);
            if (fu >= 0.0 && fv >= 0.0 && fu < n1 && fv < n2) put((int)fu, (int)fv, 1);
            redo &= redo - 1;
        }
    }
    put(ci[0], cj[0], cn[0]);
    put(ci[1], cj[1], cn[1]);
    __syncthreads();
    for (int k = threadIdx.x; k < W * W; k += 64) {
        const unsigned c = win[k];
        if (c) atomicAdd(counts + (int64_t)(j0 + k / W) * g.n1 + i0 + k % W, (unsigned long long)c);
    }
}

// the edge's width in pixels: the rounding of a position in the map, the sum of the
// lens's linear terms (the smooth sheet's among them), a deflection of about that
// size and the map's corner
double patch_edge(const Region &R, const LensConst &lc, const MapGeom &g)
{
    const double x = std::max(std::fabs(R.x0), std::fabs(R.x0 + (double)R.nr1 * R.d1));
    const double y = std::max(std::fabs(R.y0), std::fabs(R.y0 + (double)R.nr2 * R.d2));
    const double size = (1.0 + std::fabs(lc.lam1) + std::fabs(lc.lam2) + 2.0 * lc.kappa_star) * (x + y) +
                        std::fabs(g.ylo1) + std::fabs(g.ylo2) + g.pix1 * g.n1 + g.pix2 * g.n2;
    return std::max(EDGE, EDGE_UNITS * 0x1p-53 * size / std::min(g.pix1, g.pix2));
}

PatchArgs patch_args(const Region &R, const LensConst &lc, const MapGeom &g, int P)
{
    PatchArgs pa;
    pa.hx = 0.5 * (P - 1) * R.d1;
    pa.hy = 0.5 * (P - 1) * R.d2;
    pa.r = std::sqrt(pa.hx * pa.hx + pa.hy * pa.hy);
    pa.ir = 1.0 / pa.r;
    pa.span = g.pix1 * g.n1 + g.pix2 * g.n2;
    pa.sure = 0.5 - patch_edge(R, lc, g);
    return pa;
}

}  // namespace

// Where the grid is shot by patches, and their side, by the rays per leaf (of the
// leaves the rays meet), which say how far the stars lie from a patch, and by how
// many rays there are to hide the coefficients' latency.  Measured on the 1e5-star
// map with more and fewer rays, ms ray by ray / 16 x 16 / 32 x 32 (in brackets:
// inverse ray shooting):
//   3300 rays a leaf, 2.9e7 rays   0.47 / 0.42 / 0.58   (0.95 / 0.61 / 1.20)
//   6700, 5.8e7                    0.81 / 0.67 / 0.75   (1.59 / 0.86 / 1.15)
//   10000, 8.7e7                   1.30 / 1.15 / 1.04   (2.23 / 1.29 / 1.38)
//   13300, 1.2e8                   1.74 / 1.49 / 1.05   (2.74 / 1.64 / 1.43)
//   101500, 2.4e8                  5.06 / 2.50 / 1.61   (4.19 / 2.30 / 1.37)
// and with 330 leaves met, so that the rays are few:
//   6000, 2.0e6                    0.045 / 0.047 / 0.098   (0.062 / 0.055 / 0.192)
//   8000, 2.6e6                    0.058 / 0.048 / 0.108   (0.083 / 0.065 / 0.209)
//   24000, 7.9e6                   0.142 / 0.085 / 0.092   (0.197 / 0.118 / 0.111)
//   32000, 1.0e7                   0.180 / 0.111 / 0.084   (0.238 / 0.149 / 0.120)
// and 32 x 32 / 64 x 64, whose coefficients cost a quarter and whose stars lie
// nearer in their units:
//   101500, 2.4e8                  1.62 / 1.76   (1.38 / 1.60)
//   330000, 4.2e7                  0.220 / 0.193   (0.226 / 0.220)
//   714000, 1.5e8                  0.803 / 0.701   (0.754 / 0.742)
//   5074000, 1.2e10                68.4 / 54.8   (48.0 / 35.6)
// Uneven fields are no worse off, though many leaves of a group hold less than a
// patch each: m leaves have at most rays / P^2 + 2 sqrt(m rays) / P + m patches, and
// in a group each of those replaces rays with full lists of near stars.  40 rays a
// pixel, ray by ray / by patches: a tight cluster 3.26 / 1.50, a fold caustic's
// field 4.79 / 1.66.
int patch_side(const Region &R, const Tree &T, int64_t rows)
{
    if (T.mixed || T.p < 1) return 0;
    // leaves that mostly hold more near stars than a patch takes would go ray by ray,
    // and there more slowly than by k_shoot.  Shooting ray by ray / by patches, ms, by
    // the mean number of a ray's near stars (8 rays a pixel; inverse ray shooting of
    // 60): 46: 2.30 / 0.42 (16.4 / 1.9); 53: 2.49 / 1.30 (16.9 / 3.2); 63: 2.52 /
    // 2.18 (17.7 / 11.1) and 4.09 / 3.89 (28.7 / 24.7); 76: 2.66 / 2.95 (18.8 / 19.0);
    // 78: 2.03 / 2.31 (13.9 / 16.7).
    if (T.near_total > PC_STARS * T.nactive_leaves) return 0;
    const double rays = (double)R.nr1 * (double)rows, per_leaf = rays / (double)std::max<int64_t>(T.nactive_leaves, 1);
    if (per_leaf >= LARGE_PATCH_RAYS_PER_LEAF && rays >= PATCH_MANY_RAYS) return 64;
    if (per_leaf >= PATCH_RAYS_PER_LEAF[rays >= PATCH_MANY_RAYS ? 1 : 0]) return 32;
    return per_leaf >= SMALL_PATCH_RAYS_PER_LEAF[rays >= SMALL_PATCH_MANY_RAYS ? 1 : 0] ? 16 : 0;
}

bool irs_by_patches(const Region &R, const LensConst &lc, const MapGeom &g) { return patch_edge(R, lc, g) <= EDGE_MOST; }

static void patch_coefs(mlm_lens *lens, const Tree &T, const LensConst &lc, const ShootArgs &sa, const PatchArgs &pa,
                        int side, int64_t npatch, hipStream_t st)
{
    Workspace &ws = lens->ws;
    if (!ws.binom.p) {
        double h[32 * 32] = {};
        for (int l = 0; l < 32; ++l) {
            h[l * 32] = 1.0;
            for (int j = 1; j <= l; ++j) h[l * 32 + j] = h[(l - 1) * 32 + j - 1] + (j < l ? h[(l - 1) * 32 + j] : 0.0);
        }
        MLM_HIP(hipMemcpy(ws.binom.reserve(sizeof h), h, sizeof h, hipMemcpyHostToDevice));
    }
    PatchInfo *info = static_cast<PatchInfo *>(ws.patch_info.reserve((size_t)npatch * sizeof(PatchInfo)));
    double2 *coef = static_cast<double2 *>(ws.patch_coef.reserve((size_t)npatch * PC_MAX * sizeof(double2)));
    hipLaunchKernelGGL(side == 64 ? k_patch_coef<64> : side == 32 ? k_patch_coef<32> : k_patch_coef<16>, dim3((unsigned)((npatch + 3) / 4)), dim3(64), 0, st, sa, lc, pa, npatch,
                       ws.tile_leaf.as<int32_t>(), ws.tile_off.as<int32_t>(), T.leaves, T.near, T.deriv,
                       ws.binom.as<double>(), info, coef);
}

void launch_shoot_patches(mlm_lens *lens, const Tree &T, const Region &R, const LensConst &lc, const MapGeom &g,
                          int side, int64_t npatch, int64_t vb0, double2 *verts, hipStream_t st)
{
    if (npatch <= 0) return;
    const ShootArgs sa{R.x0, R.y0, R.d1, R.d2, R.nr1, vb0, T.p, 0, 0.0};
    const PatchArgs pa = patch_args(R, lc, g, side);
    patch_coefs(lens, T, lc, sa, pa, side, npatch, st);
    hipLaunchKernelGGL(side == 64 ? k_shoot_patch<64> : side == 32 ? k_shoot_patch<32> : k_shoot_patch<16>, dim3((unsigned)npatch), dim3(64), 0, st, sa, lc, g, pa,
                       lens->ws.patch_info.as<PatchInfo>(), lens->ws.patch_coef.as<double2>(), T.leaves, T.near,
                       T.deriv, verts);
}

void launch_shoot_thin(const Tree &T, const Region &R, const LensConst &lc, const MapGeom &g, int64_t cb0,
                       int64_t vb0, const ThinList &thin, const double2 *verts, hipStream_t st)
{
    const ShootArgs sa{R.x0, R.y0, R.d1, R.d2, R.nr1, vb0, T.p, 0, 0.0};
    const LeafFinder find{T.nlevels, T.L0_exp, T.L0, T.child0, T.leaf, T.node_leaf};
    hipLaunchKernelGGL(k_shoot_thin, dim3(THIN_BLOCKS), dim3(64), 0, st, sa, lc, g, find, cb0, T.leaves, T.near, T.deriv,
                       thin, verts);
}

void launch_irs_patches(mlm_lens *lens, const Tree &T, const Region &R, const LensConst &lc, const MapGeom &g,
                        int side, int64_t npatch, int64_t cb0, unsigned long long *counts, hipStream_t st)
{
    if (npatch <= 0) return;
    const ShootArgs sa{R.x0, R.y0, R.d1, R.d2, R.nr1 - 1, cb0, T.p, 0, 0.5};
    const PatchArgs pa = patch_args(R, lc, g, side);
    patch_coefs(lens, T, lc, sa, pa, side, npatch, st);
    // the window: a patch's unlensed image is side d / pixel wide
    const bool wide = side * std::max(R.d1 / R.pix1, R.d2 / R.pix2) > 4.0;
    auto *k = side == 64   ? (wide ? k_irs_patch<64, 32, false> : k_irs_patch<64, 16, false>)
              : side == 32 ? (wide ? k_irs_patch<32, 32, false> : k_irs_patch<32, 16, false>)
                           : (wide ? k_irs_patch<16, 32, false> : k_irs_patch<16, 16, false>);
    if (pa.sure < 0.5 - EDGE)   // (a rare map: one window for all)
        k = side == 64 ? k_irs_patch<64, 32, true> : side == 32 ? k_irs_patch<32, 32, true> : k_irs_patch<16, 32, true>;
    hipLaunchKernelGGL(k, dim3((unsigned)npatch), dim3(64), 0, st, sa,
                       lc, g, pa, lens->ws.patch_info.as<PatchInfo>(), lens->ws.patch_coef.as<double2>(), T.leaves,
                       T.near, T.deriv, counts);
}

}  // namespace mlm
