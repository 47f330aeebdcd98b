// FMM passes (sec. 3.3, app. C.2): P2M at the leaves, M2M upward, then per
// level L2L from the parent + M2L from same-level interaction nodes + P2L from
// the stars of interaction squares that lie inside coarser leaves.
//
// Coefficients are normalised to each node's half-length (app. C.2), which
// makes every translation a fixed linear operator: M2M and L2L depend only on
// the child's quadrant, M2L only on the offset between the two squares (one
// of 40 in a 7x7 stencil).  The operators are tabulated once on the host in
// extended precision.
#include <algorithm>
#include <cmath>
#include <complex>
#include <vector>

#include "dev.hpp"

namespace mlm {

int64_t scan_total_public(mlm_lens *lens, const int32_t *in, int32_t *out, int64_t n, hipStream_t st);

namespace {

constexpr int BLK = 256;

// first node of each level (and one past the last's)
struct LevelRange {
    int32_t first[MAX_LEVELS];
};

inline unsigned nblocks(int64_t n, int b = BLK) { return (unsigned)((n + b - 1) / b); }

using cld = std::complex<long double>;

long double binom_ld(int n, int k)
{
    if (k < 0 || k > n) return 0.0L;
    long double r = 1.0L;
    for (int t = 1; t <= k; ++t) r = r * (long double)(n - k + t) / (long double)t;
    return r;
}

cld ipow(cld z, int n)
{
    cld r(1.0L, 0.0L);
    for (int t = 0; t < n; ++t) r *= z;
    return r;
}

// The tables of M2M and L2L are stored [quadrant][source coefficient k][target
// coefficient l], so that the lanes of a wavefront (one target coefficient
// each) read consecutive entries.

// M2M, child quadrant (qi, qj): z0 = child centre - parent centre in child
// half-lengths = (2qi-1) + i(2qj-1);  b_l = z0^l [-a_0/l + sum_{k=1}^{l} a_k z0^-k C(l-1,k-1)] / 2^l
void table_m2m(int p, std::vector<double2> &out)
{
    int P1 = p + 1;
    out.assign(4 * P1 * P1, make_double2(0, 0));
    for (int quad = 0; quad < 4; ++quad) {
        cld z0((long double)(2 * (quad & 1) - 1), (long double)(2 * (quad >> 1) - 1));
        for (int l = 0; l <= p; ++l)
            for (int k = 0; k <= p; ++k) {
                cld v(0.0L, 0.0L);
                if (l == 0) {
                    if (k == 0) v = 1.0L;
                } else if (k == 0) {
                    v = -ipow(z0, l) / (long double)l;
                } else if (k <= l) {
                    v = ipow(z0, l - k) * binom_ld(l - 1, k - 1);
                }
                v /= std::ldexp(1.0L, l);
                out[(quad * P1 + k) * P1 + l] = make_double2((double)v.real(), (double)v.imag());
            }
    }
}

// The M2L operator factorised: with z0 the source-to-target offset (in
// half-lengths) and b' = b_k (-z0)^-k,
//   c_l = z0^-l [ sum_{k>=1} C(l+k-1, k-1) b'_k - b_0 / l ],
// so every offset shares one real matrix P[l-1][k-1] = C(l+k-1, k-1) and
// differs only by the diagonal scalings S[off][k] = (-z0)^-k (sources) and
// T[off][l] = z0^-l (targets).  Tables of 32 entries per offset (p <= 31);
// P is 32 x 32, zero beyond p.
void table_m2l_factors(int p, std::vector<double2> &S, std::vector<double2> &T, std::vector<double> &P)
{
    S.assign(49 * 32, make_double2(0, 0));
    T.assign(49 * 32, make_double2(0, 0));
    P.assign(32 * 32, 0.0);
    for (int dy = -3; dy <= 3; ++dy)
        for (int dx = -3; dx <= 3; ++dx) {
            if (std::abs(dx) <= 1 && std::abs(dy) <= 1) continue;
            int off = (dx + 3) + 7 * (dy + 3);
            cld z0(2.0L * dx, 2.0L * dy);
            for (int k = 0; k <= p; ++k) {
                cld sv = ipow(-1.0L / z0, k), tv = ipow(1.0L / z0, k);
                S[off * 32 + k] = make_double2((double)sv.real(), (double)sv.imag());
                T[off * 32 + k] = make_double2((double)tv.real(), (double)tv.imag());
            }
        }
    for (int l = 1; l <= p; ++l)
        for (int k = 1; k <= p; ++k) P[(l - 1) * 32 + (k - 1)] = (double)binom_ld(l + k - 1, k - 1);
}

// L2L, child quadrant (qi, qj): delta = child centre - parent centre in parent
// half-lengths = ((2qi-1) + i(2qj-1)) / 2;  d_l = sum_{k>=l} c_k C(k,l) delta^(k-l) / 2^l
void table_l2l(int p, std::vector<double2> &out)
{
    int P1 = p + 1;
    out.assign(4 * P1 * P1, make_double2(0, 0));
    for (int quad = 0; quad < 4; ++quad) {
        cld delta(0.5L * (2 * (quad & 1) - 1), 0.5L * (2 * (quad >> 1) - 1));
        for (int l = 0; l <= p; ++l)
            for (int k = l; k <= p; ++k) {
                cld v = ipow(delta, k - l) * binom_ld(k, l) / std::ldexp(1.0L, l);
                out[(quad * P1 + k) * P1 + l] = make_double2((double)v.real(), (double)v.imag());
            }
    }
}

// a b with its roundings fixed (which of its products are contracted is
// otherwise the compiler's choice, line by line; the mixed mode rounds the
// coefficients to FP32, where one unit of difference here may show)
template <class R> __device__ inline R mul_re(R ax, R ay, R bx, R by) { return fma(ax, bx, -(ay * by)); }
template <class R> __device__ inline R mul_im(R ax, R ay, R bx, R by) { return fma(ay, bx, ax * by); }
template <class C2> __device__ inline void add_product(C2 &acc, const C2 &a, const C2 &b)
{
    acc.x += mul_re(a.x, a.y, b.x, b.y);
    acc.y += mul_im(a.x, a.y, b.x, b.y);
}

// Upward pass of one level: P2M at a leaf, M2M from the four children elsewhere;
// half a wavefront per node, lane k its coefficient k.  A launch starts with cold
// caches, and a load takes about 1 us then: the operator table (28 KB at order 20)
// goes to LDS in one round of loads while the nodes' own data are fetched, all of
// a node's data at once, and the lanes load a leaf's stars, or the children's
// coefficients, side by side and hand them round (a level of
// the 1000-star tree: 7.2 us, and 8.2 with each lane loading every star and entry
// itself; of the 1e5-star tree: 10.7 on average, and 15.9).  Large levels
// are walked by as many workgroups as fit the chip.  R is the arithmetic type of
// the coefficients; star offsets from the node centre are always formed in FP64.
constexpr int UP_BLOCKS = 1024;

struct UpArgs {
    int p;
    double L0;
    const uint64_t *code;
    const int32_t *leaf, *slo, *shi, *child0;
    const double *sx, *sy, *sm;
};

// z^k for k < 32 by binary powering, without branches (a lane per k)
__device__ inline double2 cpow32(double2 z, int k)
{
    double2 r = make_double2(1.0, 0.0);
#pragma unroll
    for (int b = 0; b < 5; ++b) {
        const double tx = mul_re(r.x, r.y, z.x, z.y), ty = mul_im(r.x, r.y, z.x, z.y);
        r.x = (k >> b) & 1 ? tx : r.x;
        r.y = (k >> b) & 1 ? ty : r.y;
        const double zx = fma(z.x, z.x, -(z.y * z.y)), zy = z.x * z.y;
        z = make_double2(zx, zy + zy);
    }
    return r;
}

// a leaf's coefficient k: a_0 = sum m_i, a_k = -(1/k) sum m_i zeta_i^k
template <class R>
__device__ inline void p2m(const UpArgs &u, uint64_t code, int32_t s0, int32_t s1, int k, int lev, R &ax, R &ay)
{
    using C2 = typename Cx<R>::c2;
    double cx, cy, L, invL;
    node_geom(code, lev, u.L0, cx, cy, L, invL);
    ax = ay = 0;
    for (int32_t base = s0; base < s1; base += 32) {
        const int32_t s = min(base + k, s1 - 1);
        const R zx = (R)((u.sx[s] - cx) * invL), zy = (R)((u.sy[s] - cy) * invL), ms = (R)u.sm[s];
        const int n = min(32, s1 - base);
        for (int j = 0; j < n; j += 2) {   // two stars' powers side by side
            const int j1 = min(j + 1, n - 1);
            const R m0 = __shfl(ms, j, 32), m1 = __shfl(ms, j1, 32);
            const C2 z0 = Cx<R>::make(__shfl(zx, j, 32), __shfl(zy, j, 32));
            const C2 z1 = Cx<R>::make(__shfl(zx, j1, 32), __shfl(zy, j1, 32));
            const C2 w0 = cpow32(z0, k), w1 = cpow32(z1, k);
            ax = k ? fma(-m0, w0.x, ax) : ax + m0;
            ay = k ? fma(-m0, w0.y, ay) : ay;
            if (j + 1 < n) {
                ax = k ? fma(-m1, w1.x, ax) : ax + m1;
                ay = k ? fma(-m1, w1.y, ay) : ay;
            }
        }
    }
    if (k > 0) {
        const R ik = (R)1 / (R)k;
        ax *= ik;
        ay *= ik;
    }
}

// (the first workgroup also clears the local expansions of the first `none` nodes)
template <class R>
__global__ __launch_bounds__(BLK) void k_upward(UpArgs u, int64_t lo, int64_t end, int lev,
                                                const typename Cx<R>::c2 *__restrict__ m2m, typename Cx<R>::c2 *mult,
                                                typename Cx<R>::c2 *__restrict__ local, int64_t none)
{
    extern __shared__ double2 up_lds[];
    using C2 = typename Cx<R>::c2;
    constexpr int PER = BLK / 32;
    const int P1 = u.p + 1, n = 4 * P1, h = threadIdx.x >> 5, k = threadIdx.x & 31;
    C2 *op = reinterpret_cast<C2 *>(up_lds), *a = op + n * P1 + h * n;
    for (int e = threadIdx.x; e < n * P1; e += BLK) op[e] = m2m[e];
    if (blockIdx.x == 0)
        for (int64_t e = threadIdx.x; e < none * P1; e += BLK) local[e] = Cx<R>::make(0, 0);
    bool first = true;
    for (int64_t q0 = lo + (int64_t)blockIdx.x * PER; q0 < end; q0 += (int64_t)gridDim.x * PER) {
        const bool valid = q0 + h < end;
        const int64_t q = valid ? q0 + h : lo;   // (the first node stands in for one beyond the end)
        const int32_t leaf = u.leaf[q], c0 = u.child0[q], s0 = u.slo[q], s1 = u.shi[q];
        const uint64_t code = u.code[q];
        const bool inner = leaf == 0;
        R ax = 0, ay = 0;
        if (inner) {
            const C2 *c = mult + (int64_t)c0 * P1;
#pragma unroll
            for (int e = 0; e < (MAX_ORDER + 1) / 8; ++e)
                if (e * 32 + k < n) a[e * 32 + k] = c[e * 32 + k];
        } else {
            p2m<R>(u, code, s0, s1, k, lev, ax, ay);
        }
        if (first) __syncthreads();   // (the table; the trips are the workgroup's)
        first = false;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (k <= u.p && inner) {
            // (the table has zeros above the diagonal: every lane runs all the terms)
#pragma unroll 4
            for (int e = 0; e < n; ++e) {
                const C2 o = op[e * P1 + k], v = a[e];
                ax += mul_re(o.x, o.y, v.x, v.y);
                ay += mul_im(o.x, o.y, v.x, v.y);
            }
        }
        if (k <= u.p && valid) mult[q * P1 + k] = Cx<R>::make(ax, ay);
    }
}

// Matrix-core product of the factorised M2L: Y (32 x 64) = P (32 x 32) B
// (32 x 64), as 16 x 16 x 4 FP64 tiles; lane l holds A(l % 16, l / 16) and
// B(l / 16, l % 16); its four results are D(4 i + l / 16, l % 16), i < 4.
// (The coefficient passes run in FP64 in both precision modes.)
typedef double f64x4 __attribute__((ext_vector_type(4)));
__device__ inline f64x4 mma16(double a, double b, f64x4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
template <class R> struct V4T;
template <> struct V4T<double> {
    using t = f64x4;
    __device__ static int row(int i, int g4) { return 4 * i + g4; }
};

// The sources of a node go through the matrix cores in groups of GS: a
// group's scaled coefficients fill a 32 x 2 GS block of LDS (row stride BRS,
// one more than its columns so the rows of a column fall in other banks).  The
// pass is a chain of latencies, so it is the wavefronts a CU holds that count:
// five per SIMD at 5 KB and 96 registers each (groups of 16, 9 KB and 116
// registers: 330 us for 78k nodes, here 300; all 27 at once, 17 KB: 370).
constexpr int GS = 8;
constexpr int BRS = 2 * GS + 1;
template <class R> struct DownLds {
    R B[32 * BRS];         // a group's scaled source coefficients: row k - 1, columns (2 s, 2 s + 1) =
                           // (re, im) of source s of the group; then, in place, P B
    typename Cx<R>::c2 b0[32];
    int off[32], src[32];
};

__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// coefficient l of node q with its parent's part (levels 0 and 1 have no far field)
template <class R>
__device__ inline typename Cx<R>::c2 add_l2l(typename Cx<R>::c2 acc, int64_t q, int l, int lev, int p,
                                             const uint64_t *__restrict__ code, const int32_t *__restrict__ parent,
                                             const typename Cx<R>::c2 *__restrict__ l2l,
                                             const typename Cx<R>::c2 *local)
{
    using C2 = typename Cx<R>::c2;
    if (lev < 3) return acc;
    const uint64_t c = code[q];
    const int quad = (int)((c & 1ull) | (((c >> 1) & 1ull) << 1)), P1 = p + 1;
    const C2 *op = l2l + quad * P1 * P1 + l;
    const C2 *cp = local + (int64_t)parent[q] * P1;
    // (the table is 0 for k < l)
    // (loads in rounds of ten, beyond p on the last index, so that none is left
    // over for a loop of single ones)
    for (int k0 = 1; k0 <= p; k0 += 10) {
        C2 o[10], v[10];
#pragma unroll
        for (int j = 0; j < 10; ++j) {
            o[j] = op[min(k0 + j, p) * P1];
            v[j] = cp[min(k0 + j, p)];
        }
#pragma unroll
        for (int j = 0; j < 10; ++j)
            if (k0 + j <= p) add_product(acc, o[j], v[j]);
    }
    return acc;
}

// What the far squares give the listed nodes of the levels >= 2, those whose
// square meets the rays' rectangle (a star disc mostly reaches far beyond it: on
// the 1e5-star map one node in seven does), one wavefront per node: M2L from the
// same-level interaction nodes through the factorised operator (the shared real
// matrix on the matrix cores, the scalings on the vector units), P2L from the
// stars of interaction squares inside coarser leaves (lane l: coefficient l).
// No level needs another's result here, so all levels go in one launch (with the
// parents' part in it, level by level, the 1000-star tree took 52 us of kernels;
// this and k_l2l take 28, and of the 1e5-star tree 415 where that took 500)
// (listed.first[lev] listed nodes come before level lev's); k_l2l adds the
// parents' part.  p2l: the P2L part per listed node, kept apart since a
// coefficient's sum runs M2L, L2L, P2L.  Without p2l (inside a scratch arena) a
// launch takes one level, and adds the parents' part itself.
template <class R>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(5))) void k_m2l(LevelRange lo, LevelRange listed, int nlevels, int k0, int count, int p, double L0,
                                            const int32_t *__restrict__ act, const uint64_t *__restrict__ code,
                                            const IEntry *__restrict__ ilist, const double *__restrict__ sx,
                                            const double *__restrict__ sy, const double *__restrict__ sm,
                                            const typename Cx<R>::c2 *__restrict__ Sf,
                                            const typename Cx<R>::c2 *__restrict__ Tf, const R *__restrict__ Pm,
                                            const int32_t *__restrict__ parent,
                                            const typename Cx<R>::c2 *__restrict__ l2l,
                                            const typename Cx<R>::c2 *__restrict__ mult,
                                            typename Cx<R>::c2 *local, typename Cx<R>::c2 *__restrict__ p2l_out)
{
    using C2 = typename Cx<R>::c2;
    using V4 = typename V4T<R>::t;
    __shared__ DownLds<R> L;   // one wavefront per workgroup and node
    const int lane = threadIdx.x;
    const int P1 = p + 1;
    // consecutive nodes, whose sources are mostly the same, to one XCD (their
    // workgroups are dealt out to the eight in turn): one L2 then holds them
    const int per = (int)(gridDim.x / NXCD), at = (int)(blockIdx.x % NXCD) * per + (int)(blockIdx.x / NXCD);
    if (at >= count) return;
    const int k = k0 + at;
    int lev = 2;
    while (lev + 1 < nlevels && k >= listed.first[lev + 1]) ++lev;
    const int64_t q = act[lo.first[lev] + k - listed.first[lev]];
    const int lgr = p <= 16 ? 4 : 5;
    const int mt_n = (p + 15) / 16, kt_n = (p + 3) / 4;
    const int r = lane & 15, g4 = lane >> 4;
    // this lane's operands of P for every product below, loaded once: P is the
    // same for every node and group, and reading it inside the product loop
    // made each matrix-core step wait for a global load
    constexpr int KTMAX = (MAX_ORDER + 4) / 4;
    R pa[KTMAX], pb[KTMAX];
#pragma unroll
    for (int ks = 0; ks < KTMAX; ++ks) {
        pa[ks] = ks < kt_n ? Pm[r * 32 + ks * 4 + g4] : (R)0;
        pb[ks] = ks < kt_n && mt_n > 1 ? Pm[(16 + r) * 32 + ks * 4 + g4] : (R)0;
    }
    const uint64_t c = code[q];
    // the node's M2L sources into slots 0 .. ns-1 (lanes 0..26 hold the entries)
    const IEntry *list = ilist + q * NLIST;
    IEntry en{-2, 0, 0, 0};
    if (lane < NLIST) en = list[lane];
    const uint64_t mask = __ballot(lane < NLIST && en.src >= 0);
    const int ns = __popcll(mask);
    const int slot = __popcll(mask & ((1ull << lane) - 1ull));
    if (lane < NLIST && en.src >= 0) {
        L.off[slot] = en.off;
        L.src[slot] = en.src;
        L.b0[slot] = mult[(int64_t)en.src * P1];
    }
    wave_sync();
    // M2L, coefficient l = lane: sum over the sources of z0^-l (y_l - b_0 / l),
    // y = P B with B the coefficients b_k (-z0)^-k (rows k - 1 = 0 .. p - 1;
    // only the rows the products read: 16 for p <= 16, else 32)
    const int l = lane;
    const R il = l > 0 ? (R)1 / (R)l : (R)0;
    C2 acc = Cx<R>::make(0, 0);
    for (int g0 = 0; g0 < ns; g0 += GS) {
        const int gn = min(GS, ns - g0);
        const int ncol = ((2 * gn + 15) / 16) * 16;
        // a lane keeps its row k1 = k - 1 and walks the sources (loaded on any index
        // where there is nothing to load, so that several rounds' loads are in
        // flight)
        const int k1 = lane & ((1 << lgr) - 1), kc = min(k1, p - 1) + 1, step = 64 >> lgr;
        R *to = L.B + k1 * BRS;
#pragma unroll 4
        for (int s2 = lane >> lgr; s2 < ncol / 2; s2 += step) {
            const int sc = g0 + min(s2, gn - 1);
            const C2 b = mult[(int64_t)L.src[sc] * P1 + kc], f = Sf[L.off[sc] * 32 + kc];
            const bool in = s2 < gn && k1 < p;
            to[2 * s2] = in ? mul_re(b.x, b.y, f.x, f.y) : (R)0;
            to[2 * s2 + 1] = in ? mul_im(b.x, b.y, f.x, f.y) : (R)0;
        }
        wave_sync();
        // Y = P B on the matrix cores, in place: a 16-column block of B is read
        // whole (both 16-row tiles of P) before Y's block overwrites it
        for (int nt = 0; nt < ncol / 16; ++nt) {
            V4 acc0 = {}, acc1 = {};
#pragma unroll
            for (int ks = 0; ks < KTMAX; ++ks) {
                if (ks < kt_n) {
                    const R b = L.B[(ks * 4 + g4) * BRS + nt * 16 + r];
                    acc0 = mma16(pa[ks], b, acc0);
                    if (mt_n > 1) acc1 = mma16(pb[ks], b, acc1);
                }
            }
            wave_sync();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                L.B[V4T<R>::row(i, g4) * BRS + nt * 16 + r] = acc0[i];
                if (mt_n > 1) L.B[(16 + V4T<R>::row(i, g4)) * BRS + nt * 16 + r] = acc1[i];
            }
        }
        wave_sync();
        if (l >= 1 && l <= p)
#pragma unroll 8
            for (int s2 = 0; s2 < gn; ++s2) {
                const C2 t = Tf[L.off[g0 + s2] * 32 + l];
                const R yr = L.B[(l - 1) * BRS + 2 * s2] - L.b0[g0 + s2].x * il;
                const R yi = L.B[(l - 1) * BRS + 2 * s2 + 1] - L.b0[g0 + s2].y * il;
                add_product(acc, t, Cx<R>::make(yr, yi));
            }
        wave_sync();   // the next group overwrites B
    }
    // P2L from the stars of interaction squares that are not nodes (parts of
    // coarser leaves): c_l += -m / (l zeta^l).  Lanes take the stars, the
    // powers zeta^-l follow by one product per order, and each order's sum over
    // the wavefront (lanes 32 apart first, then 16, ...) lands in lane l.  Eight
    // orders are summed together: of a pair of lanes each keeps half of them.
    double cx, cy, Lh, invL;
    node_geom(c, lev, L0, cx, cy, Lh, invL);
    C2 p2l = Cx<R>::make(0, 0);
    const int cnt = (lane < NLIST && en.src == -1) ? en.shi - en.slo : 0;
    int total;
    const int excl = wave_excl_scan(cnt, lane, total);
    for (int base = 0; base < total; base += 64) {
        const int item = base + lane;
        const int E = wave_find(excl, item);
        const int s = __shfl(en.slo, E, 64) + item - __shfl(excl, E, 64);
        C2 w = Cx<R>::make(0, 0);
        R mq = 0;
        if (item < total) {
            w = cinv(Cx<R>::make((R)((sx[s] - cx) * invL), (R)((sy[s] - cy) * invL)));
            mq = -(R)sm[s];
        }
        C2 t = cscale(w, mq);   // -m zeta^-1
        for (int o0 = 1; o0 <= p; o0 += 8) {
            R vx[8], vy[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                vx[i] = t.x;
                vy[i] = t.y;
                t = Cx<R>::make(mul_re(w.x, w.y, t.x, t.y), mul_im(w.x, w.y, t.x, t.y));
            }
#pragma unroll
            for (int h = 4; h >= 1; h >>= 1) {
                const bool up = lane & (8 * h);   // lane distances 32, 16, 8
#pragma unroll
                for (int i = 0; i < h; ++i) {
                    const R gx = up ? vx[i] : vx[i + h], gy = up ? vy[i] : vy[i + h];
                    vx[i] = (up ? vx[i + h] : vx[i]) + __shfl_xor(gx, 8 * h, 64);
                    vy[i] = (up ? vy[i + h] : vy[i]) + __shfl_xor(gy, 8 * h, 64);
                }
            }
#pragma unroll
            for (int o = 4; o >= 1; o >>= 1) {
                vx[0] += __shfl_xor(vx[0], o, 64);
                vy[0] += __shfl_xor(vy[0], o, 64);
            }
            // order o0 + i is with the lanes whose bits 5, 4, 3 are i's
            const int i = lane - o0, from = ((i & 4) << 3) | ((i & 2) << 3) | ((i & 1) << 3);
            const R sxk = __shfl(vx[0], from, 64), syk = __shfl(vy[0], from, 64);
            if (i >= 0 && i < 8) {
                p2l.x += sxk;
                p2l.y += syk;
            }
        }
    }
    // coefficient l = lane (c_0 only shifts the potential)
    if (l > p) return;
    if (l == 0) {
        acc = p2l = Cx<R>::make(0, 0);
    } else if (!p2l_out || lev == 2) {   // (level 2 has no parents' part)
        acc = add_l2l<R>(acc, q, l, lev, p, code, parent, l2l, local);
        acc.x += p2l.x * il;
        acc.y += p2l.y * il;
    }
    local[q * P1 + l] = acc;
    if (p2l_out && lev > 2) p2l_out[(int64_t)k * P1 + l] = p2l;
}

// The parents' part for n listed nodes of one level, after their own M2L, and
// the P2L part after it: half a wavefront per node, lane l its coefficient l.
template <class R>
__global__ __launch_bounds__(BLK) void k_l2l(int64_t lo, int n, int lev, int p, const int32_t *__restrict__ act,
                                             const uint64_t *__restrict__ code, const int32_t *__restrict__ parent,
                                             const typename Cx<R>::c2 *__restrict__ l2l,
                                             const typename Cx<R>::c2 *__restrict__ p2l,
                                             typename Cx<R>::c2 *local)
{
    using C2 = typename Cx<R>::c2;
    const int P1 = p + 1;
    const int k = (int)(((int64_t)blockIdx.x * BLK + threadIdx.x) >> 5), l = threadIdx.x & 31;
    if (k >= n || l == 0 || l > p) return;
    const int64_t q = act[lo + k];
    C2 acc = add_l2l<R>(local[q * P1 + l], q, l, lev, p, code, parent, l2l, local);
    const C2 d = p2l[(int64_t)k * P1 + l];
    const R il = (R)1 / (R)l;
    acc.x += d.x * il;
    acc.y += d.y * il;
    local[q * P1 + l] = acc;
}

// per-leaf data for the ray kernels, of the leaves that meet the rays'
// rectangle: geometry, the far field at the centre (FP64), derivative of the
// Taylor series (rounded to R) and the stars of the leaf's 3x3 block relative
// to its centre (FP64 in both modes: a ray's offset from a star is formed from
// them).  One wavefront per leaf: lane l its coefficient l, lanes 0 .. 8 the
// star ranges of the block's squares (from the colleague references), then
// every lane copies stars.  (One thread per leaf, searching the whole key
// array for each square, spent 83 us on the latency of its loads for the
// 1e5-star map's 59k leaves, and 45 us for 1000 stars.)
template <class R>
__global__ __launch_bounds__(BLK) void k_leaf_tables(int64_t nleaves, int p, double L0, RayBox box,
                              const int32_t *__restrict__ leaf_node,
                              const uint64_t *__restrict__ code, const int32_t *__restrict__ level,
                              const int32_t *__restrict__ near_offs, const int32_t *__restrict__ coll,
                              const int32_t *__restrict__ slo, const int32_t *__restrict__ shi,
                              const uint64_t *__restrict__ keys, const double *__restrict__ sx,
                              const double *__restrict__ sy, const double *__restrict__ sm,
                              const double2 *__restrict__ local, LeafInfo *__restrict__ info,
                              typename Cx<R>::c2 *__restrict__ deriv, double4 *__restrict__ near)
{
    const int64_t lf = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int lane = threadIdx.x & 63;
    if (lf >= nleaves) return;
    const int32_t q = leaf_node[lf];
    const int lev = level[q];
    const uint64_t c = code[q];
    if (!in_box(c, lev, L0, box)) return;
    double cx, cy, L, invL;
    node_geom(c, lev, L0, cx, cy, L, invL);
    // star ranges of the 3x3 block
    int32_t s0 = 0, s1 = 0;
    if (lane < 9) {
        const int64_t a = (int64_t)compact_bits(c) + lane % 3 - 1, b = (int64_t)compact_bits(c >> 1) + lane / 3 - 1;
        const int32_t ref = coll[(int64_t)q * 9 + lane];   // -1 outside the root
        if (ref != -1) ref_stars(ref, morton2((uint32_t)a, (uint32_t)b), 2 * (KEY_BITS - lev), slo, shi, keys, s0, s1);
    }
    int total;
    const int excl = wave_excl_scan(s1 - s0, lane, total);
    const int32_t off = near_offs[lf];
    if (lane == 0) {
        LeafInfo li;
        li.cx = cx;
        li.cy = cy;
        li.L = L;
        li.invL = invL;
        li.near_off = off;
        li.near_cnt = total;
        li.a_lo = li.na = li.b_lo = li.nb = li.ntx = li.pad = 0;
        // d psi / dz = (1/L) sum_{l>=1} l c_l zeta^(l-1); its value at the centre
        // (l = 1) is the whole field of the far stars, kept in FP64
        const double2 d0 = cscale(local[(int64_t)q * (p + 1) + 1], invL);
        li.f0x = d0.x;
        li.f0y = d0.y;
        info[lf] = li;
    }
    if (lane < p) {
        const double2 d = cscale(local[(int64_t)q * (p + 1) + lane + 1], (double)(lane + 1) * invL);
        deriv[lf * p + lane] = Cx<R>::make((R)d.x, (R)d.y);
    }
    for (int base = 0; base < total; base += 64) {
        const int item = base + lane;
        const int e = wave_find(excl, item);
        const int32_t s = __shfl(s0, e, 64) + item - __shfl(excl, e, 64);
        if (item < total) near[off + item] = make_double4(sx[s] - cx, sy[s] - cy, sm[s], 0.0);
    }
}

__global__ void k_leaf_block(int64_t nleaves, double L0, RayBox box, const int32_t *__restrict__ leaf_node,
                             const uint64_t *__restrict__ code, const int32_t *__restrict__ level,
                             const int32_t *__restrict__ block, int32_t *__restrict__ cnt)
{
    int64_t lf = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (lf >= nleaves) return;
    const int32_t q = leaf_node[lf];
    cnt[lf] = in_box(code[q], level[q], L0, box) ? block[q] : 0;
}

}  // namespace

namespace {

template <class R>
void upload_ops(DevBuf &buf, const std::vector<double2> &h)
{
    using C2 = typename Cx<R>::c2;
    std::vector<C2> c(h.size());
    for (size_t k = 0; k < h.size(); ++k) c[k] = Cx<R>::make((R)h[k].x, (R)h[k].y);
    void *d = buf.reserve(c.size() * sizeof(C2));
    MLM_HIP(hipMemcpy(d, c.data(), c.size() * sizeof(C2), hipMemcpyHostToDevice));
}

template <class R>
void run_fmm_t(mlm_lens *lens, Tree &T, int p, bool all, hipStream_t st, typename Cx<R>::c2 *&mult,
               typename Cx<R>::c2 *&local)
{
    using C2 = typename Cx<R>::c2;
    Workspace &ws = lens->ws;
    const int P1 = p + 1;
    const int key = p;
    if (ws.ops_p != key) {
        std::vector<double2> h, S, T;
        std::vector<double> Pm;
        table_m2m(p, h);
        upload_ops<R>(ws.ops_m2m, h);
        table_l2l(p, h);
        upload_ops<R>(ws.ops_l2l, h);
        table_m2l_factors(p, S, T, Pm);
        // one buffer: S (49 x 32 complex), T (49 x 32 complex), P (32 x 32 real)
        std::vector<C2> st(2 * 49 * 32);
        for (size_t k = 0; k < S.size(); ++k) {
            st[k] = Cx<R>::make((R)S[k].x, (R)S[k].y);
            st[S.size() + k] = Cx<R>::make((R)T[k].x, (R)T[k].y);
        }
        std::vector<R> pr(Pm.size());
        for (size_t k = 0; k < Pm.size(); ++k) pr[k] = (R)Pm[k];
        char *d = static_cast<char *>(ws.ops_m2l.reserve(st.size() * sizeof(C2) + pr.size() * sizeof(R)));
        MLM_HIP(hipMemcpy(d, st.data(), st.size() * sizeof(C2), hipMemcpyHostToDevice));
        MLM_HIP(hipMemcpy(d + st.size() * sizeof(C2), pr.data(), pr.size() * sizeof(R), hipMemcpyHostToDevice));
        ws.ops_p = key;
    }
    const C2 *Sf = ws.ops_m2l.as<C2>(), *Tf = Sf + 49 * 32;
    const R *Pm = reinterpret_cast<const R *>(Sf + 2 * 49 * 32);
    mult = static_cast<C2 *>(ws.mult.reserve((size_t)T.nnodes * P1 * sizeof(C2)));
    local = static_cast<C2 *>(ws.local.reserve((size_t)T.nnodes * P1 * sizeof(C2)));
    LevelRange lo{}, listed{};
    for (int lev = 0; lev < T.nlevels; ++lev) {
        lo.first[lev] = (int32_t)T.level_lo[lev];
        lo.first[lev + 1] = (int32_t)T.level_hi[lev];
        listed.first[lev + 1] = listed.first[lev] + (lev >= 2 ? T.nactive[lev] : 0);
    }
    // upward, to level 2, the coarsest that a list holds (all: to the root);
    // levels 0, 1 have no far field
    constexpr int per = BLK / 32;
    constexpr size_t most = (4 * (MAX_ORDER + 1) * (MAX_ORDER + 1) + per * 4 * (MAX_ORDER + 1)) * sizeof(C2);
    allow_lds(reinterpret_cast<const void *>(&k_upward<R>), most);
    const UpArgs u{p, T.L0, T.code, T.leaf, T.slo, T.shi, T.child0, T.x, T.y, T.m};
    const int64_t none = T.nlevels > 2 ? T.level_lo[2] : T.nnodes;
    const int top = all ? 0 : std::min(2, T.nlevels - 1);
    for (int lev = T.nlevels - 1; lev >= top; --lev)
        hipLaunchKernelGGL(k_upward<R>,
                           dim3(std::min(nblocks(T.level_hi[lev] - T.level_lo[lev], per), (unsigned)UP_BLOCKS)),
                           dim3(BLK), (4 * P1 + 4 * per) * P1 * sizeof(C2), st, u, T.level_lo[lev], T.level_hi[lev], lev,
                           ws.ops_m2m.as<C2>(), mult, local, lev == top ? none : 0);
    // downward
    const int32_t n = listed.first[T.nlevels];
    if (n == 0) return;
    C2 *p2l = thread_arena() ? nullptr : static_cast<C2 *>(ws.p2l.reserve((size_t)n * P1 * sizeof(C2)));
    const auto m2l = [&](int k0, int32_t cnt) {
        hipLaunchKernelGGL(k_m2l<R>, dim3(nblocks(cnt, NXCD) * NXCD), dim3(64), 0, st, lo, listed, T.nlevels, k0, cnt, p, T.L0, T.active,
                           T.code, T.ilist, T.x, T.y, T.m, Sf, Tf, Pm, T.parent, ws.ops_l2l.as<C2>(), mult, local, p2l);
    };
    if (p2l) m2l(0, n);
    for (int lev = p2l ? 3 : 2; lev < T.nlevels && T.nactive[lev] > 0; ++lev) {   // (where a level has none, nor has any finer)
        if (p2l)
            hipLaunchKernelGGL(k_l2l<R>, dim3(nblocks((int64_t)T.nactive[lev] * 32)), dim3(BLK), 0, st, T.level_lo[lev],
                               T.nactive[lev], lev, p, T.active, T.code, T.parent, ws.ops_l2l.as<C2>(),
                               p2l + (size_t)listed.first[lev] * P1, local);
        else
            m2l(listed.first[lev], T.nactive[lev]);
    }
}

}  // namespace

void run_fmm(mlm_lens *lens, Tree &T, int p, hipStream_t st, bool all)
{
    if (p < 1 || p > MAX_ORDER) fail(MLM_EINVAL, "expansion order %d outside [1, %d]", p, MAX_ORDER);
    T.p = p;
    // FP64 in both modes: the low-order Taylor coefficients carry the field of
    // the whole star disc (about kappa_* |z|), far above what FP32 translation
    // chains could hold to a fraction of a pixel
    run_fmm_t<double>(lens, T, p, all, st, T.mult, T.local);
}

void build_leaf_tables(mlm_lens *lens, Tree &T, hipStream_t st)
{
    Workspace &ws = lens->ws;
    int64_t nl = T.nleaves;
    if (!T.near_numbered) {
        int32_t *cnt = static_cast<int32_t *>(ws.flags.reserve(nl * 4));
        T.near_offs = static_cast<int32_t *>(ws.near_offs.reserve(nl * 4));
        hipLaunchKernelGGL(k_leaf_block, dim3(nblocks(nl)), dim3(BLK), 0, st, nl, T.L0, ray_box(T), T.leaf_node,
                           T.code, T.level, T.block, cnt);
        T.near_total = scan_total_public(lens, cnt, T.near_offs, nl, st);
    }
    T.leaves = static_cast<LeafInfo *>(ws.leaves.reserve(nl * sizeof(LeafInfo)));
    const size_t nn = (size_t)(T.near_total > 0 ? T.near_total : 1);
    T.near = static_cast<double4 *>(ws.near.reserve(nn * sizeof(double4)));
    if (T.mixed) {
        T.deriv_f = static_cast<float2 *>(ws.deriv.reserve((size_t)nl * T.p * sizeof(float2)));
        hipLaunchKernelGGL(k_leaf_tables<float>, dim3(nblocks(nl * 64)), dim3(BLK), 0, st, nl, T.p, T.L0, ray_box(T),
                           T.leaf_node, T.code, T.level, T.near_offs, T.coll, T.slo, T.shi, T.keys, T.x, T.y, T.m, T.local,
                           T.leaves, T.deriv_f, T.near);
    } else {
        T.deriv = static_cast<double2 *>(ws.deriv.reserve((size_t)nl * T.p * sizeof(double2)));
        hipLaunchKernelGGL(k_leaf_tables<double>, dim3(nblocks(nl * 64)), dim3(BLK), 0, st, nl, T.p, T.L0, ray_box(T),
                           T.leaf_node, T.code, T.level, T.near_offs, T.coll, T.slo, T.shi, T.keys, T.x, T.y, T.m, T.local,
                           T.leaves, T.deriv, T.near);
    }
}

}  // namespace mlm
