// Products of a map (sec. 4.1, 5): light curves of a point source moving
// along a straight track, and the distribution of log10 magnification.  Both
// read the map once and are bound by memory traffic.
#include "dev.hpp"

namespace mlm {

namespace {

constexpr int HIST_BLK = 1024;
constexpr int HIST_MAX_LDS_BINS = 8192;   // bins kept in LDS per workgroup (32 KiB)
constexpr int HIST_UNROLL = 4;            // pairs of pixels a thread has in flight

// mu at source point (y1, y2): bilinear interpolation between the centres of
// the four nearest pixels; within half a pixel of the map's edge the nearest
// row or column is repeated; NaN outside the map
__device__ inline double interp(const double *__restrict__ mu, const MapGeom &g, double y1, double y2)
{
    const double u = (y1 - g.ylo1) / g.pix1, v = (y2 - g.ylo2) / g.pix2;
    if (!(u >= 0.0 && v >= 0.0 && u <= (double)g.n1 && v <= (double)g.n2)) return nan("");
    const double s = fmin(fmax(u - 0.5, 0.0), (double)(g.n1 - 1));
    const double t = fmin(fmax(v - 0.5, 0.0), (double)(g.n2 - 1));
    const int64_t i0 = (int64_t)fmin(floor(s), (double)(g.n1 - 1)), j0 = (int64_t)fmin(floor(t), (double)(g.n2 - 1));
    const int64_t i1 = i0 + 1 < g.n1 ? i0 + 1 : i0, j1 = j0 + 1 < g.n2 ? j0 + 1 : j0;
    const double fs = s - (double)i0, ft = t - (double)j0;
    const double a = mu[j0 * g.n1 + i0], b = mu[j0 * g.n1 + i1];
    const double c = mu[j1 * g.n1 + i0], d = mu[j1 * g.n1 + i1];
    return (1.0 - ft) * ((1.0 - fs) * a + fs * b) + ft * ((1.0 - fs) * c + fs * d);
}

// point k of npts evenly spaced from (y1a, y2a) to (y1b, y2b), both ends included
__global__ void k_light_curve(const double *__restrict__ mu, MapGeom g, double y1a, double y2a, double y1b,
                              double y2b, int64_t npts, double *__restrict__ out)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= npts) return;
    const double f = npts > 1 ? (double)k / (double)(npts - 1) : 0.0;
    out[k] = interp(mu, g, y1a + f * (y1b - y1a), y2a + f * (y2b - y2a));
}

// bin of log10(mu): 0 underflow (mu <= 0 or below lo), 1 .. nbins the bins
// [lo + (b - 1) w, lo + b w), nbins + 1 overflow (and NaN)
__device__ inline int hist_bin(double m, double lo, double inv_w, int nbins)
{
    if (!(m > 0.0)) return isnan(m) ? nbins + 1 : 0;
    const double x = (log10(m) - lo) * inv_w;
    if (x < 0.0) return 0;
    if (!(x < (double)nbins)) return nbins + 1;
    return 1 + (int)x;
}

// The same bin, mostly without the FP64 logarithm (some 90 instructions): from
// log2 of the mantissa in FP32, good to 2^-22, so a position within eps bins of a
// bin's edge is formed again in full.  eps: HIST_EPS in log10, and the rounding of
// the differences from a far lower end (HIST_ROUND of the ends' size: half a unit of
// the difference and of the product, in either form), in bins.
constexpr double HIST_EPS = 5e-7, HIST_ROUND = 0x1p-50;
__device__ inline int hist_bin_fast(double m, double lo, double inv_w, int nbins, double eps)
{
    // (0.30103 = log10 2; the exponent of zeros, infinities and NaN is 0 here)
    const double l = (double)__builtin_amdgcn_logf((float)__builtin_amdgcn_frexp_mant(m)) +
                     (double)__builtin_amdgcn_frexp_exp(m);
    const double x = (l * 0.30102999566398119521 - lo) * inv_w, f = floor(x);
    const bool sure = m > 0x1p-1022 && m < 0x1p1023 && x - f >= eps && x - f <= 1.0 - eps;
    if (!sure) return hist_bin(m, lo, inv_w, nbins);
    return x < 0.0 ? 0 : (x < (double)nbins ? 1 + (int)x : nbins + 1);
}

// counts per bin; a workgroup privatises the bins in LDS and adds them to
// the device counts once.  Workgroups are large and few: their additions meet at
// the same addresses (a 2000 x 2000 map in 200 bins: 12 us, with 977 workgroups of
// 256 threads 26, and with 64-bit counts and every pixel's FP64 logarithm besides
// 32; its 32 MB take 7).  head: pixels before the first 16-byte boundary (0 or
// 1), pairs: pairs of pixels behind it.
__global__ __launch_bounds__(HIST_BLK) void k_histogram(const double *__restrict__ mu, int64_t npix, int head,
                                                        int64_t pairs, double lo, double inv_w, int nbins, double eps,
                                                        unsigned long long *__restrict__ counts)
{
    extern __shared__ unsigned h[];   // (a workgroup's share is far below 2^32 pixels)
    const int nb = nbins + 2;
    for (int b = threadIdx.x; b < nb; b += blockDim.x) h[b] = 0;
    __syncthreads();
    auto put = [&](double m) { atomicAdd(&h[hist_bin_fast(m, lo, inv_w, nbins, eps)], 1u); };
    const double2 *mp = reinterpret_cast<const double2 *>(mu + head);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, k0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t k = k0;
    for (; k + (HIST_UNROLL - 1) * stride < pairs; k += HIST_UNROLL * stride) {
        double2 v[HIST_UNROLL];
#pragma unroll
        for (int i = 0; i < HIST_UNROLL; ++i) v[i] = mp[k + i * stride];
#pragma unroll
        for (int i = 0; i < HIST_UNROLL; ++i) {
            put(v[i].x);
            put(v[i].y);
        }
    }
    for (; k < pairs; k += stride) {
        const double2 v = mp[k];
        put(v.x);
        put(v.y);
    }
    if (k0 == 0) {
        if (head) put(mu[0]);
        if (head + 2 * pairs < npix) put(mu[npix - 1]);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += blockDim.x)
        if (h[b]) atomicAdd(&counts[b], (unsigned long long)h[b]);
}

// the same without LDS, for more bins than a workgroup's LDS holds
__global__ void k_histogram_global(const double *__restrict__ mu, int64_t npix, double lo, double inv_w, int nbins,
                                   unsigned long long *__restrict__ counts)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < npix) atomicAdd(&counts[hist_bin(mu[k], lo, inv_w, nbins)], 1ull);
}

__global__ void k_zero_counts(unsigned long long *c, int n)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) c[k] = 0;
}

}  // namespace

void launch_light_curve(const double *mu, const MapGeom &g, double y1a, double y2a, double y1b, double y2b,
                        int64_t npts, double *out, hipStream_t st)
{
    if (npts > 0)
        hipLaunchKernelGGL(k_light_curve, dim3((unsigned)((npts + 255) / 256)), dim3(256), 0, st, mu, g, y1a, y2a, y1b,
                           y2b, npts, out);
}

void launch_histogram(const double *mu, int64_t npix, double lo, double hi, int nbins, unsigned long long *counts,
                      hipStream_t st)
{
    const int nb = nbins + 2;
    hipLaunchKernelGGL(k_zero_counts, dim3((unsigned)((nb + 255) / 256)), dim3(256), 0, st, counts, nb);
    if (npix <= 0) return;
    const double inv_w = (double)nbins / (hi - lo);
    if (nb <= HIST_MAX_LDS_BINS) {
        const double eps = (HIST_EPS + HIST_ROUND * (std::fabs(lo) + std::fabs(hi))) * inv_w;
        const int head = (reinterpret_cast<uintptr_t>(mu) & 15) ? 1 : 0;   // (mu is aligned to its doubles)
        const int64_t pairs = (npix - head) / 2;
        // 16 pixels a thread, 4 where that leaves fewer than 192 workgroups: pixels at
        // a bin's edge (a map of magnification 1 in bins that begin there) take the
        // logarithm in FP64 as well, and few workgroups then wait for it (1000 x 1000
        // of them, the whole call: 40 us by 62 workgroups, 32 by 245; spread over the
        // bins 29 and 28)
        int64_t want = (npix + HIST_BLK * 16 - 1) / (HIST_BLK * 16);
        if (want < 192) want = std::min<int64_t>((npix + HIST_BLK * 4 - 1) / (HIST_BLK * 4), 256);
        const unsigned grid = (unsigned)std::min<int64_t>(std::max<int64_t>(want, 1), 512);
        hipLaunchKernelGGL(k_histogram, dim3(grid), dim3(HIST_BLK), (size_t)nb * sizeof(unsigned), st, mu, npix, head,
                           pairs, lo, inv_w, nbins, eps, counts);
    } else {
        hipLaunchKernelGGL(k_histogram_global, dim3((unsigned)((npix + 255) / 256)), dim3(256), 0, st, mu, npix, lo,
                           inv_w, nbins, counts);
    }
}

}  // namespace mlm
