// The macro map of a lens with third-order terms on the lattice that is
// searched for the images of a map: one arithmetic for the host and the device
// (plain IEEE double operations, evaluated as written).
#pragma once
#include "internal.hpp"

namespace mlm {

constexpr int LAT = 2048;   // lattice points per axis

struct CubicSearch {
    double lam1, lam2, a, b, c, d;         // macro map
    double lo1, hi1, lo2, hi2;             // the map widened by the border (source plane)
    double ext1, ext2, s1, s2;             // half-sizes of the lattice and its steps

    __host__ __device__ inline double x(int i) const
    {
#pragma clang fp contract(off)
        return -ext1 + i * s1;
    }
    __host__ __device__ inline double y(int j) const
    {
#pragma clang fp contract(off)
        return -ext2 + j * s2;
    }
    // whether the image-plane point maps into the widened map
    __host__ __device__ inline bool hit(double x, double y) const
    {
#pragma clang fp contract(off)
        const double w1 = lam1 * x - 0.5 * (a * x * x + 2.0 * b * x * y + c * y * y);
        const double w2 = lam2 * y - 0.5 * (b * x * x + 2.0 * c * x * y + d * y * y);
        return w1 >= lo1 && w1 <= hi1 && w2 >= lo2 && w2 <= hi2;
    }
};

// box: the lattice's first and last column and row with a hit (first > last: none)
struct LatticeBox {
    int32_t i0, i1, j0, j1;
};
LatticeBox search_lattice(const CubicSearch &S, Workspace &ws, hipStream_t st);

}  // namespace mlm
