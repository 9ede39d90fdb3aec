// Inner loops of the host eigensolver of the subspace matrices, built for the
// wide vectors of current processors as well.  Elementwise along contiguous
// memory, with every sum of a product written as one fused operation: left to
// the compiler, the builds that have the instruction fuse and the others do not,
// and the bits of a solve follow the host's processor.
#pragma once

#include <cstddef>

#ifndef HINQS_WIDE
#ifdef __HIP_DEVICE_COMPILE__
#define HINQS_WIDE
#else
#define HINQS_WIDE __attribute__((target_clones("avx512f", "arch=haswell", "default")))
#endif
#endif

namespace hinqs {
namespace {

// p[0:n) = sum_j x[j] a_j[0:n), rows a_j of a with leading dimension lda
HINQS_WIDE void rows_combine(int n, int rows, const double *__restrict__ a, int lda,
                             const double *__restrict__ x, double *__restrict__ p) {
    for (int i = 0; i < n; ++i) p[i] = 0.0;
    for (int j = 0; j < rows; ++j)
        for (int i = 0; i < n; ++i) p[i] = __builtin_fma(x[j], a[(size_t)j * lda + i], p[i]);
}

// a -= v q^T + q v^T
HINQS_WIDE void rank2_update(int n, double *__restrict__ a, int lda, const double *__restrict__ v,
                             const double *__restrict__ q) {
    for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j)
            a[(size_t)i * lda + j] = __builtin_fma(-q[i], v[j], __builtin_fma(-v[i], q[j], a[(size_t)i * lda + j]));
}

// rows z0, z1 <- c z0 + s z1, c z1 - s z0.  Rotations come one after another, the
// z1 of one the z0 of the next, which a single operation separates.
HINQS_WIDE void rotate_pair(int n, double c, double s, double *__restrict__ z0, double *__restrict__ z1) {
    for (int q = 0; q < n; ++q) {
        const double x = z0[q], y = z1[q], sy = s * y, cy = c * y;
        z0[q] = __builtin_fma(c, x, sy);
        z1[q] = __builtin_fma(-s, x, cy);
    }
}

// z -= (beta v) (v^T z) for the rows x nvec matrix z; t: nvec elements
HINQS_WIDE void reflect(int rows, int nvec, double beta, const double *__restrict__ v, double *__restrict__ z,
                        double *__restrict__ t) {
    for (int q = 0; q < nvec; ++q) t[q] = 0.0;
    for (int i = 0; i < rows; ++i)
        for (int q = 0; q < nvec; ++q) t[q] = __builtin_fma(v[i], z[(size_t)i * nvec + q], t[q]);
    for (int i = 0; i < rows; ++i)
        for (int q = 0; q < nvec; ++q)
            z[(size_t)i * nvec + q] = __builtin_fma(-(beta * v[i]), t[q], z[(size_t)i * nvec + q]);
}

}  // namespace
}  // namespace hinqs
