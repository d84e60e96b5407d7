// solve_kernels.hpp -- the natural-gradient step's shifted solve on the device.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstddef>
#include <cstdint>

namespace qng {

// One shifted system (Re G + eps I) x = -dt grad, all in device memory.  G:
// P x P complex row-major (its real part is used); grad: P doubles; A: scratch
// of (P + 1) P doubles (the lower triangle and, as row P, the right-hand side);
// x: P doubles; status: two words, 0 or -7 (QNG_E_NOT_SPD) when the matrix is not
// positive definite (x is then not meaningful), and then the number of the first
// pivot that is not positive and finite.
struct SolveItem {
    const double *G;
    const double *grad;
    double *A;
    double *x;
    int32_t *status;
    int32_t P;
    int32_t pad;
};

// Solves one system, or `n` systems listed in device memory (max_P: the
// largest of them) together.  Bitwise reproducible.
void launch_shifted_solve(const SolveItem &one, double eps, double dt, hipStream_t st);
void launch_shifted_solves(const SolveItem *items_dev, int n, int max_P, double eps, double dt, hipStream_t st);

// dst[0 .. count) <- src when *status is 0 (device words).
void launch_copy_if_ok(const int32_t *status, const double *src, double *dst, int64_t count, hipStream_t st);

}  // namespace qng
