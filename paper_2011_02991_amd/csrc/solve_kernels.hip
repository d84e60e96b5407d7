// solve_kernels.hip -- the natural-gradient step's shifted solve on the device.
//
// The step of Sec. 1 is g dtheta = -dt grad E with g = Re G, solved with a
// Tikhonov shift: (Re G + eps I) dtheta = -dt grad E.  The steps keep G and
// grad E on the device, so the solve runs there too, by Cholesky in FP64:
// right-looking in panels of kNB columns, with the right-hand side carried as
// one more row of the matrix (its panel solve is the forward substitution).
//
//   k_solve_panel   one work-group per system: factors the kNB x kNB diagonal
//                   block in one wavefront and solves the rows below against it,
//                   one row per thread.  Latency (a chain of kNB pivots).
//   k_solve_update  one work-group per 32 x 32 tile of the trailing triangle:
//                   A_IJ -= L_I L_J^T from two panels in LDS.
//   k_solve_back    one work-group per system: L^T x = z from the last panel up.
//
// P is a few hundred and P^3/3 a few ten million multiply-adds, so what counts
// is the serial chain: a column at a time (one work-group, three barriers and a
// sweep over the trailing triangle in memory per column) took 12.6 ms at P = 432
// and 7.2 ms at P = 352; in panels of 32 the triangle is read and written
// P / 32 times, by as many work-groups as it has tiles, and the whole solve takes
// 0.40 ms and 0.33 ms (k_solve_panel 16 us, k_solve_update 7 us a panel, most of
// both latency; k_solve_back 46 us).  Systems of a batch share every launch.
//
// A non-positive or non-finite pivot sets the system's status word to
// QNG_E_NOT_SPD and the word after it to the pivot's number, and the later kernels
// leave that system alone; k_copy_if_ok lets every output follow the status.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "solve_kernels.hpp"

namespace qng {

namespace {

constexpr int kNB = 32;            // columns per panel, rows and columns per update tile
constexpr int kInitThreads = 256;
constexpr int kPanelThreads = 512;
constexpr int kBackThreads = 1024;

__device__ __forceinline__ SolveItem pick(const SolveItem *items, const SolveItem &one, int k) {
    return items ? items[k] : one;
}

// The value of lane `lane` (a constant or uniform) in every lane.
__device__ __forceinline__ double from_lane(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Lower triangle of Re G + eps I, the right-hand side as row P, status 0.
__global__ __launch_bounds__(kInitThreads) void k_solve_init(const SolveItem *items, SolveItem one, double eps,
                                                             double dt) {
    const SolveItem s = pick(items, one, blockIdx.y);
    const int P = s.P;
    const int64_t n = (int64_t)(P + 1) * P;
    for (int64_t idx = blockIdx.x * (int64_t)kInitThreads + threadIdx.x; idx < n;
         idx += (int64_t)gridDim.x * kInitThreads) {
        const int i = (int)(idx / P), j = (int)(idx % P);
        if (i == P) s.A[idx] = -dt * s.grad[j];
        else if (j <= i) s.A[idx] = s.G[2 * idx] + (i == j ? eps : 0.0);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) s.status[0] = s.status[1] = 0;
}

__global__ __launch_bounds__(kPanelThreads) void k_solve_panel(const SolveItem *items, SolveItem one, int k0) {
    const SolveItem s = pick(items, one, blockIdx.x);
    const int P = s.P;
    if (k0 >= P || *s.status != 0) return;
    const int nb = P - k0 < kNB ? P - k0 : kNB;
    // the diagonal block, then its factor transposed (a row holds a column of
    // L, so the row solves read consecutive entries) and its reciprocal diagonal
    __shared__ __align__(16) double D[kNB][kNB + 2];
    __shared__ double inv[kNB];
    __shared__ int bad;
    const int tid = threadIdx.x;
    double *A = s.A;
    // rows and columns beyond nb: the identity
    for (int t = tid; t < kNB * kNB; t += kPanelThreads) {
        const int i = t / kNB, j = t % kNB;
        D[i][j] = (i < nb && j <= i) ? A[(int64_t)(k0 + i) * P + k0 + j] : (i == j ? 1.0 : 0.0);
    }
    if (tid == 0) bad = 0;
    __syncthreads();
    if (tid < 64) {
        // lane i holds row i of the block; the entries of column k pass between
        // lanes through scalar registers
        const int i = tid & (kNB - 1);
        double r[kNB];
#pragma unroll
        for (int j = 0; j < kNB; ++j) r[j] = D[i][j];
        int fail = 0;
#pragma unroll
        for (int k = 0; k < kNB; ++k) {
            const double d = from_lane(r[k], k);
            if (!(d > 0.0) || !isfinite(d)) fail = 1;
            // (lanes above the diagonal carry values nobody reads)
            const double l = r[k] * (1.0 / (fail ? 1.0 : sqrt(d)));
            r[k] = l;
#pragma unroll
            for (int j = k + 1; j < kNB; ++j) r[j] -= l * from_lane(l, j);
            __builtin_amdgcn_sched_barrier(0);   // one column's lane values at a time in the scalar registers
        }
        if (tid < kNB) {
#pragma unroll
            for (int j = 0; j < kNB; ++j) D[j][i] = r[j];
        }
        if (tid == 0) bad = fail;
    }
    __syncthreads();
    if (bad) {
        if (tid == 0) {
            // the first bad pivot is on the diagonal as it was (kept in the loop, its
            // number would cost the chain 491 spilled scalars)
            int k = 0;
            while (k < nb - 1 && D[k][k] > 0.0 && isfinite(D[k][k])) ++k;
            s.status[0] = -7;   // QNG_E_NOT_SPD
            s.status[1] = k0 + k;
        }
        return;
    }
    for (int t = tid; t < kNB * kNB; t += kPanelThreads) {
        const int i = t / kNB, j = t % kNB;
        if (i < nb && j <= i) A[(int64_t)(k0 + i) * P + k0 + j] = D[j][i];
        if (i == j) inv[i] = 1.0 / D[i][i];
    }
    __syncthreads();
    if (nb < kNB) {
        // the last panel: only the right-hand side is below it
        if (tid < 64) {
            const int j = tid & (kNB - 1);
            double *a = A + (int64_t)P * P + k0;
            double v = j < nb ? a[j] : 0.0;
            for (int k = 0; k < nb; ++k) {
                const double xk = __shfl(v, k) * inv[k];
                v = j == k ? xk : j > k ? v - D[k][j] * xk : v;
            }
            if (tid < nb) a[j] = v;
        }
        return;
    }
    // rows below (the right-hand side among them): x L_D^T = a
    for (int row = k0 + kNB + tid; row <= P; row += kPanelThreads) {
        double *a = A + (int64_t)row * P + k0;
        double v[kNB];
#pragma unroll
        for (int j = 0; j < kNB; ++j) v[j] = a[j];
#pragma unroll
        for (int j = 0; j < kNB; ++j) {
            int jj = j;
            asm volatile("" : "+s"(jj));   // or all of D is loaded before the rows, and spills
            v[j] *= inv[jj];
#pragma unroll
            for (int k = j + 1; k < kNB; ++k) v[k] -= v[j] * D[jj][k];
        }
#pragma unroll
        for (int j = 0; j < kNB; ++j) a[j] = v[j];
    }
}

// Tile (ti >= tj) of the rows and columns from k1 = k0 + kNB on (rows to P: the
// right-hand side): A -= L_I L_J^T over the panel's columns.
__global__ __launch_bounds__(256) void k_solve_update(const SolveItem *items, SolveItem one, int k0) {
    const SolveItem s = pick(items, one, blockIdx.y);
    const int P = s.P, k1 = k0 + kNB;
    if (k1 >= P || *s.status != 0) return;
    // tile pairs in rows: ti (ti + 1) / 2 + tj
    int ti = (int)((sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);
    while ((ti + 1) * (ti + 2) / 2 <= (int)blockIdx.x) ++ti;
    while (ti * (ti + 1) / 2 > (int)blockIdx.x) --ti;
    const int tj = (int)blockIdx.x - ti * (ti + 1) / 2;
    const int r0 = k1 + ti * kNB, c0 = k1 + tj * kNB;
    if (r0 > P || c0 >= P) return;
    __shared__ double LI[kNB][kNB + 1], LJ[kNB][kNB + 1];
    const int tid = threadIdx.x;
    double *A = s.A;
    for (int t = tid; t < kNB * kNB; t += 256) {
        const int i = t / kNB, j = t % kNB;
        LI[i][j] = r0 + i <= P ? A[(int64_t)(r0 + i) * P + k0 + j] : 0.0;
        LJ[i][j] = c0 + i < P ? A[(int64_t)(c0 + i) * P + k0 + j] : 0.0;
    }
    __syncthreads();
    // 2 x 2 entries per thread: rows y, y + 16, columns x, x + 16
    const int x = tid & 15, y = tid >> 4;
    double a00 = 0, a01 = 0, a10 = 0, a11 = 0;
#pragma unroll
    for (int k = 0; k < kNB; ++k) {
        const double p0 = LI[y][k], p1 = LI[y + 16][k], q0 = LJ[x][k], q1 = LJ[x + 16][k];
        a00 += p0 * q0;
        a01 += p0 * q1;
        a10 += p1 * q0;
        a11 += p1 * q1;
    }
    auto put = [&](int i, int j, double v) {
        const int r = r0 + i, c = c0 + j;
        if (r <= P && c < P && c <= r) A[(int64_t)r * P + c] -= v;
    };
    put(y, x, a00);
    put(y, x + 16, a01);
    put(y + 16, x, a10);
    put(y + 16, x + 16, a11);
}

__global__ __launch_bounds__(kBackThreads) void k_solve_back(const SolveItem *items, SolveItem one) {
    const SolveItem s = pick(items, one, blockIdx.x);
    const int P = s.P;
    if (P <= 0 || *s.status != 0) return;
    double *A = s.A, *z = s.A + (int64_t)P * P;
    __shared__ double D[kNB][kNB + 1], inv[kNB], xs[kNB];
    const int tid = threadIdx.x;
    for (int k0 = (P - 1) / kNB * kNB; k0 >= 0; k0 -= kNB) {
        const int nb = P - k0 < kNB ? P - k0 : kNB;
        __syncthreads();   // z and xs of the step before
        for (int t = tid; t < kNB * kNB; t += kBackThreads) {
            const int i = t / kNB, j = t % kNB;
            const double d = (i < nb && j <= i) ? A[(int64_t)(k0 + i) * P + k0 + j] : (i == j ? 1.0 : 0.0);
            D[i][j] = d;
            if (i == j) inv[i] = 1.0 / d;
        }
        __syncthreads();
        if (tid < 64) {
            // lane j holds unknown j and column j of the block
            const int j = tid & (kNB - 1);
            double c[kNB];
#pragma unroll
            for (int k = 0; k < kNB; ++k) c[k] = k > j ? D[k][j] : 0.0;
            const double ij = inv[j];
            double v = j < nb ? z[k0 + j] : 0.0;
#pragma unroll
            for (int k = kNB - 1; k >= 0; --k) {
                const double xk = from_lane(v * ij, k);
                v -= c[k] * xk;   // (c is zero on and below the diagonal)
            }
            v *= ij;
            if (tid < kNB) {
                xs[j] = v;
                if (j < nb) s.x[k0 + j] = v;
            }
        }
        __syncthreads();
        for (int i = tid; i < k0; i += kBackThreads) {
            double v0 = z[i], v1 = 0.0;
            const double *col = A + (int64_t)k0 * P + i;
            if (nb == kNB) {
#pragma unroll
                for (int k = 0; k < kNB; k += 2) {
                    v0 -= col[(int64_t)k * P] * xs[k];
                    v1 -= col[(int64_t)(k + 1) * P] * xs[k + 1];
                }
            } else {
                for (int k = 0; k < nb; ++k) v0 -= col[(int64_t)k * P] * xs[k];
            }
            z[i] = v0 + v1;
        }
    }
}

__global__ void k_copy_if_ok(const int32_t *status, const double *__restrict__ src, double *__restrict__ dst,
                             int64_t count) {
    if (*status != 0) return;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

inline void check_launch() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) throw e;
}

// 2 ceil(P / 32) + 1 launches.
void launch_all(const SolveItem *items, const SolveItem &one, int n, int max_P, double eps, double dt,
                hipStream_t st) {
    int64_t blocks = ((int64_t)(max_P + 1) * max_P + kInitThreads - 1) / kInitThreads;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(k_solve_init, dim3((unsigned)blocks, n), dim3(kInitThreads), 0, st, items, one, eps, dt);
    for (int k0 = 0; k0 < max_P; k0 += kNB) {
        hipLaunchKernelGGL(k_solve_panel, dim3(n), dim3(kPanelThreads), 0, st, items, one, k0);
        const int rows = max_P + 1 - (k0 + kNB);   // the right-hand side's row among them
        if (rows <= 1) continue;
        const int t = (rows + kNB - 1) / kNB;
        hipLaunchKernelGGL(k_solve_update, dim3(t * (t + 1) / 2, n), dim3(256), 0, st, items, one, k0);
    }
    hipLaunchKernelGGL(k_solve_back, dim3(n), dim3(kBackThreads), 0, st, items, one);
    check_launch();
}

}  // namespace

void launch_shifted_solve(const SolveItem &one, double eps, double dt, hipStream_t st) {
    if (one.P <= 0) return;
    launch_all(nullptr, one, 1, one.P, eps, dt, st);
}

void launch_shifted_solves(const SolveItem *items_dev, int n, int max_P, double eps, double dt, hipStream_t st) {
    constexpr int kMost = 32768;   // systems per launch (the grid's second dimension)
    if (max_P <= 0) return;
    for (int k = 0; k < n; k += kMost)
        launch_all(items_dev + k, SolveItem{}, n - k < kMost ? n - k : kMost, max_P, eps, dt, st);
}

void launch_copy_if_ok(const int32_t *status, const double *src, double *dst, int64_t count, hipStream_t st) {
    if (count <= 0) return;
    int64_t blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_copy_if_ok, dim3((unsigned)blocks), dim3(256), 0, st, status, src, dst, count);
    check_launch();
}

}  // namespace qng
