// lbm_internal.h -- definitions shared by the HIP sources of liblbm.
//
// D2Q9 lattice of Sec. 2 (numbering as in the paper), FP64 reductions and the
// host-side error plumbing. Device code is written for gfx950 (wave64).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>

#include "lbm.h"

namespace lbm {

// D2Q9 weights: 4/9 for the rest population, 1/9 for the axis directions,
// 1/36 for the diagonals.
constexpr double kW0 = 4.0 / 9.0;
constexpr double kW1 = 1.0 / 9.0;
constexpr double kW5 = 1.0 / 36.0;

__host__ __device__ constexpr double weight(int a) { return a == 0 ? kW0 : (a <= 4 ? kW1 : kW5); }
__host__ __device__ constexpr int ex(int a)
{
    return (a == 1 || a == 5 || a == 8) ? 1 : ((a == 3 || a == 6 || a == 7) ? -1 : 0);
}
__host__ __device__ constexpr int ey(int a)
{
    return (a == 2 || a == 5 || a == 6) ? 1 : ((a == 4 || a == 7 || a == 8) ? -1 : 0);
}
__host__ __device__ constexpr int opposite(int a) { return a == 0 ? 0 : (a <= 4 ? 1 + (a + 1) % 4 : 5 + (a - 3) % 4); }

constexpr size_t kAlign = 256;
__host__ __device__ constexpr size_t align_up(size_t v, size_t a = kAlign) { return (v + a - 1) / a * a; }

// Host-side error state (thread local), set by the entry points.
lbm_status set_error(lbm_status s, const std::string &msg);
lbm_status hip_check(hipError_t e, const char *what);
#define LBM_HIP(call)                                            \
    do {                                                         \
        hipError_t e_ = (call);                                  \
        if (e_ != hipSuccess) return ::lbm::hip_check(e_, #call); \
    } while (0)

// Number of compute units of the current device (cached per device).
int device_cu_count();

// ---------------------------------------------------------------------------
// Wave- and block-level FP64 sums with a fixed summation order, so results do
// not depend on scheduling.
// ---------------------------------------------------------------------------

__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// A periodic lattice with a tensor drag and a force per cell, run from rest until
// its velocity field changes by no more than tol (relative, L2) between checks
// (the middle range of the coarse solve, in lbm_fine.hip).
struct FieldRun {
    lbm_params p;
    char *ws;              // a fine-grid workspace for p, its coefficient planes filled
    void *prev;            // 2 n values of the population type
    unsigned long long *done;  // a device counter
    double tol;
    int check_every;
    int64_t max_steps;     // a multiple of check_every
    double *u, *rho;       // [2][n], [n] or null
    hipStream_t stream;
};

// Where a fine-grid workspace for p holds its coefficient and force planes.
void fine_coef_planes(const lbm_params &p, char *ws, char **coef, char **force);

// result: steps and flag (0 converged or no tolerance, 1 step cap, 2 non-finite).
lbm_status run_to_steady_field(const FieldRun &f, long long result[2]);

}  // namespace lbm

// The first launch of a fine-grid solver of these parameters over a stretch of
// `steps` steps, on a device of `cus` compute units: steps, kernel (in the order
// of lbm_fine.hip's Shape, -1: k_step) and tile, and its predicted time. Host
// only; for the tests, which have to reach every kernel.
extern "C" lbm_status lbm_plan_of(const lbm_params *p, int32_t force, int32_t cus, int64_t steps, int32_t out[4],
                                  double *us);

// What a D3Q19 solver of these parameters does on a device of `cus` compute
// units: steps per launch, tile (x, y) and planes per run (0, 0, 1 for single
// steps). Host only; for the tests, which have to reach every kernel.
extern "C" lbm_status lbm3d_plan_of(const lbm3d_params *p, int32_t cus, int32_t out[4]);
