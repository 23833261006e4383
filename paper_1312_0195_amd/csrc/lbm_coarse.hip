// lbm_coarse.hip -- coarse-grid solve of the upscaled scheme (Sec. 3, Sec. 4.3).
//
// Each coarse cell stands for an r x r subdomain of the fine grid and carries
// the effective permeability found by the local problems. The coarse run uses
// the same scheme as the fine grid with the same physical rho0, nu_eff, eps,
// nu and G, while dx and dt both grow by r (Sec. 4.3: dx 0.0025 -> 0.025 m and
// dt 2.5e-5 -> 2.5e-4 s, tau 0.50012 -> 0.500012). In lattice units:
//   tau_c = 1/2 + (tau_f - 1/2) / r,  nu_c = nu_f / r,
//   kappa_c = kappa_f / r^2,           G_c = r G_f,   u_c = u_f.
// The drag uses either the scalar kappa* = (kxx + kyy) / 2 (Sec. 4.3) or the
// full tensor (Eq. f_m-depends-on-u-and-tensor-k), through the per-cell matrix
// M = (K + eps nu I / 2)^{-1} K with rho u = M (j + eps rho G / 2).
//
// Three ranges of size. Up to 1664 cells one persistent workgroup, one or two
// cells per thread, with the in-place streaming of the local solver takes every
// step without a launch. From there to 4096 cells (FP64 state 2048) the fine
// grid's many-step launches run the lattice on all CUs, and the same
// convergence test on the velocity field is taken on the device; with few steps
// between checks the one workgroup stays the faster (in_one_group). Larger coarse
// grids are a fine-grid solve with a tensor permeability (its own test, on the
// mean velocity). us per step with FP32 / FP64 state, a check every 100: 8 x 8
// 0.57 / 0.24 -> 0.24 / 0.21, 32 x 32 1.65 / 0.61 -> 0.62 / 0.57, 45 x 45 2.50 /
// 1.19 -> 0.83 / 0.81, 64 x 64 3.5 -> 0.82; before, one workgroup ran up to four
// cells per thread. The line between the first two: at 40 x 40 one workgroup takes
// 0.9 us per step, the launches 0.8 and 0.1 ms more per solve.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "lbm_internal.h"

namespace lbm {
namespace {

constexpr int kOneGroup = 1664;  // cells up to which one workgroup runs every solve
// cells up to which the convergence test is on the velocity field
constexpr int kField32 = 4096, kField64 = 2048;

template <typename R>
struct CoarseArgs {
    int nx, ny;
    const R *__restrict__ M;         // [4][N] per-cell drag deficit E = I - M (e00, e01, e10, e11),
                                     // M = (K + h I)^{-1} K; E keeps its relative precision in FP32
    const R *__restrict__ heg;       // [2][N] eps G_c / 2 per cell
    double om, omc, twotau, omtt;
    double tol;
    int check_every;
    int max_steps;
    double *__restrict__ u_out;      // [2][N]
    double *__restrict__ rho_out;    // [N] or null
    long long *__restrict__ status;  // [0] steps, [1] flag
    const int *__restrict__ bad;     // set by k_coarse_coef: nothing is run
};

// Coefficients of the coarse lattice from the effective permeability (FP64),
// rounded once to the storage type R.
template <typename R>
__global__ void k_coarse_coef(const double *__restrict__ keff, const double *__restrict__ force, int n,
                              int tensor, double r, double eps, double nu_c, double gxf, double gyf,
                              R *__restrict__ M, R *__restrict__ heg, double *__restrict__ perm_c,
                              double *__restrict__ force_c, int *__restrict__ bad)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    const double s = 1.0 / (r * r);  // kappa_c = kappa_f / r^2
    double kxx = keff[4 * c] * s, kxy = keff[4 * c + 1] * s, kyx = keff[4 * c + 2] * s, kyy = keff[4 * c + 3] * s;
    if (!tensor) {
        const double k = 0.5 * (kxx + kyy);
        kxx = kyy = k;
        kxy = kyx = 0.0;
    }
    const double h = 0.5 * eps * nu_c;
    const double det = kxx * kyy - kxy * kyx;
    const double axx = kxx + h, ayy = kyy + h;
    const double adet = axx * ayy - kxy * kyx;
    if (!(std::isfinite(det) && det > 0.0 && std::isfinite(adet) && adet != 0.0 && kxx > 0.0 && kyy > 0.0))
        atomicOr(bad, 1);
    // E = I - M = h (K + h I)^{-1}: rounded to FP32, M itself would lose the
    // relative precision of the drag I - M of permeable cells
    const double ia = h / adet;
    const int N = n;
    M[c] = (R)(ia * ayy);
    M[N + c] = (R)(-ia * kxy);
    M[2 * N + c] = (R)(-ia * kyx);
    M[3 * N + c] = (R)(ia * axx);
    const double gx = r * (force ? force[2 * c] : gxf), gy = r * (force ? force[2 * c + 1] : gyf);
    heg[c] = (R)(0.5 * eps * gx);
    heg[N + c] = (R)(0.5 * eps * gy);
    if (perm_c) {
        perm_c[4 * c] = kxx;
        perm_c[4 * c + 1] = kxy;
        perm_c[4 * c + 2] = kyx;
        perm_c[4 * c + 3] = kyy;
        force_c[2 * c] = gx;
        force_c[2 * c + 1] = gy;
    }
}

// Collision in FP64 (deviation form, tensor drag), f in and out.
template <typename R>
__device__ __forceinline__ void collide_t(double f[9], const R m[4], R hx0, R hy0, const CoarseArgs<R> &a)
{
    const double dr = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
    const double jx = (f[1] - f[3]) + ((f[5] - f[6]) + (f[8] - f[7]));
    const double jy = (f[2] - f[4]) + ((f[5] + f[6]) - (f[7] + f[8]));
    const double rho = 1.0 + dr;
    const double hx = jx + (double)hx0 * rho, hy = jy + (double)hy0 * rho;
    // M h = h - E h
    const double mx = a.twotau * ((hx - (double)m[0] * hx) - (double)m[1] * hy) + a.omtt * jx;
    const double my = a.twotau * ((hy - (double)m[3] * hy) - (double)m[2] * hx) + a.omtt * jy;
    const double om = a.om, omc = a.omc;
    const double s0 = (4.0 / 9.0) * om * dr;
    const double b = (1.0 / 9.0) * om * dr;
    const double bx = (1.0 / 3.0) * om * mx;
    const double by = (1.0 / 3.0) * om * my;
    const double cc = (1.0 / 36.0) * om * dr;
    const double cx = (1.0 / 12.0) * om * mx;
    const double cy = (1.0 / 12.0) * om * my;
    const double pp = cx + cy, qq = cx - cy;
    f[0] = omc * f[0] + s0;
    f[1] = omc * f[1] + (b + bx);
    f[2] = omc * f[2] + (b + by);
    f[3] = omc * f[3] + (b - bx);
    f[4] = omc * f[4] + (b - by);
    f[5] = omc * f[5] + (cc + pp);
    f[6] = omc * f[6] + (cc - qq);
    f[7] = omc * f[7] + (cc - pp);
    f[8] = omc * f[8] + (cc + qq);
}

// Velocity of a cell in FP64 from its pre-collision deviations.
template <typename R>
__device__ __forceinline__ void cell_velocity(const double fd[9], const R m[4], R hx0, R hy0, double &ux,
                                              double &uy, double &rho)
{
    const double dr = ((fd[0] + fd[1]) + (fd[2] + fd[3])) + ((fd[4] + fd[5]) + (fd[6] + fd[7])) + fd[8];
    const double jx = (fd[1] - fd[3]) + ((fd[5] - fd[6]) + (fd[8] - fd[7]));
    const double jy = (fd[2] - fd[4]) + ((fd[5] + fd[6]) - (fd[7] + fd[8]));
    rho = 1.0 + dr;
    const double hx = jx + (double)hx0 * rho, hy = jy + (double)hy0 * rho;
    ux = ((hx - (double)m[0] * hx) - (double)m[1] * hy) / rho;
    uy = ((hy - (double)m[3] * hy) - (double)m[2] * hx) / rho;
}

// One workgroup runs the whole periodic coarse lattice to steady state.
// Convergence: relative L2 change of the velocity field between checks. The
// previous field is kept in the storage type R, and the new field is rounded
// to R before the difference, so a state that no longer changes gives
// exactly zero. Bound by the chain of LDS reads, collision, writes and barrier
// of a step (about 0.25 us), and from four waves per SIMD on by the collision.
template <typename R, int T, int CPT>
__global__ __launch_bounds__(T) void k_coarse_onchip(CoarseArgs<R> a)
{
    constexpr int S = T * CPT;  // plane stride
    __shared__ R A[8 * S];
    __shared__ double red[T / 64][2];
    const int nx = a.nx, ny = a.ny, N = nx * ny;
    if (*a.bad) return;
    R f0[CPT], m[CPT][4], hg[CPT][2], upx[CPT], upy[CPT];
    int x[CPT], xm[CPT], xp[CPT], r0[CPT], rm[CPT], rp[CPT];
    bool own[CPT];
#pragma unroll
    for (int k = 0; k < CPT; ++k) {
        const int c = threadIdx.x + k * T;
        own[k] = c < N;
        f0[k] = upx[k] = upy[k] = (R)0;
        const int y = c / nx;
        x[k] = c - y * nx;
        xm[k] = x[k] == 0 ? nx - 1 : x[k] - 1;
        xp[k] = x[k] == nx - 1 ? 0 : x[k] + 1;
        r0[k] = y * nx;
        rm[k] = (y == 0 ? ny - 1 : y - 1) * nx;
        rp[k] = (y == ny - 1 ? 0 : y + 1) * nx;
        if (own[k]) {
#pragma unroll
            for (int q = 0; q < 4; ++q) m[k][q] = a.M[q * N + c];
            hg[k][0] = a.heg[c];
            hg[k][1] = a.heg[N + c];
#pragma unroll
            for (int q = 0; q < 8; ++q) A[q * S + c] = (R)0;
        }
    }
    __syncthreads();
    int steps = 0, flag = 1;
    bool have_prev = false;
    while (true) {
        for (int st = 0; st < a.check_every; st += 2) {
#pragma unroll
            for (int k = 0; k < CPT; ++k)
                if (own[k]) {  // own slots, written back reversed
                    const int c = threadIdx.x + k * T;
                    double f[9];
                    f[0] = (double)f0[k];
#pragma unroll
                    for (int q = 1; q < 9; ++q) f[q] = (double)A[(q - 1) * S + c];
                    collide_t(f, m[k], hg[k][0], hg[k][1], a);
                    A[2 * S + c] = (R)f[1];
                    A[3 * S + c] = (R)f[2];
                    A[0 * S + c] = (R)f[3];
                    A[1 * S + c] = (R)f[4];
                    A[6 * S + c] = (R)f[5];
                    A[7 * S + c] = (R)f[6];
                    A[4 * S + c] = (R)f[7];
                    A[5 * S + c] = (R)f[8];
                    f0[k] = (R)f[0];
                }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < CPT; ++k)
                if (own[k]) {  // the neighbours' slots
                    double f[9];
                    f[0] = (double)f0[k];
                    f[1] = (double)A[2 * S + r0[k] + xm[k]];
                    f[2] = (double)A[3 * S + rm[k] + x[k]];
                    f[3] = (double)A[0 * S + r0[k] + xp[k]];
                    f[4] = (double)A[1 * S + rp[k] + x[k]];
                    f[5] = (double)A[6 * S + rm[k] + xm[k]];
                    f[6] = (double)A[7 * S + rm[k] + xp[k]];
                    f[7] = (double)A[4 * S + rp[k] + xp[k]];
                    f[8] = (double)A[5 * S + rp[k] + xm[k]];
                    collide_t(f, m[k], hg[k][0], hg[k][1], a);
                    A[0 * S + r0[k] + xp[k]] = (R)f[1];
                    A[1 * S + rp[k] + x[k]] = (R)f[2];
                    A[2 * S + r0[k] + xm[k]] = (R)f[3];
                    A[3 * S + rm[k] + x[k]] = (R)f[4];
                    A[4 * S + rp[k] + xp[k]] = (R)f[5];
                    A[5 * S + rp[k] + xm[k]] = (R)f[6];
                    A[6 * S + rm[k] + xm[k]] = (R)f[7];
                    A[7 * S + rm[k] + xp[k]] = (R)f[8];
                    f0[k] = (R)f[0];
                }
            __syncthreads();
        }
        steps += a.check_every;
        double d2 = 0.0, u2 = 0.0;
        double ux[CPT], uy[CPT], rho[CPT];
#pragma unroll
        for (int k = 0; k < CPT; ++k)
            if (own[k]) {
                double fd[9];
                fd[0] = (double)f0[k];
#pragma unroll
                for (int q = 1; q < 9; ++q) fd[q] = (double)A[(q - 1) * S + threadIdx.x + k * T];
                cell_velocity(fd, m[k], hg[k][0], hg[k][1], ux[k], uy[k], rho[k]);
                const R rx = (R)ux[k], ry = (R)uy[k];
                const double dx = (double)rx - (double)upx[k], dy = (double)ry - (double)upy[k];
                d2 += dx * dx + dy * dy;
                u2 += ux[k] * ux[k] + uy[k] * uy[k];
                upx[k] = rx;
                upy[k] = ry;
            }
        d2 = wave_sum(d2);
        u2 = wave_sum(u2);
        if ((threadIdx.x & 63) == 0) {
            red[threadIdx.x >> 6][0] = d2;
            red[threadIdx.x >> 6][1] = u2;
        }
        __syncthreads();
        double td = 0.0, tu = 0.0;
        for (int w = 0; w < T / 64; ++w) {
            td += red[w][0];
            tu += red[w][1];
        }
        bool stop = false;
        if (!isfinite(td) || !isfinite(tu)) {
            flag = 2;
            stop = true;
        } else if (have_prev && a.tol > 0.0 && sqrt(td) <= a.tol * sqrt(tu)) {
            flag = 0;
            stop = true;
        } else if (steps >= a.max_steps) {
            flag = (a.tol > 0.0) ? 1 : 0;
            stop = true;
        }
        have_prev = true;
        __syncthreads();
        if (stop) {  // the fields of this check (even order after an even number of steps)
#pragma unroll
            for (int k = 0; k < CPT; ++k)
                if (own[k]) {
                    const int c = threadIdx.x + k * T;
                    a.u_out[c] = ux[k];
                    a.u_out[N + c] = uy[k];
                    if (a.rho_out) a.rho_out[c] = rho[k];
                }
            break;
        }
    }
    if (threadIdx.x == 0) {
        a.status[0] = steps;
        a.status[1] = flag;
    }
}

__global__ void k_zero_i32c(int *p) { p[0] = 0; }

// Mean of each r x r block of nplanes fields [plane][ny][nx]: one workgroup
// per output value, fixed-order FP64 sum.
__global__ __launch_bounds__(256) void k_block_average(const double *__restrict__ in, int nx, int ny, int r,
                                                       double *__restrict__ out)
{
    __shared__ double red[4];
    const int ncx = nx / r, ncy = ny / r;
    const int o = blockIdx.x;  // plane * ncx * ncy + J * ncx + I
    const int plane = o / (ncx * ncy), rem = o % (ncx * ncy);
    const int J = rem / ncx, I = rem % ncx;
    const double *f = in + (size_t)plane * nx * ny;
    double s = 0.0;
    for (int k = threadIdx.x; k < r * r; k += 256) {
        const int y = J * r + k / r, x = I * r + k % r;
        s += f[(size_t)y * nx + x];
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[o] = ((red[0] + red[1]) + (red[2] + red[3])) / ((double)r * r);
}

// Whether one workgroup takes the whole solve. Beyond kOneGroup cells the launches
// pay for each check: an interval of m steps takes at least 12 us (launches, the
// check, its trip to the host), 5.9 + 0.8 m where the steps set it; one workgroup
// takes 2.5 us for the check and for a step 0.62 ns per cell with two cells per
// thread, 0.64 with three and 1.15 with four. us per step at m = 2 / 4 / 8 / 16:
// 45 x 45 FP64 2.4 / 1.8 / 1.5 / 1.3 in one workgroup, 6.0 / 3.1 / 1.6 / 1.2 in
// launches; 55 x 55 3.9 / 2.9 / 2.4 / 2.1 and 6.2 / 3.2 / 1.7 / 1.25.
bool in_one_group(int n, bool f64, int check_every)
{
    if (n <= kOneGroup) return true;
    if (n > (f64 ? kField64 : kField32)) return false;
    const double m = check_every, step = n * (n <= 2048 ? 0.62e-3 : n <= 3072 ? 0.64e-3 : 1.15e-3);
    return 2.5 + m * step <= std::max(12.0 + 0.15 * m, 5.9 + 0.8 * m);
}

struct CoarseLayout {
    bool field;  // the test on the field
    size_t off_M, off_heg, off_status, off_flag, off_perm, off_force, off_fine, fine_bytes, total;
};

CoarseLayout coarse_layout(int ncx, int ncy, bool f64)
{
    CoarseLayout L{};
    const size_t n = (size_t)ncx * ncy;
    L.field = n <= (size_t)(f64 ? kField64 : kField32);
    size_t off = 0;
    L.off_M = off;      off = align_up(off + 4 * n * sizeof(double));
    L.off_heg = off;    off = align_up(off + 2 * n * sizeof(double));
    L.off_status = off; off = align_up(off + 4 * sizeof(long long));
    L.off_flag = off;   off = align_up(off + sizeof(int));
    // the other paths need the coarse tensor, force and a fine-solver
    // workspace; sized for them always
    L.off_perm = off;   off = align_up(off + 4 * n * sizeof(double));
    L.off_force = off;  off = align_up(off + 2 * n * sizeof(double));
    lbm_params q{};
    q.nx = ncx; q.ny = ncy; q.tau = 0.75; q.eps = 0.5; q.nu = 0.1; q.rho0 = 1.0;
    q.walls_y = 0; q.pop_dtype = LBM_F64; q.perm_kind = LBM_PERM_TENSOR;
    L.fine_bytes = lbm_workspace_bytes(&q);
    L.off_fine = off;   off = align_up(off + L.fine_bytes);
    L.total = off;
    return L;
}

template <typename R>
lbm_status launch_onchip(const lbm_params &pc, char *ws, const CoarseLayout &L, double tol, int check_every,
                         int64_t max_steps, double *d_u, double *d_rho, hipStream_t stream)
{
    CoarseArgs<R> a{};
    a.nx = pc.nx;
    a.ny = pc.ny;
    a.M = reinterpret_cast<const R *>(ws + L.off_M);
    a.heg = reinterpret_cast<const R *>(ws + L.off_heg);
    a.om = 1.0 / pc.tau;
    a.omc = 1.0 - 1.0 / pc.tau;
    a.twotau = 2.0 * pc.tau;
    a.omtt = 1.0 - 2.0 * pc.tau;
    a.tol = tol;
    a.check_every = check_every;
    a.max_steps = (int)std::min<int64_t>(max_steps, (int64_t)1 << 30);
    a.u_out = d_u;
    a.rho_out = d_rho;
    a.status = reinterpret_cast<long long *>(ws + L.off_status);
    a.bad = reinterpret_cast<const int *>(ws + L.off_flag);
    const int n = pc.nx * pc.ny;
    if (n <= 256)
        hipLaunchKernelGGL((k_coarse_onchip<R, 256, 1>), dim3(1), dim3(256), 0, stream, a);
    else if (n <= 1024)
        hipLaunchKernelGGL((k_coarse_onchip<R, 1024, 1>), dim3(1), dim3(1024), 0, stream, a);
    else if (n <= 2048)
        hipLaunchKernelGGL((k_coarse_onchip<R, 1024, 2>), dim3(1), dim3(1024), 0, stream, a);
    if constexpr (sizeof(R) == 4) {  // FP64 planes of more cells do not fit LDS
        if (n > 3072)
            hipLaunchKernelGGL((k_coarse_onchip<R, 1024, 4>), dim3(1), dim3(1024), 0, stream, a);
        else if (n > 2048)
            hipLaunchKernelGGL((k_coarse_onchip<R, 1024, 3>), dim3(1), dim3(1024), 0, stream, a);
    }
    LBM_HIP(hipGetLastError());
    return LBM_OK;
}

}  // namespace
}  // namespace lbm

using namespace lbm;

extern "C" lbm_status lbm_coarse_params(const lbm_params *fine, int32_t r, lbm_params *coarse)
{
    if (!fine || !coarse) return set_error(LBM_EINVAL, "lbm_coarse_params: NULL argument");
    if (r < 1) return set_error(LBM_EINVAL, "lbm_coarse_params: r must be >= 1");
    if (fine->nx % r || fine->ny % r) return set_error(LBM_EINVAL, "lbm_coarse_params: r must divide nx and ny");
    if (fine->walls_y != 0) return set_error(LBM_EINVAL, "lbm_coarse_params: the coarse grid is periodic (walls_y = 0)");
    if (lbm_workspace_bytes(fine) == 0) return set_error(LBM_EINVAL, "lbm_coarse_params: invalid fine parameters");
    *coarse = *fine;
    coarse->nx = fine->nx / r;
    coarse->ny = fine->ny / r;
    coarse->tau = 0.5 + (fine->tau - 0.5) / r;
    coarse->nu = fine->nu / r;
    coarse->gx = fine->gx * r;
    coarse->gy = fine->gy * r;
    return LBM_OK;
}

extern "C" size_t lbm_coarse_workspace_bytes(int32_t ncx, int32_t ncy)
{
    if (ncx < 1 || ncy < 1) return 0;
    return coarse_layout(ncx, ncy, true).total;
}

extern "C" lbm_status lbm_coarse_solve(const lbm_params *fine, int32_t r, const double *d_keff, int32_t keff_mode,
                                       const double *d_force, int64_t max_steps, double tol, int32_t check_every,
                                       double *d_u, double *d_rho, int64_t *steps_done, void *d_ws,
                                       size_t ws_bytes, hipStream_t stream)
{
    const std::string fn = "lbm_coarse_solve: ";
    lbm_params pc{};
    lbm_status s = lbm_coarse_params(fine, r, &pc);
    if (s != LBM_OK) return s;
    if (fine->scheme != LBM_SCHEME_SHAN_CHEN) return set_error(LBM_EINVAL, fn + "the coarse solver runs the Shan-Chen form (scheme 0)");
    if (!d_keff || !d_u) return set_error(LBM_EINVAL, fn + "NULL keff or u");
    if (keff_mode != LBM_KEFF_SCALAR && keff_mode != LBM_KEFF_TENSOR) return set_error(LBM_EINVAL, fn + "bad keff_mode");
    if (check_every < 2 || (check_every & 1)) return set_error(LBM_EINVAL, fn + "check_every must be even and >= 2");
    if (max_steps < 1 || max_steps > (int64_t)1 << 30) return set_error(LBM_EINVAL, fn + "max_steps must lie in [1, 2^30]");
    if (!(tol >= 0.0)) return set_error(LBM_EINVAL, fn + "tol must be >= 0");
    const int ncx = pc.nx, ncy = pc.ny, n = ncx * ncy;
    const bool f64 = fine->pop_dtype == LBM_F64;
    const CoarseLayout L = coarse_layout(ncx, ncy, f64);
    const bool one_group = in_one_group(n, f64, check_every);
    const size_t need = L.total;
    if (!d_ws || ((uintptr_t)d_ws % kAlign) != 0 || ws_bytes < need)
        return set_error(LBM_EWORKSPACE, fn + "workspace NULL, misaligned or smaller than " + std::to_string(need));
    char *ws = static_cast<char *>(d_ws);
    long long *status = reinterpret_cast<long long *>(ws + L.off_status);
    int *flag = reinterpret_cast<int *>(ws + L.off_flag);
    double *perm_c = reinterpret_cast<double *>(ws + L.off_perm);
    double *force_c = reinterpret_cast<double *>(ws + L.off_force);
    pc.perm_kind = LBM_PERM_TENSOR;
    pc.pop_dtype = f64 ? LBM_F64 : LBM_F32_SHIFTED;
    hipLaunchKernelGGL(k_zero_i32c, dim3(1), dim3(1), 0, stream, flag);
    const int tensor = keff_mode == LBM_KEFF_TENSOR ? 1 : 0;
    const dim3 cg((n + 255) / 256), cb(256);
    // the coefficients go where the path that uses them reads them
    char *coef = ws + L.off_M, *heg = ws + L.off_heg;
    if (L.field && !one_group) fine_coef_planes(pc, ws + L.off_fine, &coef, &heg);
    double *pp = L.field ? nullptr : perm_c, *fp = L.field ? nullptr : force_c;
    if (f64)
        hipLaunchKernelGGL(k_coarse_coef<double>, cg, cb, 0, stream, d_keff, d_force, n, tensor, (double)r, pc.eps, pc.nu,
                           fine->gx, fine->gy, reinterpret_cast<double *>(coef), reinterpret_cast<double *>(heg), pp, fp,
                           flag);
    else
        hipLaunchKernelGGL(k_coarse_coef<float>, cg, cb, 0, stream, d_keff, d_force, n, tensor, (double)r, pc.eps, pc.nu,
                           fine->gx, fine->gy, reinterpret_cast<float *>(coef), reinterpret_cast<float *>(heg), pp, fp,
                           flag);
    LBM_HIP(hipGetLastError());

    const int64_t ms = std::min<int64_t>((max_steps + check_every - 1) / check_every * check_every, (int64_t)1 << 30);
    long long result[2] = {0, 0};
    int bad = 0;
    if (one_group) {
        // the permeability check is read back with the result: with a bad one the kernel leaves at once
        const lbm_status ls = f64 ? launch_onchip<double>(pc, ws, L, tol, check_every, ms, d_u, d_rho, stream)
                                  : launch_onchip<float>(pc, ws, L, tol, check_every, ms, d_u, d_rho, stream);
        if (ls != LBM_OK) return ls;
        LBM_HIP(hipMemcpyAsync(result, status, sizeof(result), hipMemcpyDeviceToHost, stream));
    }
    LBM_HIP(hipMemcpyAsync(&bad, flag, sizeof(int), hipMemcpyDeviceToHost, stream));
    LBM_HIP(hipStreamSynchronize(stream));
    if (bad) return set_error(LBM_EINVAL, fn + "effective permeability must be positive definite");
    if (L.field) {
        if (!one_group) {
            FieldRun f{};
            f.p = pc;
            f.p.rho0 = 1.0;  // as the one-group kernel: deviations from 1
            f.ws = ws + L.off_fine;
            f.prev = ws + L.off_perm;
            f.done = reinterpret_cast<unsigned long long *>(status);
            f.tol = tol;
            f.check_every = check_every;
            f.max_steps = ms;
            f.u = d_u;
            f.rho = d_rho;
            f.stream = stream;
            const lbm_status ls = run_to_steady_field(f, result);
            if (ls != LBM_OK) return ls;
        }
        if (steps_done) *steps_done = result[0];
        if (result[1] == 2) return set_error(LBM_ENONFINITE, fn + "non-finite velocity");
        if (result[1] == 1) return set_error(LBM_ENOTCONV, fn + "tolerance not reached within max_steps");
        return LBM_OK;
    }

    // the fine-grid solver with the coarse tensor permeability
    lbm_handle *h = nullptr;
    s = lbm_init(&h, &pc, perm_c, force_c, ws + L.off_fine, L.fine_bytes, stream);
    if (s != LBM_OK) return s;
    int64_t done = 0;
    double mu[2];
    s = lbm_step(h, max_steps, tol, check_every, &done, mu);
    if (steps_done) *steps_done = done;
    if (s == LBM_OK || s == LBM_ENOTCONV) {
        lbm_status s2 = lbm_fields(h, d_u, d_rho);
        if (s2 != LBM_OK) s = s2;
        else {
            hipError_t e = hipStreamSynchronize(stream);
            if (e != hipSuccess) s = hip_check(e, "lbm_coarse_solve");
        }
    }
    lbm_destroy(h);
    return s;
}

extern "C" lbm_status lbm_block_average(const double *d_in, int32_t nx, int32_t ny, int32_t nplanes, int32_t r,
                                        double *d_out, hipStream_t stream)
{
    if (!d_in || !d_out || nx < 1 || ny < 1 || nplanes < 1 || r < 1 || nx % r || ny % r)
        return set_error(LBM_EINVAL, "lbm_block_average: NULL pointer, or r does not divide nx and ny");
    const int64_t nout = (int64_t)nplanes * (nx / r) * (ny / r);
    if (nout >= (int64_t)1 << 31) return set_error(LBM_EINVAL, "lbm_block_average: too many blocks");
    hipLaunchKernelGGL(k_block_average, dim3((unsigned)nout), dim3(256), 0, stream, d_in, nx, ny, r, d_out);
    LBM_HIP(hipGetLastError());
    return LBM_OK;
}
