// lbm_fine.hip -- fine-grid solver of liblbm (Sec. 2.2 of the paper).
//
// A time step is a pull: every cell pulls its nine incoming post-collision
// populations from its neighbours (streaming of Eq. f-evolution-of-S-C read
// backwards), collides them in registers and writes the nine new
// post-collision values to its own cell. k_step does one step per pass over
// HBM; k_tile and k_rows do several steps per pass, the intermediate steps
// staying on chip (temporal blocking, bit-identical to single steps).
// The state in memory is therefore the post-collision populations of the
// previous step; the pre-collision populations at the current step are the
// pulled ones, which is what lbm_fields and lbm_get_populations report.
//
// Storage: structure of arrays, plane a holds population a for all cells
// (x fastest), so each of the 9 loads and 9 stores of a wavefront is 64
// consecutive elements. FP32 planes store deviations f_a - w_a rho0 from the
// rest state: the velocity signal is ~1e-5 of a population, and storing the
// deviations keeps FP32 rounding relative to the signal, not to w_a rho0.
//
// Collision in deviation form, with dr = sum f~, j = sum e f~, rho = rho0 + dr:
//   rho u    = D (j + eps rho G / 2)                  Eq. explicit-u-in-Guo
//   rho u_eq = 2 tau rho u + (1 - 2 tau) j            Eq. final-ueq-of-S-C
//   f~eq_a   = w_a (dr + 3 e_a . rho u_eq)            Eq. feq minus w_a rho0
//   f~*_a    = f~_a + (f~eq_a - f~_a) / tau           Eq. f-evolution-of-S-C
// with D = 1 / (1 + eps nu / (2 kappa)) per cell, or, for a tensor
// permeability K, rho u = (K + eps nu I / 2)^{-1} K (j + eps rho G / 2) (Eq.
// u-of-S-C with Eq. f_m-depends-on-u-and-tensor-k). No division is needed in
// the step. The coefficient planes hold the drag deficit E = 1 - D =
// h / (kappa + h), h = eps nu / 2 (tensor: I - M = h (K + h I)^{-1}), not D:
// rounded to FP32, D would lose the relative precision of the drag 1 - D in
// permeable cells (its absolute rounding error 2^-25 is 2e-4 of 1 - D at
// kappa = 130, eps nu = 0.04), E keeps it; D = 1 - E is formed in FP64. The algebra is exact; only the rounding order differs from a
// literal transcription. The collision arithmetic is FP64 for both storage
// types; FP32 storage only rounds the nine values written per cell.
#include <hip/hip_runtime.h>

#include <unistd.h>

#include <chrono>
#include <cmath>
#include <cstring>
#include <algorithm>
#include <new>
#include <type_traits>

#include "lbm_internal.h"

namespace lbm {
namespace {

constexpr int kBlock = 256;
constexpr size_t kPlanePadBytes = 16384;

template <typename R>
struct StepArgs {
    const R *__restrict__ fin;
    R *__restrict__ fout;
    const R *__restrict__ coef;    // perm_kind planes of cstride elements
    const R *__restrict__ hforce;  // 2 planes: eps G / 2 per cell (or null)
    int nx, ny;
    int stride;   // plane stride of the populations, elements
    int cstride;  // plane stride of coef / hforce, elements
    R om;         // 1 / tau
    R omc;        // 1 - 1 / tau
    R twotau;     // 2 tau
    R omtt;       // 1 - 2 tau
    R hegx, hegy; // eps G / 2 for a uniform force
    R rho0;
    // FP64 copies of the constants for the FP64 arithmetic
    double hegx_d, hegy_d, om_d, omc_d, twotau_d, omtt_d, rho0_d;
};

// The relaxation constants in the arithmetic type A of a collision: FP64
// arithmetic uses the FP64 copies, FP32 arithmetic the storage-type ones.
template <typename A, typename R>
struct Kc {
    A om, omc, twotau, omtt, hegx, hegy, rho0;
    A hegx2, hegy2;  // 2 hegx, 2 hegy (exact)
    __device__ explicit Kc(const StepArgs<R> &a)
    {
        if constexpr (sizeof(A) == 8) {
            om = a.om_d; omc = a.omc_d; twotau = a.twotau_d; omtt = a.omtt_d;
            hegx = a.hegx_d; hegy = a.hegy_d; rho0 = a.rho0_d;
        } else {
            om = (A)a.om; omc = (A)a.omc; twotau = (A)a.twotau; omtt = (A)a.omtt;
            hegx = (A)a.hegx; hegy = (A)a.hegy; rho0 = (A)a.rho0;
        }
        hegx2 = hegx + hegx;
        hegy2 = hegy + hegy;
    }
};

// Plane accessors: element i of plane q of an SoA array with a plane stride.
// GMem indexes through a 64-bit pointer per lane. BMem goes through a buffer
// resource per plane, built in scalar registers from the (uniform) plane base,
// so a lane only supplies a 32-bit byte offset: this removes the 64-bit
// address arithmetic from the VALU. An offset past the plane reads zero and a
// store there is dropped (the hardware bounds check of raw buffer accesses).
// Plane bytes stay below 2^31 (the grid-size limit of params_ok).
template <typename R>
struct GMem {
    const R *p;
    R *w;
    int stride;
    __device__ R ld(int q, int i) const { return p[(size_t)q * stride + i]; }
    __device__ void st(int q, int i, R v) const { w[(size_t)q * stride + i] = v; }
};

template <typename R>
struct BMem {
    const R *p;
    R *w;
    int stride;
    static constexpr int kFlags = 0x00020000;  // gfx9 dword 3: 32-bit data format
    __device__ R ld(int q, int i) const
    {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(p + (size_t)q * stride), 0, stride * (int)sizeof(R), kFlags);
        if constexpr (sizeof(R) == 4)
            return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(r, i * 4, 0, 0));
        else
            return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b64(r, i * 8, 0, 0));
    }
    __device__ void st(int q, int i, R v) const
    {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(w + (size_t)q * stride), 0, stride * (int)sizeof(R), kFlags);
        if constexpr (sizeof(R) == 4)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, i * 4, 0, 0);
        else
            __builtin_amdgcn_raw_buffer_store_b64(
                __builtin_bit_cast(decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0)), v), r, i * 8, 0, 0);
    }
};

// Pull the nine pre-collision deviations of cell (x, y): f_a(x) = f*_a(x - e_a)
// from the previous step, with periodic wrap in x (and in y without walls)
// and halfway bounce-back f_a(x) = f*_opp(a)(x) where x - e_a is beyond a wall.
template <typename R, bool WALLS>
__device__ __forceinline__ void pull(const R *__restrict__ fin, int stride, int nx, int ny, int x,
                                     int y, R f[9])
{
    const int xm = (x == 0) ? nx - 1 : x - 1;
    const int xp = (x == nx - 1) ? 0 : x + 1;
    const int rc = y * nx;
    const R *p0 = fin;
    const R *p1 = fin + stride;
    const R *p2 = fin + 2 * (size_t)stride;
    const R *p3 = fin + 3 * (size_t)stride;
    const R *p4 = fin + 4 * (size_t)stride;
    const R *p5 = fin + 5 * (size_t)stride;
    const R *p6 = fin + 6 * (size_t)stride;
    const R *p7 = fin + 7 * (size_t)stride;
    const R *p8 = fin + 8 * (size_t)stride;
    f[0] = p0[rc + x];
    f[1] = p1[rc + xm];
    f[3] = p3[rc + xp];
    if (WALLS) {
        const bool lo = (y == 0), hi = (y == ny - 1);
        const int rm = (lo ? y : y - 1) * nx;
        const int rp = (hi ? y : y + 1) * nx;
        f[2] = lo ? p4[rc + x] : p2[rm + x];
        f[5] = lo ? p7[rc + x] : p5[rm + xm];
        f[6] = lo ? p8[rc + x] : p6[rm + xp];
        f[4] = hi ? p2[rc + x] : p4[rp + x];
        f[7] = hi ? p5[rc + x] : p7[rp + xp];
        f[8] = hi ? p6[rc + x] : p8[rp + xm];
    } else {
        const int rm = ((y == 0) ? ny - 1 : y - 1) * nx;
        const int rp = ((y == ny - 1) ? 0 : y + 1) * nx;
        f[2] = p2[rm + x];
        f[5] = p5[rm + xm];
        f[6] = p6[rm + xp];
        f[4] = p4[rp + x];
        f[7] = p7[rp + xp];
        f[8] = p8[rp + xm];
    }
}

// pull through a plane accessor (same indices as pull)
template <typename R, bool WALLS, class M>
__device__ __forceinline__ void pullm(const M &in, int nx, int ny, int x, int y, R f[9])
{
    const int xm = (x == 0) ? nx - 1 : x - 1;
    const int xp = (x == nx - 1) ? 0 : x + 1;
    const int rc = y * nx;
    f[0] = in.ld(0, rc + x);
    f[1] = in.ld(1, rc + xm);
    f[3] = in.ld(3, rc + xp);
    if (WALLS) {
        const bool lo = (y == 0), hi = (y == ny - 1);
        const int rm = (lo ? y : y - 1) * nx;
        const int rp = (hi ? y : y + 1) * nx;
        f[2] = lo ? in.ld(4, rc + x) : in.ld(2, rm + x);
        f[5] = lo ? in.ld(7, rc + x) : in.ld(5, rm + xm);
        f[6] = lo ? in.ld(8, rc + x) : in.ld(6, rm + xp);
        f[4] = hi ? in.ld(2, rc + x) : in.ld(4, rp + x);
        f[7] = hi ? in.ld(5, rc + x) : in.ld(7, rp + xp);
        f[8] = hi ? in.ld(6, rc + x) : in.ld(8, rp + xm);
    } else {
        const int rm = ((y == 0) ? ny - 1 : y - 1) * nx;
        const int rp = ((y == ny - 1) ? 0 : y + 1) * nx;
        f[2] = in.ld(2, rm + x);
        f[5] = in.ld(5, rm + xm);
        f[6] = in.ld(6, rm + xp);
        f[4] = in.ld(4, rp + x);
        f[7] = in.ld(7, rp + xp);
        f[8] = in.ld(8, rp + xm);
    }
}

template <typename R>
__device__ __forceinline__ void moments(const R f[9], R &dr, R &jx, R &jy)
{
    dr = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
    jx = (f[1] - f[3]) + ((f[5] - f[6]) + (f[8] - f[7]));
    jy = (f[2] - f[4]) + ((f[5] + f[6]) - (f[7] + f[8]));
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2). Renumber them so that each XCD gets one contiguous run of row
// segments: the cache lines that neighbouring segments share (x-shifted
// populations) and the rows above and below then stay in one L2.
__device__ __forceinline__ int xcd_block(int bid, int nb)
{
    constexpr int kXcd = 8;
    const int q = nb / kXcd, rem = nb % kXcd;
    const int k = bid % kXcd, slot = bid / kXcd;
    return k * q + (k < rem ? k : rem) + slot;
}

// Post-collision values of cell c in place (FP64 arithmetic): the deviation
// form of Eqs. explicit-u-in-Guo, final-ueq-of-S-C, feq, f-evolution-of-S-C.
// The Guo form (Sec. 2.1) taken literally, for the cost comparison of the two
// forms: u from Eq. explicit-u-in-Guo (one division), the drag force f_m of
// Eq. f_m-depends-on-u, f_eq at u (Eq. feq), the forcing term F_a of Eq.
// Fi-of-Guo and the update of Eq. f-evolution-of-Guo. coef holds eps nu / kappa.
template <typename R, bool FF, class CM, class FM>
__device__ __forceinline__ void collide_guo(const StepArgs<R> &a, double f[9], int c, int cf,
                                            const CM &cm, const FM &fm)
{
    double dr, jx, jy;
    moments(f, dr, jx, jy);
    const double rho = a.rho0_d + dr;
    double hgx, hgy;  // eps G / 2
    if (FF) {
        hgx = (double)fm.ld(0, cf);
        hgy = (double)fm.ld(1, cf);
    } else {
        hgx = a.hegx_d;
        hgy = a.hegy_d;
    }
    {
        // every fused multiply-add written out and no other contraction, so
        // that all kernels round alike
#pragma clang fp contract(off)
        const double cnu = (double)cm.ld(0, c);
        const double den = rho * __builtin_fma(0.5, cnu, 1.0);
        const double ux = __builtin_fma(hgx, rho, jx) / den, uy = __builtin_fma(hgy, rho, jy) / den;
        // rho f_m = rho (eps G - (eps nu / kappa) u)
        const double tx = __builtin_fma(-cnu, ux, 2.0 * hgx), ty = __builtin_fma(-cnu, uy, 2.0 * hgy);
        const double fmx = rho * tx, fmy = rho * ty;
        const double om = a.om_d;
        const double kf = 3.0 * __builtin_fma(-0.5, om, 1.0);  // (1 - 1/(2 tau)) / c_s^2
        const double r3 = 3.0 * rho;
        // deviations: f~eq_a = w_a (dr + 3 rho e_a . u), F_a = w_a kf e_a . rho f_m
        const double w0 = 4.0 / 9.0, w1 = 1.0 / 9.0, w5 = 1.0 / 36.0;
        const double k1 = w1 * kf, k5 = w5 * kf;
        const double px = __builtin_fma(r3, ux, dr), mx = __builtin_fma(-r3, ux, dr);
        const double py = __builtin_fma(r3, uy, dr), my = __builtin_fma(-r3, uy, dr);
        auto relax = [&](double fa, double w, double e) { return __builtin_fma(om, __builtin_fma(w, e, -fa), fa); };
        f[0] = relax(f[0], w0, dr);
        f[1] = __builtin_fma(k1, fmx, relax(f[1], w1, px));
        f[2] = __builtin_fma(k1, fmy, relax(f[2], w1, py));
        f[3] = __builtin_fma(-k1, fmx, relax(f[3], w1, mx));
        f[4] = __builtin_fma(-k1, fmy, relax(f[4], w1, my));
        const double s5 = __builtin_fma(rho, tx, fmy);
        f[5] = __builtin_fma(k5, s5, relax(f[5], w5, __builtin_fma(r3, uy, px)));
        f[6] = __builtin_fma(k5, __builtin_fma(-rho, tx, fmy), relax(f[6], w5, __builtin_fma(r3, uy, mx)));
        f[7] = __builtin_fma(-k5, s5, relax(f[7], w5, __builtin_fma(-r3, uy, mx)));
        f[8] = __builtin_fma(k5, __builtin_fma(rho, tx, -fmy), relax(f[8], w5, __builtin_fma(-r3, uy, px)));
    }
}

// Coefficient sources besides the plane accessors: one value already in a
// register, or an array in LDS indexed like the tile buffer.
template <typename R>
struct OneCoef {
    R v;
    __device__ R ld(int, int) const { return v; }
};
template <typename R>
struct LdsCoef {
    const R *p;
    __device__ R ld(int, int i) const { return p[i]; }
};

// PK: 1 scalar drag deficit E = 1 - D, 4 tensor I - M (Shan-Chen form); 0 the Guo
// form with coef = eps nu / kappa. Coefficients come from cm at index c, the
// per-cell force from fm at index cf.
// E2 (FP32 arithmetic, scalar drag): cm gives 2E, so the exact factor 2 of
// om rho u_eq is folded into the coefficient (2 fma(-E, h, g) = fma(-2E, h,
// 2g) exactly). GY false: no drive along y (hegy = 0), so hy = jy and the
// y terms of g vanish; om rho u_eq is bit for bit the same either way.
template <typename R, int PK, bool FF, bool E2 = false, bool GY = true, class CM, class FM, typename A>
__device__ __forceinline__ void collide_m(const StepArgs<R> &a, A f[9], int c, int cf, const CM &cm,
                                          const FM &fm)
{
    if constexpr (PK == 0) {
        static_assert(sizeof(A) == 8, "the Guo form runs in FP64 arithmetic");
        collide_guo<R, FF>(a, f, c, cf, cm, fm);
        return;
    } else {
    const Kc<A, R> k(a);
    A dr, jx, jy;
    moments(f, dr, jx, jy);
    const A rho = k.rho0 + dr;
    A gx, gy;  // eps rho G / 2
    if (FF) {
        gx = (A)fm.ld(0, cf) * rho;
        gy = (A)fm.ld(1, cf) * rho;
    } else {
        gx = k.hegx * rho;
        gy = k.hegy * rho;
    }
    const A hx = jx + gx, hy = jy + gy;
    const A om = k.om, omc = k.omc;
    if constexpr (sizeof(A) == 8) {
        // rho u_eq = 2 tau M h + (1 - 2 tau) j with M = I - E, formed exactly
        // enough in FP64, then the weights
        A mx, my;
        if (PK == 1) {
            const A tD = k.twotau - k.twotau * (A)cm.ld(0, c);
            mx = tD * hx + k.omtt * jx;
            my = tD * hy + k.omtt * jy;
        } else {
            const A e00 = cm.ld(0, c), e01 = cm.ld(1, c);
            const A e10 = cm.ld(2, c), e11 = cm.ld(3, c);
            mx = k.twotau * ((hx - e00 * hx) - e01 * hy) + k.omtt * jx;
            my = k.twotau * ((hy - e11 * hy) - e10 * hx) + k.omtt * jy;
        }
        // equilibrium terms: w_a om dr and 3 w_a e_a . om rho u_eq
        const A s0 = (A)(4.0 / 9.0) * om * dr;
        const A b = (A)(1.0 / 9.0) * om * dr;
        const A bx = (A)(1.0 / 3.0) * om * mx;
        const A by = (A)(1.0 / 3.0) * om * my;
        const A cc = (A)(1.0 / 36.0) * om * dr;
        const A cx = (A)(1.0 / 12.0) * om * mx;
        const A cy = (A)(1.0 / 12.0) * om * my;
        const A pp = cx + cy, qq = cx - cy;
        f[0] = omc * f[0] + s0;
        f[1] = omc * f[1] + (b + bx);
        f[2] = omc * f[2] + (b + by);
        f[3] = omc * f[3] + (b - bx);
        f[4] = omc * f[4] + (b - by);
        f[5] = omc * f[5] + (cc + pp);
        f[6] = omc * f[6] + (cc - qq);
        f[7] = omc * f[7] + (cc - pp);
        f[8] = omc * f[8] + (cc + qq);
    } else {
        // FP32: every rounded constant that multiplies a conserved or slowly
        // relaxing quantity would bias it by a fixed fraction each step, which
        // the slow modes of the flow accumulate (measured 6.5e-5 of the
        // velocity after 20 000 steps at tau 0.8). So:
        //  * om rho u_eq = om j + 2 (eps rho G / 2 - E h): (1/tau) (2 tau) is
        //    the exact 2, not a product of two rounded constants;
        //  * the rest weight and the diagonal momentum weight are remainders,
        //    so the nine terms sum to om dr and om rho u_eq up to unbiased
        //    rounding (the subtraction in cx is exact by Sterbenz's lemma);
        //  * omc = 1 - om exactly (set on the host);
        //  * every fused multiply-add written out and no other contraction,
        //    so all kernels that inline this (interior and edge paths, one and
        //    several steps per launch) round alike.
#pragma clang fp contract(off)
        // h = j + eps rho G / 2 with one rounding (g x rho fused into the sum)
        const A gcx = FF ? (A)fm.ld(0, cf) : k.hegx, gcy = FF ? (A)fm.ld(1, cf) : k.hegy;
        const A hxf = __builtin_fmaf(gcx, rho, jx), hyf = __builtin_fmaf(gcy, rho, jy);
        A tx, ty;  // 2 (eps rho G / 2 - E h)
        if constexpr (PK == 1 && E2) {
            static_assert(!FF, "the doubled coefficient is for a uniform drive");
            const A e2 = (A)cm.ld(0, c);  // 2E
            tx = __builtin_fmaf(-e2, hxf, k.hegx2 * rho);
            ty = GY ? __builtin_fmaf(-e2, hyf, k.hegy2 * rho) : -e2 * jy;
        } else if constexpr (PK == 1) {
            const A e = (A)cm.ld(0, c);
            tx = (A)2 * __builtin_fmaf(-e, hxf, gcx * rho);
            ty = (A)2 * __builtin_fmaf(-e, hyf, gcy * rho);
        } else {
            const A e00 = cm.ld(0, c), e01 = cm.ld(1, c);
            const A e10 = cm.ld(2, c), e11 = cm.ld(3, c);
            tx = (A)2 * (gcx * rho - __builtin_fmaf(e00, hxf, e01 * hyf));
            ty = (A)2 * (gcy * rho - __builtin_fmaf(e10, hxf, e11 * hyf));
        }
        const A Mx = __builtin_fmaf(om, jx, tx), My = __builtin_fmaf(om, jy, ty);
        const A D = om * dr;
        const A b = D * (A)(1.0 / 9.0);
        const A cc = D * (A)(1.0 / 36.0);
        const A s0 = __builtin_fmaf((A)-4, b + cc, D);
        // momentum: 2 t3 M on the axes and 4 c12 M on the diagonals, with t3
        // = fl(1/3) and c12 = (1 - 2 t3) / 4 exact in FP32: they sum to M
        // exactly, each term rounded once
        constexpr A t3 = (A)1 / (A)3, c12 = ((A)1 - (A)2 * t3) * (A)0.25;
        const A cx = Mx * c12, cy = My * c12;
        const A pp = cx + cy, qq = cx - cy;
        f[0] = __builtin_fmaf(omc, f[0], s0);
        f[1] = __builtin_fmaf(omc, f[1], __builtin_fmaf(Mx, t3, b));
        f[2] = __builtin_fmaf(omc, f[2], __builtin_fmaf(My, t3, b));
        f[3] = __builtin_fmaf(omc, f[3], __builtin_fmaf(-Mx, t3, b));
        f[4] = __builtin_fmaf(omc, f[4], __builtin_fmaf(-My, t3, b));
        f[5] = __builtin_fmaf(omc, f[5], cc + pp);
        f[6] = __builtin_fmaf(omc, f[6], cc - qq);
        f[7] = __builtin_fmaf(omc, f[7], cc - pp);
        f[8] = __builtin_fmaf(omc, f[8], cc + qq);
    }
    }
}

// Collision of lattice cell c with coefficients and force read through plane
// accessors of type M.
template <typename R, int PK, bool FF, class M = GMem<R>, typename A>
__device__ __forceinline__ void collide_cell(const StepArgs<R> &a, A f[9], int c)
{
    const M cm{a.coef, nullptr, a.cstride}, fm{a.hforce, nullptr, a.cstride};
    collide_m<R, PK, FF>(a, f, c, c, cm, fm);
}

// One time step per launch: pull, collide, store (one HBM pass).
template <typename R, bool WALLS, int PK, bool FF, typename A = double>
__global__ __launch_bounds__(kBlock) void k_step(StepArgs<R> a)
{
    const int bid = xcd_block(blockIdx.x, gridDim.x);
    const int nbx = (a.nx + kBlock - 1) / kBlock;
    const int y = bid / nbx;
    const int x = (bid - y * nbx) * kBlock + threadIdx.x;
    if (x >= a.nx) return;
    R fr[9];
    pull<R, WALLS>(a.fin, a.stride, a.nx, a.ny, x, y, fr);
    const int c = y * a.nx + x;
    // The arithmetic runs in FP64 whatever the storage type (LBM_F32_SHIFTED,
    // LBM_F64), or in FP32 with FP32 storage (LBM_F32_FAST).
    A f[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = (A)fr[i];
    collide_cell<R, PK, FF>(a, f, c);
    R *o = a.fout;
    const size_t S = (size_t)a.stride;
#pragma unroll
    for (int q = 0; q < 9; ++q) o[q * S + c] = (R)f[q];
}

// Several time steps per launch (temporal blocking). A workgroup owns a tile of
// output cells and takes step t on the tile plus a (D - 1)-cell halo, pulling
// from HBM; steps t + 1 .. t + D - 2 run on regions that shrink by one cell per
// step, on chip; step t + D - 1 runs on the tile and writes to HBM. Every
// value is rounded to the storage type exactly where a store to HBM would
// round it, so the result is bit-identical to D one-step launches, while HBM
// sees one read and one write of the state per D steps (plus the halo, which
// neighbouring tiles mostly find in L2).
//
// Each thread owns the same cells in every step: their rest populations and
// coefficients (drag, and the force per cell) stay in its registers, read once
// per launch. The eight moving populations live in LDS, one plane each,
// streamed in place: after a step that leaves each cell's own post-collision
// values in its own slots, the next step reads f_a from (a, x - e_a) and
// writes f*_opp(a) to that same slot, and the step after reads its own slots
// reversed and writes them in order again. A step's reads and writes touch the
// same slots and no cell shares one, so a step needs one barrier and one copy
// of the state. A cell reads its neighbours' slots only if it lies at least one
// cell inside the halo tile, so every slot lies in its plane. (The kernel before
// this one copied the state through registers between two barriers, recomputed
// its cells' coordinates in every step and, with a force or a tensor, read the
// coefficients from L2 in every step.)
template <typename R>
struct RegCoef {
    R v[4];
    __device__ R ld(int q, int) const { return v[q]; }
};
__device__ constexpr int kOpp[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};

// Any tile tx x ty whose halo tile fits BS x KM cells, any depth D >= 2. AXC: the
// halo tile's row length at compile time, or 0. Used where the grid is small
// (one tile per CU, see plan_launches) and for FP64 state.
template <typename R, bool WALLS, int PK, bool FF, int BS, int KM, int AXC, typename A>
__global__ __launch_bounds__(BS) void k_tile(StepArgs<R> a, int D, int tx, int ty)
{
    constexpr int CAP = BS * KM;
    __shared__ R S[8 * CAP];
    const int nx = a.nx, ny = a.ny;
    const int H = D - 1, AX = AXC ? AXC : tx + 2 * H;
    const int ntx = (nx + tx - 1) / tx;
    const int bid = xcd_block(blockIdx.x, gridDim.x);
    const int x0 = (bid % ntx) * tx, y0 = (bid / ntx) * ty;
    const int w1 = min(tx, nx - x0) + 2 * H, h1 = min(ty, ny - y0) + 2 * H;  // ragged tiles at the far edges
    const BMem<R> mem{a.fin, a.fout, a.stride};
    // every cell the launch touches lies inside the grid, away from the walls
    const bool interior = x0 >= H + 1 && x0 + w1 - H <= nx - 1 && y0 >= H + 1 && y0 + h1 - H <= ny - 1;
    auto body = [&](auto interior_tag) {
        constexpr bool EDGE = !decltype(interior_tag)::value;
        constexpr bool WB = WALLS && EDGE;
        int depth[KM];  // the last step (0-based) this cell takes part in; < 0: none
        int cell[KM];
        bool lo[KM], hi[KM];  // against the lower, upper wall
        R f0[KM];
        RegCoef<R> cf[KM], fc[KM];
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            const int i = threadIdx.x + k * BS;
            const int px = i % AX, py = i / AX;
            int x = x0 - H + px, y = y0 - H + py;
            bool in = px < w1 && py < h1;
            if (EDGE) {
                x %= nx;
                x = x < 0 ? x + nx : x;
                if (WALLS) {
                    in = in && y >= 0 && y < ny;
                } else {
                    y %= ny;
                    y = y < 0 ? y + ny : y;
                }
            }
            depth[k] = in ? min(min(px, w1 - 1 - px), min(py, h1 - 1 - py)) : -1;
            lo[k] = WB && y == 0;
            hi[k] = WB && y == ny - 1;
            const int c = y * nx + x;
            cell[k] = c;
            if (in) {
                R fr[9];
                if constexpr (EDGE) {
                    pullm<R, WALLS>(mem, nx, ny, x, y, fr);
                } else {
                    fr[0] = mem.ld(0, c);
                    fr[1] = mem.ld(1, c - 1);
                    fr[3] = mem.ld(3, c + 1);
                    fr[2] = mem.ld(2, c - nx);
                    fr[5] = mem.ld(5, c - nx - 1);
                    fr[6] = mem.ld(6, c - nx + 1);
                    fr[4] = mem.ld(4, c + nx);
                    fr[7] = mem.ld(7, c + nx + 1);
                    fr[8] = mem.ld(8, c + nx - 1);
                }
                const BMem<R> cm{a.coef, nullptr, a.cstride}, fm{a.hforce, nullptr, a.cstride};
#pragma unroll
                for (int q = 0; q < (PK == 4 ? 4 : 1); ++q) cf[k].v[q] = cm.ld(q, c);
                if (FF) {
                    fc[k].v[0] = fm.ld(0, c);
                    fc[k].v[1] = fm.ld(1, c);
                }
                A f[9];
#pragma unroll
                for (int q = 0; q < 9; ++q) f[q] = (A)fr[q];
                collide_m<R, PK, FF>(a, f, 0, 0, cf[k], fc[k]);
                f0[k] = (R)f[0];
#pragma unroll
                for (int q = 1; q < 9; ++q) S[(q - 1) * CAP + i] = (R)f[q];
            }
        }
        // the slots a cell's neighbours (or, against a wall, the cell itself)
        // hold for it after a step in own order
        auto slots = [&](int k, int (&r)[9]) {
            const int c = threadIdx.x + k * BS;
            r[1] = 0 * CAP + c - 1;
            r[3] = 2 * CAP + c + 1;
            r[2] = lo[k] ? 3 * CAP + c : 1 * CAP + c - AX;
            r[5] = lo[k] ? 6 * CAP + c : 4 * CAP + c - AX - 1;
            r[6] = lo[k] ? 7 * CAP + c : 5 * CAP + c - AX + 1;
            r[4] = hi[k] ? 1 * CAP + c : 3 * CAP + c + AX;
            r[7] = hi[k] ? 4 * CAP + c : 6 * CAP + c + AX + 1;
            r[8] = hi[k] ? 5 * CAP + c : 7 * CAP + c + AX - 1;
        };
        for (int s = 1; s < H; ++s) {
            __syncthreads();
            if (s & 1) {
#pragma unroll
                for (int k = 0; k < KM; ++k)
                    if (depth[k] >= s) {
                        A f[9];
                        int r[9];
                        slots(k, r);
                        f[0] = (A)f0[k];
#pragma unroll
                        for (int q = 1; q < 9; ++q) f[q] = (A)S[r[q]];
                        collide_m<R, PK, FF>(a, f, 0, 0, cf[k], fc[k]);
#pragma unroll
                        for (int q = 1; q < 9; ++q) S[r[q]] = (R)f[kOpp[q]];
                        f0[k] = (R)f[0];
                    }
            } else {
#pragma unroll
                for (int k = 0; k < KM; ++k)
                    if (depth[k] >= s) {
                        A f[9];
                        const int c = threadIdx.x + k * BS;
                        f[0] = (A)f0[k];
#pragma unroll
                        for (int q = 1; q < 9; ++q) f[q] = (A)S[(kOpp[q] - 1) * CAP + c];
                        collide_m<R, PK, FF>(a, f, 0, 0, cf[k], fc[k]);
#pragma unroll
                        for (int q = 1; q < 9; ++q) S[(q - 1) * CAP + c] = (R)f[q];
                        f0[k] = (R)f[0];
                    }
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KM; ++k)
            if (depth[k] >= H) {
                A f[9];
                f[0] = (A)f0[k];
                if (H & 1) {
                    int r[9];
                    slots(k, r);
#pragma unroll
                    for (int q = 1; q < 9; ++q) f[q] = (A)S[r[q]];
                } else {
#pragma unroll
                    for (int q = 1; q < 9; ++q) f[q] = (A)S[(kOpp[q] - 1) * CAP + threadIdx.x + k * BS];
                }
                collide_m<R, PK, FF>(a, f, 0, 0, cf[k], fc[k]);
#pragma unroll
                for (int q = 0; q < 9; ++q) mem.st(q, cell[k], (R)f[q]);
            }
    };
    if (AXC != 0 && interior)
        body(std::true_type{});
    else
        body(std::false_type{});
}

// The same with halo tiles of 64 x (BS KM / 64) cells, a wave holding whole
// rows: which rows take part in a step, and the walls, are then uniform over
// the wave (scalar branches), all LDS offsets are compile-time constants, and
// a step skips the rows it no longer needs without idle lanes. For large grids
// with FP32 state; two workgroups of 768 threads fill a CU (73.7 KB of LDS
// each). WPE: waves per SIMD the registers must allow.
template <bool WALLS, int PK, bool FF, int BS, int KM, int WPE, typename A, bool GY>
__global__ __launch_bounds__(BS, WPE) void k_rows(StepArgs<float> a, int D)
{
    using R = float;
    constexpr int CAP = BS * KM, NWV = BS / 64, AX = 64, AY = CAP / 64;
    // FP32 arithmetic keeps 2E (the exact factor 2 of the collision)
    constexpr bool E2 = PK == 1 && !FF && sizeof(A) == 4;
    static_assert(GY || E2, "the variant without a y drive is the FP32 scalar one");
    __shared__ R lds[8 * CAP];
    const int H = D - 1, tx = AX - 2 * H, ty = AY - 2 * H;
    const int nx = a.nx, ny = a.ny;
    const int ntx = (nx + tx - 1) / tx;
    const int bid = xcd_block(blockIdx.x, gridDim.x);
    const int tr = bid / ntx;
    const int x0 = (bid - tr * ntx) * tx, y0 = tr * ty;
    const int w1 = min(tx, nx - x0) + 2 * H, h1 = min(ty, ny - y0) + 2 * H;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    R *S = lds + threadIdx.x;
    const int dcol = min(lane, w1 - 1 - lane);
    const bool interior = x0 >= H + 1 && x0 + w1 - H <= nx - 1 && y0 >= H + 1 && y0 + h1 - H <= ny - 1;
    auto body = [&](auto interior_tag) {
        constexpr bool EDGE = !decltype(interior_tag)::value;
        constexpr bool WB = WALLS && EDGE;
        R f0[KM];
        RegCoef<R> cf[KM], fc[KM];
        auto row_y = [&](int k) { return y0 - H + wv + k * NWV; };
        auto row_depth = [&](int k) {  // the last step row k of this wave takes part in; < 0: none
            const int py = wv + k * NWV;
            const int d = min(py, h1 - 1 - py);
            return WB && (row_y(k) < 0 || row_y(k) >= ny) ? -1 : d;
        };
        if (dcol >= 0) {
            int x = x0 - H + lane;
            if (EDGE) {
                x %= nx;
                x = x < 0 ? x + nx : x;
            }
            const int xm = EDGE && x == 0 ? nx - 1 : x - 1, xp = EDGE && x == nx - 1 ? 0 : x + 1;
            // one buffer resource per row: its base in scalar registers, a lane's offset its x
            auto ld = [&](const R *p, int stride, int q, int row, int xx) -> R {
                const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
                    (void *)(p + (size_t)q * stride + (size_t)row * nx), 0, nx * (int)sizeof(R), BMem<R>::kFlags);
                return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(r, xx * 4, 0, 0));
            };
#pragma unroll
            for (int k = 0; k < KM; ++k) {
                if (row_depth(k) < 0) continue;
                int y = row_y(k);
                if (EDGE && !WALLS) {
                    y %= ny;
                    y = y < 0 ? y + ny : y;
                }
                const bool lo = WB && y == 0, hi = WB && y == ny - 1;
                const int ym = EDGE && y == 0 ? ny - 1 : y - 1, yp = EDGE && y == ny - 1 ? 0 : y + 1;
                R fr[9];
                fr[0] = ld(a.fin, a.stride, 0, y, x);
                fr[1] = ld(a.fin, a.stride, 1, y, xm);
                fr[3] = ld(a.fin, a.stride, 3, y, xp);
                fr[2] = lo ? ld(a.fin, a.stride, 4, y, x) : ld(a.fin, a.stride, 2, ym, x);
                fr[5] = lo ? ld(a.fin, a.stride, 7, y, x) : ld(a.fin, a.stride, 5, ym, xm);
                fr[6] = lo ? ld(a.fin, a.stride, 8, y, x) : ld(a.fin, a.stride, 6, ym, xp);
                fr[4] = hi ? ld(a.fin, a.stride, 2, y, x) : ld(a.fin, a.stride, 4, yp, x);
                fr[7] = hi ? ld(a.fin, a.stride, 5, y, x) : ld(a.fin, a.stride, 7, yp, xp);
                fr[8] = hi ? ld(a.fin, a.stride, 6, y, x) : ld(a.fin, a.stride, 8, yp, xm);
#pragma unroll
                for (int q = 0; q < (PK == 4 ? 4 : 1); ++q) cf[k].v[q] = ld(a.coef, a.cstride, q, y, x);
                if (E2) cf[k].v[0] += cf[k].v[0];
                if (FF) {
                    fc[k].v[0] = ld(a.hforce, a.cstride, 0, y, x);
                    fc[k].v[1] = ld(a.hforce, a.cstride, 1, y, x);
                }
                A f[9];
#pragma unroll
                for (int q = 0; q < 9; ++q) f[q] = (A)fr[q];
                collide_m<R, PK, FF, E2, GY>(a, f, 0, 0, cf[k], fc[k]);
                f0[k] = (R)f[0];
#pragma unroll
                for (int q = 1; q < 9; ++q) S[(q - 1) * CAP + k * BS] = (R)f[q];
            }
        }
        auto neighbour_step = [&](int k, A (&f)[9], auto store) {
            R *P = S + k * BS;
            const bool lo = WB && row_y(k) == 0, hi = WB && row_y(k) == ny - 1;
            f[0] = (A)f0[k];
            f[1] = (A)P[0 * CAP - 1];
            f[3] = (A)P[2 * CAP + 1];
            if (WB && lo) {
                f[2] = (A)P[3 * CAP];
                f[5] = (A)P[6 * CAP];
                f[6] = (A)P[7 * CAP];
            } else {
                f[2] = (A)P[1 * CAP - AX];
                f[5] = (A)P[4 * CAP - AX - 1];
                f[6] = (A)P[5 * CAP - AX + 1];
            }
            if (WB && hi) {
                f[4] = (A)P[1 * CAP];
                f[7] = (A)P[4 * CAP];
                f[8] = (A)P[5 * CAP];
            } else {
                f[4] = (A)P[3 * CAP + AX];
                f[7] = (A)P[6 * CAP + AX + 1];
                f[8] = (A)P[7 * CAP + AX - 1];
            }
            collide_m<R, PK, FF, E2, GY>(a, f, 0, 0, cf[k], fc[k]);
            if constexpr (decltype(store)::value) {
                P[0 * CAP - 1] = (R)f[3];
                P[2 * CAP + 1] = (R)f[1];
                if (WB && lo) {
                    P[3 * CAP] = (R)f[4];
                    P[6 * CAP] = (R)f[7];
                    P[7 * CAP] = (R)f[8];
                } else {
                    P[1 * CAP - AX] = (R)f[4];
                    P[4 * CAP - AX - 1] = (R)f[7];
                    P[5 * CAP - AX + 1] = (R)f[8];
                }
                if (WB && hi) {
                    P[1 * CAP] = (R)f[2];
                    P[4 * CAP] = (R)f[5];
                    P[5 * CAP] = (R)f[6];
                } else {
                    P[3 * CAP + AX] = (R)f[2];
                    P[6 * CAP + AX + 1] = (R)f[5];
                    P[7 * CAP + AX - 1] = (R)f[6];
                }
                f0[k] = (R)f[0];
            }
        };
        auto own_step = [&](int k, A (&f)[9], auto store) {
            R *P = S + k * BS;
            f[0] = (A)f0[k];
#pragma unroll
            for (int q = 1; q < 9; ++q) f[q] = (A)P[(kOpp[q] - 1) * CAP];
            collide_m<R, PK, FF, E2, GY>(a, f, 0, 0, cf[k], fc[k]);
            if constexpr (decltype(store)::value) {
#pragma unroll
                for (int q = 1; q < 9; ++q) P[(q - 1) * CAP] = (R)f[q];
                f0[k] = (R)f[0];
            }
        };
        for (int s = 1; s < H; ++s) {
            __syncthreads();
            if (dcol >= s) {
                if (s & 1) {
#pragma unroll
                    for (int k = 0; k < KM; ++k)
                        if (row_depth(k) >= s) {
                            A f[9];
                            neighbour_step(k, f, std::true_type{});
                        }
                } else {
#pragma unroll
                    for (int k = 0; k < KM; ++k)
                        if (row_depth(k) >= s) {
                            A f[9];
                            own_step(k, f, std::true_type{});
                        }
                }
            }
        }
        __syncthreads();
        if (dcol >= H) {
#pragma unroll
            for (int k = 0; k < KM; ++k)
                if (row_depth(k) >= H) {
                    A f[9];
                    if (H & 1)
                        neighbour_step(k, f, std::false_type{});
                    else
                        own_step(k, f, std::false_type{});
                    const BMem<R> row{nullptr, a.fout + (size_t)row_y(k) * nx, a.stride};
#pragma unroll
                    for (int q = 0; q < 9; ++q) row.st(q, x0 - H + lane, (R)f[q]);
                }
        }
    };
    if (interior)
        body(std::true_type{});
    else
        body(std::false_type{});
}

// Flow velocity (Eq. u-of-S-C) and density of the current state in FP64, and
// per-block FP64 partial sums of u for the volume average.
template <typename R, bool WALLS, int PK, bool FF>
__global__ __launch_bounds__(kBlock) void k_fields(StepArgs<R> a, double *__restrict__ u_out,
                                                   double *__restrict__ rho_out,
                                                   double *__restrict__ partials)
{
    __shared__ double red[2][kBlock / 64];
    const int x = blockIdx.x * kBlock + threadIdx.x;
    const int y = blockIdx.y;
    double ux = 0.0, uy = 0.0;
    if (x < a.nx) {
        R fr[9];
        pull<R, WALLS>(a.fin, a.stride, a.nx, a.ny, x, y, fr);
        double f[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = (double)fr[i];
        double dr, jx, jy;
        moments(f, dr, jx, jy);
        const double rho = a.rho0_d + dr;
        const int c = y * a.nx + x;
        double hx, hy;
        if (FF) {
            hx = jx + (double)a.hforce[c] * rho;
            hy = jy + (double)a.hforce[a.cstride + c] * rho;
        } else {
            hx = jx + a.hegx_d * rho;
            hy = jy + a.hegy_d * rho;
        }
        if (PK == 1) {
            const double D = 1.0 - (double)a.coef[c];
            ux = D * hx / rho;
            uy = D * hy / rho;
        } else if (PK == 0) {
            const double den = rho * (1.0 + 0.5 * (double)a.coef[c]);
            ux = hx / den;
            uy = hy / den;
        } else {
            const double e00 = a.coef[c], e01 = a.coef[a.cstride + c];
            const double e10 = a.coef[2 * a.cstride + c], e11 = a.coef[3 * a.cstride + c];
            ux = ((hx - e00 * hx) - e01 * hy) / rho;
            uy = ((hy - e11 * hy) - e10 * hx) / rho;
        }
        if (u_out) {
            const size_t N = (size_t)a.nx * a.ny;
            u_out[c] = ux;
            u_out[N + c] = uy;
        }
        if (rho_out) rho_out[c] = rho;
    }
    if (partials) {
        ux = wave_sum(ux);
        uy = wave_sum(uy);
        const int wv = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) {
            red[0][wv] = ux;
            red[1][wv] = uy;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double sx = 0.0, sy = 0.0;
            for (int w = 0; w < kBlock / 64; ++w) {
                sx += red[0][w];
                sy += red[1][w];
            }
            const int bid = blockIdx.y * gridDim.x + blockIdx.x;
            partials[2 * bid] = sx;
            partials[2 * bid + 1] = sy;
        }
    }
}

// Fixed-order sum of n (x, y) pairs, divided by the number of cells, into
// pinned host memory: out[0..1], then the number of the call in out[2], which
// the host may wait for. (Adding up in the last workgroup of k_fields instead
// was no faster at 64 x 64 cells and slower beyond, by 20 us at 256 x 1024 and
// 500 us at 2048 x 2048: its counter takes 30 ns per workgroup.)
__global__ __launch_bounds__(kBlock) void k_reduce_pairs(const double *__restrict__ partials,
                                                         int n, double inv_cells, unsigned long long call,
                                                         double *__restrict__ out)
{
    __shared__ double red[2][kBlock / 64];
    double sx = 0.0, sy = 0.0;
    // each thread adds its partials in index order, reading 16 of them ahead
    // (a loop that waited for each read took most of the reduction's time)
    constexpr int kAhead = 16;
    for (int i0 = threadIdx.x; i0 < n; i0 += kAhead * kBlock) {
        double vx[kAhead], vy[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = min(i0 + u * kBlock, n - 1);
            vx[u] = partials[2 * i];
            vy[u] = partials[2 * i + 1];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (i0 + u * kBlock < n) {
                sx += vx[u];
                sy += vy[u];
            }
    }
    sx = wave_sum(sx);
    sy = wave_sum(sy);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wv] = sx;
        red[1][wv] = sy;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double tx = 0.0, ty = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) {
            tx += red[0][w];
            ty += red[1][w];
        }
        out[0] = tx * inv_cells;
        out[1] = ty * inv_cells;
        __hip_atomic_store(reinterpret_cast<unsigned long long *>(out) + 2, call, __ATOMIC_RELEASE,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__global__ void k_zero_i32(int *__restrict__ p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Per-cell coefficient from the permeability (FP64, rounded once to R),
// eps G / 2 per cell, and the rest state (zero deviations) in buffer fin.
template <typename R, int PK>
__global__ __launch_bounds__(kBlock) void k_init(const double *__restrict__ perm,
                                                 const double *__restrict__ force, int n,
                                                 double eps, double nu, R *__restrict__ coef,
                                                 R *__restrict__ hforce, int cstride,
                                                 R *__restrict__ pops, int stride,
                                                 int *__restrict__ bad)
{
    const int c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= n) return;
    const double h = 0.5 * eps * nu;
    if (PK == 1) {
        const double k = perm[c];
        if (!(k > 0.0)) atomicOr(bad, 1);  // also catches NaN
        // E = 1 - D = h / (kappa + h) with D = 1 / (1 + eps nu / (2 kappa));
        // kappa = +inf gives 0
        coef[c] = (R)(h / (k + h));
    } else if (PK == 0) {
        const double k = perm[c];
        if (!(k > 0.0)) atomicOr(bad, 1);
        coef[c] = (R)(2.0 * h / k);  // eps nu / kappa (Guo form)
    } else {
        const double kxx = perm[4 * c], kxy = perm[4 * c + 1];
        const double kyx = perm[4 * c + 2], kyy = perm[4 * c + 3];
        const double det = kxx * kyy - kxy * kyx;
        // M = (K + h I)^{-1} K
        const double axx = kxx + h, axy = kxy, ayx = kyx, ayy = kyy + h;
        const double adet = axx * ayy - axy * ayx;
        const bool ok = std::isfinite(det) && det != 0.0 && std::isfinite(adet) && adet != 0.0;
        if (!ok) atomicOr(bad, 1);
        // E = I - M = h (K + h I)^{-1}
        const double ia = h / adet;
        coef[c] = (R)(ia * ayy);
        coef[cstride + c] = (R)(-ia * axy);
        coef[2 * cstride + c] = (R)(-ia * ayx);
        coef[3 * cstride + c] = (R)(ia * axx);
    }
    if (force) {
        const double gx = force[2 * c], gy = force[2 * c + 1];
        if (!std::isfinite(gx) || !std::isfinite(gy)) atomicOr(bad, 2);
        hforce[c] = (R)(0.5 * eps * gx);
        hforce[cstride + c] = (R)(0.5 * eps * gy);
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) pops[(size_t)q * stride + c] = (R)0;
}

// Rest state (zero deviations) of n cells.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_rest(R *__restrict__ pops, int stride, int n)
{
    const int c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= n) return;
#pragma unroll
    for (int q = 0; q < 9; ++q) pops[(size_t)q * stride + c] = (R)0;
}

// Convergence of the whole velocity field (the coarse solve's test), taken on
// the device: the fields of the current state, the relative L2 change of the
// velocity since the last check (kept rounded to R), and, in the workgroup
// that finishes last (done counts them, zero before and after), the decision.
// host, pinned: [1] flag, [2] the run has ended, then [0] the steps, for which
// the host waits. A check is queued only once the last one has been read, so
// none runs after the end; the steps queued ahead of the reading do not change
// the fields.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_field_check(StepArgs<R> a, long long steps, bool first, double tol,
                                                        long long max_steps, R *__restrict__ prev,
                                                        double *__restrict__ partials, double *__restrict__ u_out,
                                                        double *__restrict__ rho_out,
                                                        unsigned long long *__restrict__ done,
                                                        long long *__restrict__ host)
{
    __shared__ double red[2][kBlock / 64];
    __shared__ bool last;
    const int N = a.nx * a.ny, c = blockIdx.x * kBlock + threadIdx.x;
    double d2 = 0.0, u2 = 0.0;
    if (c < N) {
        R fr[9];
        pull<R, false>(a.fin, a.stride, a.nx, a.ny, c % a.nx, c / a.nx, fr);
        double f[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = (double)fr[i];
        double dr, jx, jy;
        moments(f, dr, jx, jy);
        const double rho = a.rho0_d + dr;
        const double hx = jx + (double)a.hforce[c] * rho, hy = jy + (double)a.hforce[a.cstride + c] * rho;
        const double e00 = a.coef[c], e01 = a.coef[a.cstride + c];
        const double e10 = a.coef[2 * a.cstride + c], e11 = a.coef[3 * a.cstride + c];
        const double ux = ((hx - e00 * hx) - e01 * hy) / rho, uy = ((hy - e11 * hy) - e10 * hx) / rho;
        const R rx = (R)ux, ry = (R)uy;
        const double dx = first ? 0.0 : (double)rx - (double)prev[c], dy = first ? 0.0 : (double)ry - (double)prev[N + c];
        d2 = dx * dx + dy * dy;
        u2 = ux * ux + uy * uy;
        prev[c] = rx;
        prev[N + c] = ry;
        u_out[c] = ux;
        u_out[N + c] = uy;
        if (rho_out) rho_out[c] = rho;
    }
    d2 = wave_sum(d2);
    u2 = wave_sum(u2);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = d2;
        red[1][threadIdx.x >> 6] = u2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double sd = 0.0, su = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) {
            sd += red[0][w];
            su += red[1][w];
        }
        // device-wide visible before the count says so
        __hip_atomic_store(&partials[2 * blockIdx.x], sd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&partials[2 * blockIdx.x + 1], su, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = __hip_atomic_fetch_add(done, 1ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    }
    __syncthreads();
    if (!last || threadIdx.x >= 64) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    // added in order, but read all at once (one read after the other: 7.8 us per check of 64 x 64 cells, now 6.3)
    double td = 0.0, tu = 0.0;
    for (unsigned b0 = 0; b0 < gridDim.x; b0 += 64) {
        const unsigned m = min(64u, gridDim.x - b0);
        double d = 0.0, u = 0.0;
        if (threadIdx.x < m) {
            d = __hip_atomic_load(&partials[2 * (b0 + threadIdx.x)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            u = __hip_atomic_load(&partials[2 * (b0 + threadIdx.x) + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        for (unsigned b = 0; b < m; ++b) {
            td += __shfl(d, b);
            tu += __shfl(u, b);
        }
    }
    if (threadIdx.x != 0) return;
    long long flag = -1;
    if (!isfinite(td) || !isfinite(tu)) flag = 2;
    else if (!first && tol > 0.0 && sqrt(td) <= tol * sqrt(tu)) flag = 0;
    else if (steps >= max_steps) flag = tol > 0.0 ? 1 : 0;
    *done = 0;
    host[1] = flag;
    host[2] = flag >= 0;
    __hip_atomic_store(&host[0], steps, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Full pre-collision populations of the current state, FP64 [9][ny][nx].
template <typename R, bool WALLS>
__global__ __launch_bounds__(kBlock) void k_get_pops(const R *__restrict__ fin, int stride, int nx,
                                                     int ny, double rho0, double *__restrict__ out)
{
    const int x = blockIdx.x * kBlock + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= nx) return;
    R f[9];
    pull<R, WALLS>(fin, stride, nx, ny, x, y, f);
    const size_t N = (size_t)nx * ny;
    const int c = y * nx + x;
#pragma unroll
    for (int q = 0; q < 9; ++q) out[q * N + c] = (double)f[q] + weight(q) * rho0;
}

// Inverse of the pull: store g with pull(g) = f, i.e. g_b(x) = f_b(x + e_b),
// or f_opp(b)(x) when x + e_b lies beyond a wall.
template <typename R, bool WALLS>
__global__ __launch_bounds__(kBlock) void k_set_pops(const double *__restrict__ in, int nx, int ny,
                                                     double rho0, R *__restrict__ fout, int stride)
{
    const int x = blockIdx.x * kBlock + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= nx) return;
    const size_t N = (size_t)nx * ny;
    const int c = y * nx + x;
#pragma unroll
    for (int b = 0; b < 9; ++b) {
        int xs = x + ex(b);
        int ys = y + ey(b);
        xs = (xs < 0) ? nx - 1 : (xs >= nx ? 0 : xs);
        int src_pop = b;
        if (ys < 0 || ys >= ny) {
            if (WALLS) {
                xs = x;
                ys = y;
                src_pop = opposite(b);
            } else {
                ys = (ys < 0) ? ny - 1 : 0;
            }
        }
        const double v = in[src_pop * N + (size_t)ys * nx + xs] - weight(src_pop) * rho0;
        fout[(size_t)b * stride + c] = (R)v;
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

struct Layout {
    size_t elem;      // bytes per population element
    size_t stride;    // elements per population plane
    size_t cstride;   // elements per coefficient plane
    size_t off_a, off_b, off_coef, off_force, off_part, off_flag, total;
    int nbx, nby;     // launch grid of the per-cell kernels
};

bool params_ok(const lbm_params *p, std::string &why)
{
    if (!p) { why = "params is NULL"; return false; }
    if (p->nx < 1 || p->ny < 1) { why = "nx and ny must be >= 1"; return false; }
    if (9 * ((int64_t)p->nx * p->ny + 8192) >= (int64_t)1 << 31) { why = "grid too large (9 nx ny must be below 2^31 - 73728)"; return false; }
    if (!(p->tau >= 0.5) || !std::isfinite(p->tau)) { why = "tau must be finite and >= 0.5"; return false; }
    if (!(p->eps > 0.0 && p->eps <= 1.0)) { why = "eps must lie in (0, 1]"; return false; }
    if (!(p->nu > 0.0) || !std::isfinite(p->nu)) { why = "nu must be finite and > 0"; return false; }
    if (!(p->rho0 > 0.0) || !std::isfinite(p->rho0)) { why = "rho0 must be finite and > 0"; return false; }
    if (!std::isfinite(p->gx) || !std::isfinite(p->gy)) { why = "gx, gy must be finite"; return false; }
    if (p->walls_y != 0 && p->walls_y != 1) { why = "walls_y must be 0 or 1"; return false; }
    if (p->pop_dtype != LBM_F32_SHIFTED && p->pop_dtype != LBM_F64 && p->pop_dtype != LBM_F32_FAST) {
        why = "unknown pop_dtype";
        return false;
    }
    if (p->pop_dtype == LBM_F32_FAST && p->scheme == LBM_SCHEME_GUO) {
        why = "the Guo form runs with FP64 arithmetic only (pop_dtype LBM_F32_SHIFTED or LBM_F64)";
        return false;
    }
    if (p->perm_kind != LBM_PERM_SCALAR && p->perm_kind != LBM_PERM_TENSOR) { why = "perm_kind must be 1 or 4"; return false; }
    if (p->scheme != LBM_SCHEME_SHAN_CHEN && p->scheme != LBM_SCHEME_GUO) { why = "scheme must be 0 or 1"; return false; }
    if (p->scheme == LBM_SCHEME_GUO && p->perm_kind != LBM_PERM_SCALAR) { why = "the Guo form takes a scalar permeability"; return false; }
    return true;
}

Layout layout_of(const lbm_params *p)
{
    Layout L{};
    const size_t n = (size_t)p->nx * p->ny;
    L.elem = (p->pop_dtype == LBM_F64) ? 8 : 4;
    // Planes are 16 KB apart beyond their size, so that the ten streams of a
    // step (nine planes and the coefficient) do not start on the same HBM
    // channels when the plane size is a large power of two.
    L.stride = align_up(n, 64) + kPlanePadBytes / L.elem;
    L.cstride = n;
    size_t off = 0;
    L.off_a = off;  off = align_up(off + 9 * L.stride * L.elem);
    L.off_b = off;  off = align_up(off + 9 * L.stride * L.elem);
    L.off_coef = off; off = align_up(off + (size_t)p->perm_kind * L.cstride * L.elem);
    L.off_force = off; off = align_up(off + 2 * L.cstride * L.elem);
    L.nbx = (p->nx + kBlock - 1) / kBlock;
    L.nby = p->ny;
    L.off_part = off; off = align_up(off + 2 * sizeof(double) * (size_t)L.nbx * L.nby);
    off = align_up(off + 4 * sizeof(double));  // free; the size that callers know stays
    L.off_flag = off; off = align_up(off + sizeof(int));
    L.total = off;
    return L;
}

}  // namespace
}  // namespace lbm

namespace lbm {
namespace {

// The kernels that take several steps per launch: k_tile with 512, 1024 or
// 1024 x 2 cells, with 512 x 2 cells in rows of 32 (FP64 state), k_rows with
// 768 x 3 or 1024 x 2 cells (FP32 state).
enum Shape { kTile512, kTile1024, kTile2048, kTile32, kRows768, kRows1024, kShapes };
constexpr int kMaxDepth = 12;   // steps per launch
constexpr int kPlanRoom = 64;   // longest stretch planned launch by launch

struct Launch {
    int shape, tx, ty;
    double us;  // predicted
};

struct Plan {
    Launch at[kMaxDepth + 1];              // per depth
    signed char first[kPlanRoom + 1];      // depth of the first launch over this many steps
    int longest;                           // the depth of least time per step
};

}  // namespace
}  // namespace lbm

struct lbm_handle {
    lbm_params p;
    lbm::Layout L;
    lbm::Plan plan;
    hipStream_t stream;
    char *ws;
    int cur;            // 0: state in buffer A, 1: in buffer B
    bool has_force;
    int64_t steps_total;
    double prev_u[2];
    bool have_prev;
    double *host_res;   // pinned: mean velocity, number of its call
    unsigned long long means;  // mean velocities asked for
};

namespace lbm {
namespace {

template <typename R>
StepArgs<R> step_args(const lbm_handle *h)
{
    StepArgs<R> a{};
    const Layout &L = h->L;
    a.fin = reinterpret_cast<const R *>(h->ws + (h->cur ? L.off_b : L.off_a));
    a.fout = reinterpret_cast<R *>(h->ws + (h->cur ? L.off_a : L.off_b));
    a.coef = reinterpret_cast<const R *>(h->ws + L.off_coef);
    a.hforce = h->has_force ? reinterpret_cast<const R *>(h->ws + L.off_force) : nullptr;
    a.nx = h->p.nx;
    a.ny = h->p.ny;
    a.stride = (int)L.stride;
    a.cstride = (int)L.cstride;
    const double tau = h->p.tau;
    a.om = (R)(1.0 / tau);
    // 1 - om formed in the storage type: for tau in [1/2, 2] the subtraction
    // is exact (Sterbenz), so om + omc = 1 and the FP32-arithmetic collision
    // conserves mass without a bias from the rounded 1/tau
    a.omc = (R)1 - a.om;
    a.twotau = (R)(2.0 * tau);
    a.omtt = (R)(1.0 - 2.0 * tau);
    a.hegx = (R)(0.5 * h->p.eps * h->p.gx);
    a.hegy = (R)(0.5 * h->p.eps * h->p.gy);
    a.rho0 = (R)h->p.rho0;
    a.hegx_d = 0.5 * h->p.eps * h->p.gx;
    a.hegy_d = 0.5 * h->p.eps * h->p.gy;
    a.om_d = 1.0 / tau;
    a.omc_d = 1.0 - 1.0 / tau;
    a.twotau_d = 2.0 * tau;
    a.omtt_d = 1.0 - 2.0 * tau;
    a.rho0_d = h->p.rho0;
    return a;
}

template <typename R, bool W, int PK, bool FF>
void launch_step_t(const lbm_handle *h)
{
    const dim3 grid(h->L.nbx * h->L.nby);
    if constexpr (std::is_same<R, float>::value && PK != 0) {
        if (h->p.pop_dtype == LBM_F32_FAST) {
            hipLaunchKernelGGL((k_step<R, W, PK, FF, float>), grid, dim3(kBlock), 0, h->stream, step_args<R>(h));
            return;
        }
    }
    hipLaunchKernelGGL((k_step<R, W, PK, FF>), grid, dim3(kBlock), 0, h->stream, step_args<R>(h));
}

template <typename R, bool W, int PK, bool FF>
void launch_fields_t(const lbm_handle *h, double *u, double *rho, double *part)
{
    const dim3 grid(h->L.nbx, h->L.nby);
    hipLaunchKernelGGL((k_fields<R, W, PK, FF>), grid, dim3(kBlock), 0, h->stream, step_args<R>(h),
                       u, rho, part);
}

// Dispatch on (dtype, walls, perm kind, force field) to one instantiation.
template <template <typename, bool, int, bool> class Fn, typename... Args>
void dispatch(const lbm_handle *h, Args... args)
{
    const bool w = h->p.walls_y != 0, ff = h->has_force;
    const int pk = h->p.scheme == LBM_SCHEME_GUO ? 0 : h->p.perm_kind;
#define LBM_CASE(R, W, PK, FF) \
    if (w == W && pk == PK && ff == FF) { Fn<R, W, PK, FF>::run(h, args...); return; }
    if (h->p.pop_dtype == LBM_F64) {
        LBM_CASE(double, false, 1, false) LBM_CASE(double, false, 1, true)
        LBM_CASE(double, false, 4, false) LBM_CASE(double, false, 4, true)
        LBM_CASE(double, true, 1, false)  LBM_CASE(double, true, 1, true)
        LBM_CASE(double, true, 4, false)  LBM_CASE(double, true, 4, true)
        LBM_CASE(double, false, 0, false) LBM_CASE(double, false, 0, true)
        LBM_CASE(double, true, 0, false)  LBM_CASE(double, true, 0, true)
    } else {
        LBM_CASE(float, false, 1, false) LBM_CASE(float, false, 1, true)
        LBM_CASE(float, false, 4, false) LBM_CASE(float, false, 4, true)
        LBM_CASE(float, true, 1, false)  LBM_CASE(float, true, 1, true)
        LBM_CASE(float, true, 4, false)  LBM_CASE(float, true, 4, true)
        LBM_CASE(float, false, 0, false) LBM_CASE(float, false, 0, true)
        LBM_CASE(float, true, 0, false)  LBM_CASE(float, true, 0, true)
    }
#undef LBM_CASE
}

template <typename R, bool W, int PK, bool FF>
struct StepFn {
    static void run(const lbm_handle *h) { launch_step_t<R, W, PK, FF>(h); }
};
template <typename R, bool W, int PK, bool FF>
struct StepDFn {
    template <typename A>
    static void launch(const lbm_handle *h, int D)
    {
        const Launch &l = h->plan.at[D];
        const int nt = ((h->p.nx + l.tx - 1) / l.tx) * ((h->p.ny + l.ty - 1) / l.ty);
        const StepArgs<R> sa = step_args<R>(h);
        auto tile = [&](auto kernel, int threads) {
            hipLaunchKernelGGL(kernel, dim3(nt), dim3(threads), 0, h->stream, sa, D, l.tx, l.ty);
        };
        if (l.shape == kTile512) return tile(k_tile<R, W, PK, FF, 512, 1, 0, A>, 512);
        if (l.shape == kTile1024) return tile(k_tile<R, W, PK, FF, 1024, 1, 0, A>, 1024);
        if (l.shape == kTile2048) return tile(k_tile<R, W, PK, FF, 1024, 2, 0, A>, 1024);
        if constexpr (std::is_same<R, double>::value) {
            tile(k_tile<R, W, PK, FF, 512, 2, 32, A>, 512);
        } else {
            auto rows = [&](auto kernel, int threads) {
                hipLaunchKernelGGL(kernel, dim3(nt), dim3(threads), 0, h->stream, sa, D);
            };
            if constexpr (sizeof(A) == 8) {
                // six waves per SIMD (two workgroups per CU), but for a tensor, whose four
                // coefficients per cell would spill (2048^2: 36.0 us per step against 31.2)
                rows(k_rows<W, PK, FF, 768, 3, PK == 4 ? 1 : 6, A, true>, 768);
            } else {
                if constexpr (PK == 1 && !FF) {
                    if (sa.hegy == 0.0f) {  // drive along x only
                        if (l.shape == kRows1024) return rows(k_rows<W, PK, FF, 1024, 2, 8, A, false>, 1024);
                        return rows(k_rows<W, PK, FF, 768, 3, 6, A, false>, 768);
                    }
                }
                if (l.shape == kRows1024) return rows(k_rows<W, PK, FF, 1024, 2, 8, A, true>, 1024);
                rows(k_rows<W, PK, FF, 768, 3, 6, A, true>, 768);
            }
        }
    }
    static void run(const lbm_handle *h, int D)
    {
        if constexpr (std::is_same<R, float>::value && PK != 0) {
            if (h->p.pop_dtype == LBM_F32_FAST) return launch<float>(h, D);
        }
        launch<double>(h, D);
    }
};

// Predicted time (us) of one launch of depth D on tiles tx x ty of a shape:
// a launch's own 2.7 us, the state through HBM once at 8 TB/s, and per round of
// resident tiles the D steps, each `wave` us per wavefront and SIMD in it (at
// least the 0.42 us that one step's chain of LDS reads, collision, writes and
// barrier takes). Fitted to launches of 64^2 to 2048^2 grids: 64^2 FP32 state
// D = 10 6.9 us (measured 7.0), 400^2 FP64 with a force D = 8 14.3 (14.8), 700^2
// FP32 D = 8 22.1 (22.4), 2048^2 FP64 D = 6 179 (184). Runs of 200 to 600 steps
// took 0.95 to 1.3 times their prediction over all types, coefficients and
// sizes (most where one or two rounds of tiles take the whole launch); a plan
// needs the order of its choices, not the time.
// FP32 state with a tensor in FP64 arithmetic holds 84 to 108 registers in
// k_rows, so one workgroup of 12 waves per CU (lone), whose rounds do not
// overlap. Planned as if two were resident, 600^2 took 3.35 us per step, 1000^2
// 6.70 and 3000 x 2000 39.0; now 2.73, 6.17 and 37.4 (other sizes within 2% or
// faster; over 18 grids the plan is 0.6% off the best tile and depth tried, on
// average, and was 2.5%).
// A launch that cannot take less than `limit` is not summed up (infinity).
double launch_us(const lbm_params &p, bool force, int cus, int shape, int D, int tx, int ty, double limit)
{
    const bool f64 = p.pop_dtype == LBM_F64, fast = p.pop_dtype == LBM_F32_FAST;
    const double nt = (double)((p.nx + tx - 1) / tx) * ((p.ny + ty - 1) / ty);
    const int ax = tx + 2 * (D - 1), ay = ty + 2 * (D - 1);
    const bool lone = shape == kRows768 && !fast && p.perm_kind == LBM_PERM_TENSOR;
    const bool two = (shape == kRows768 && !lone) || shape == kRows1024 || shape == kTile32;
    const double r = (two && nt > cus) ? 2.0 : 1.0;  // tiles of a CU at once
    // rounds of tiles; a last one that fills at most half of the places runs one tile per CU
    const double full = nt / (cus * r), frac = full - std::floor(full);
    const double rounds = full > (lone ? 8.0 : 4.0) ? full + 0.2
                          : std::floor(full) + (frac == 0.0 ? 0.0 : (r == 2.0 && frac <= 0.5) ? 0.6 : 1.0);
    const double wave = fast ? 0.063 : p.scheme == LBM_SCHEME_GUO ? 0.185 : f64 ? 0.127 : lone ? 0.118 : 0.112;
    double t = r == 1.0 && rounds > 1.0 ? (lone ? 1.0 : 2.0) : 0.0;  // a lone tile waits for its own reads
    const double lat = r == 1.0 || full <= 1.0 ? 0.25 : 0.12;
    const double planes = 19.0 + (force ? 2.0 : 0.0) + (p.perm_kind == LBM_PERM_TENSOR ? 3.0 : 0.0);
    const double mem = (double)p.nx * p.ny * planes * (f64 ? 8.0 : 4.0) / 8.0e6;
    const double least = D * std::max(0.42, lat + wave * r * ax * (ay - D + 1) / 256.0);  // of the sum below
    if (2.7 + rounds * (t + least) + mem > limit * (1.0 + 1e-9)) return INFINITY;
    for (int s = 0; s < D; ++s) t += std::max(0.42, lat + wave * r * ax * (ay - 2 * s) / 256.0);
    return 2.7 + rounds * t + mem;
}

// Launches of few steps on grids that fill the device are bound by the state's
// way through memory, which the model above adds to the steps' time instead of
// overlapping them. Where that misleads it their tiles come from measurements of 26
// grids from 200^2 to 4096^2, all types and coefficients (us of a launch, the
// model's choice and this one). Two steps of a state that the caches hold: tiles of
// 512 threads, several per CU, 30 x 14 for FP64 arithmetic on FP32 state, else 62 x
// 6, up to 850 000 cells (512^2 13.7 and 6.7, 700 x 500 9.1 and 7.7, with FP32
// arithmetic 8.9 and 6.3), above that where the model's rows need a second round
// for a few tiles (1024^2 17.6 and 16.0), and for a tensor, whose rows fill a CU with
// one workgroup (1024^2 24.7 and 18.5). Beyond the caches, for FP64 state, tensors
// and from 5 000 000 cells: 62 x 14 tiles of 1024 threads (2048^2 FP64 154 and 131,
// 4096^2 FP32 302 and 268). Three and four steps with a tensor: 60 x 12 and 58 x 10 of
// them (1024^2, four steps, 32.3 and 26.9).
// The time handed to the plan is the larger of both predictions, so that longer
// stretches are planned as before. us 0: the model's choice stands.
Launch few_steps(const lbm_params &p, bool force, int cus, int D)
{
    const double cells = (double)p.nx * p.ny, el = p.pop_dtype == LBM_F64 ? 8.0 : 4.0;
    const bool f32 = p.pop_dtype == LBM_F32_SHIFTED, tensor = f32 && p.perm_kind == LBM_PERM_TENSOR;
    const bool cached = 18.0 * cells * el < 240e6;
    const int rows = ((p.nx + 61) / 62) * ((p.ny + 33) / 34);  // tiles of the row kernel at two steps
    const bool sc = p.scheme == LBM_SCHEME_SHAN_CHEN;
    const bool second = f32 && sc && rows > 2 * cus && rows < 4 * cus && cells < 1.75e6;
    const bool small = D == 2 && cached && cells >= 40e3 && (cells < 850e3 || tensor || second);
    const bool large = (D == 2 && !cached && (el == 8.0 || tensor || (sc && cells > 5e6))) ||
                       (D > 2 && D <= 4 && tensor && cells >= 500e3);
    if (p.nx < 64 || p.ny < 128 || !(small || large)) return Launch{};
    const int h2 = 2 * (D - 1), w = (small && f32 ? 32 : 64) - h2;
    const int columns = (p.nx + w - 1) / w, tx = (p.nx + columns - 1) / columns;
    const int ty = (small ? 512 : 1024) / (tx + h2) - h2;
    const double bytes = cells * el * (19.0 + (force ? 2.0 : 0.0) + (p.perm_kind == LBM_PERM_TENSOR ? 3.0 : 0.0));
    return Launch{small ? kTile512 : kTile1024, tx, ty, 3.0 + bytes / (small ? 6.4e6 : 4.75e6)};
}

// Per depth, the shape and tile of least predicted time; then the sequence of
// depths that covers a stretch of up to kPlanRoom steps in the least time
// (longer stretches start with the depth of least time per step). Every depth
// and tile gives the same state bit for bit, so the plan is one of time only.
// What it comes to: small grids take tiles just large enough that all run at
// once, one per CU, ten or so steps per launch (64^2 FP32 state: 2.38 -> 0.70 us
// per step against 48 x 24 tiles on 6 CUs); large ones the 64-wide rows with FP32
// state (2048^2: FP32 arithmetic 15.0 -> 13.1, FP64 arithmetic 19.3 -> 17.6) and
// 32-wide tiles with FP64 state (38.7 -> 30.7).
Plan plan_launches(const lbm_params &p, bool force, int cus)
{
    Plan pl{};
    const bool f64 = p.pop_dtype == LBM_F64, fast = p.pop_dtype == LBM_F32_FAST;
    int even[65] = {};  // the tile width of even columns of at most w cells
    for (int w = 4; w <= 64; ++w) {
        const int columns = (p.nx + w - 1) / w;
        even[w] = (p.nx + columns - 1) / columns;
    }
    for (int D = 2; D <= kMaxDepth; ++D) {
        Launch best{kTile1024, 1, 1, 1e30};
        const int h2 = 2 * (D - 1);
        // the large grids' tile first, as a limit for the others
        double limit = 1e30;
        if (D <= 10) limit = f64 ? launch_us(p, force, cus, kTile32, D, 32 - h2, 32 - h2, limit)
                                 : launch_us(p, force, cus, kRows768, D, 64 - h2, 36 - h2, limit);
        auto offer = [&](int shape, int tx, int ty) {
            const double us = launch_us(p, force, cus, shape, D, tx, ty, std::min(limit, best.us));
            if (us < best.us) best = Launch{shape, tx, ty, us};
        };
        const int cap[3] = {512, 1024, 2048}, shape[3] = {kTile512, kTile1024, kTile2048};
        // rows of fewer than 16 cells read partial cache lines, which few steps do not
        // make up for (300^2, three steps: 6 x 75 tiles 6.3 us, 58 x 12 5.6)
        const int narrowest = D <= 5 && p.nx >= 64 && (double)p.nx * p.ny >= 40e3 ? 16 : 4;
        for (int i = 0; i < 3; ++i)
            for (int w = narrowest, last = 0; w <= 64 && w + h2 <= cap[i]; ++w) {
                const int tx = even[w];
                if (tx == last) continue;
                last = tx;
                const int room = cap[i] / (tx + h2) - h2;
                if (room < 1) break;
                const int nty = (p.ny + room - 1) / room;
                offer(shape[i], tx, (p.ny + nty - 1) / nty);
            }
        if (f64 && D <= 10) offer(kTile32, 32 - h2, 32 - h2);
        if (!f64 && D <= 10) offer(kRows768, 64 - h2, 36 - h2);
        if (fast && D <= 10) offer(kRows1024, 64 - h2, 32 - h2);
        const Launch few = few_steps(p, force, cus, D);
        pl.at[D] = few.us > 0.0 ? Launch{few.shape, few.tx, few.ty, std::max(few.us, best.us)} : best;
    }
    const double el = f64 ? 8.0 : 4.0;
    pl.at[1].us = 2.7 + (double)p.nx * p.ny * 19.0 * el / 5.0e6;
    double best[kPlanRoom + 1] = {};
    for (int r = 1; r <= kPlanRoom; ++r) {
        best[r] = 1e30;
        for (int D = 1; D <= std::min(r, kMaxDepth); ++D)
            if (pl.at[D].us + best[r - D] < best[r]) {
                best[r] = pl.at[D].us + best[r - D];
                pl.first[r] = (signed char)D;
            }
    }
    pl.longest = 1;
    for (int D = 2; D <= kMaxDepth; ++D)
        if (pl.at[D].us / D < pl.at[pl.longest].us / pl.longest) pl.longest = D;
    return pl;
}

int launch_depth(const Plan &pl, int64_t room)
{
    return room > kPlanRoom ? pl.longest : pl.first[std::max<int64_t>(room, 1)];
}

template <typename R, bool W, int PK, bool FF>
struct FieldsFn {
    static void run(const lbm_handle *h, double *u, double *rho, double *part)
    {
        launch_fields_t<R, W, PK, FF>(h, u, rho, part);
    }
};

// The mean velocity of the current state: queued here, fetched by wait_mean.
void queue_mean(lbm_handle *h)
{
    double *part = reinterpret_cast<double *>(h->ws + h->L.off_part);
    dispatch<FieldsFn>(h, (double *)nullptr, (double *)nullptr, part);
    hipLaunchKernelGGL(k_reduce_pairs, dim3(1), dim3(kBlock), 0, h->stream, part, h->L.nbx * h->L.nby,
                       1.0 / ((double)h->p.nx * h->p.ny), ++h->means, h->host_res);
}

// Wait until a kernel has stored `value` to pinned memory, with more work
// queued behind that kernel, so that waiting for the stream would idle the
// device: the host looks for the value itself for up to 5 ms, beside which the
// 10 us that an idle device loses are little, then waits for the stream.
// 64 x 64 cells, a check every 100 steps: 80 us per interval, 90 with a copy
// and a synchronisation (75 now that the steps take less).
hipError_t wait_value(const void *at, unsigned long long value, hipStream_t stream)
{
    const auto *p = static_cast<const unsigned long long *>(at);
    const auto end = std::chrono::steady_clock::now() + std::chrono::milliseconds(5);
    while (std::chrono::steady_clock::now() < end) {
        if (__atomic_load_n(p, __ATOMIC_ACQUIRE) == value) return hipSuccess;
        __builtin_ia32_pause();
    }
    return hipStreamSynchronize(stream);
}

// more: work is queued behind it. With none the stream is waited for, which a
// caller's own synchronisation (20 us after the bare result) then finds done.
lbm_status wait_mean(lbm_handle *h, bool more, double out[2])
{
    LBM_HIP(hipGetLastError());
    LBM_HIP(more ? wait_value(h->host_res + 2, h->means, h->stream) : hipStreamSynchronize(h->stream));
    out[0] = h->host_res[0];
    out[1] = h->host_res[1];
    return LBM_OK;
}

lbm_status mean_velocity(lbm_handle *h, double out[2])
{
    queue_mean(h);
    return wait_mean(h, false, out);
}

// Queue the steps of one stretch until at least `least` of them are queued.
int64_t queue_steps(lbm_handle *h, int64_t stretch, int64_t least)
{
    int64_t n = 0;
    while (n < std::min(stretch, least)) {
        const int d = launch_depth(h->plan, stretch - n);
        if (d >= 2)
            dispatch<StepDFn>(h, d);
        else
            dispatch<StepFn>(h);
        h->cur ^= 1;
        n += d;
    }
    return n;
}

template <typename R>
void field_check(const lbm_handle &h, const FieldRun &f, int64_t steps, bool first, long long *host)
{
    const int n = h.p.nx * h.p.ny;
    hipLaunchKernelGGL(k_field_check<R>, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, h.stream, step_args<R>(&h),
                       (long long)steps, first, f.tol, (long long)f.max_steps, reinterpret_cast<R *>(f.prev),
                       reinterpret_cast<double *>(h.ws + h.L.off_part), f.u, f.rho, f.done, host);
}

}  // namespace

namespace {

// The status that run_to_steady_field's checks mirror to the host: 32 bytes of
// pinned memory per thread that solves, kept from one solve to the next (freeing
// pinned memory waits for every stream of the device, so a solve that freed its
// own waited for unrelated work). A solve returns only once its stream is done, so
// no two solves use one mirror at a time. Given back when the thread ends; the
// main thread's goes with the process.
struct HostMirror {
    long long *p = nullptr;
    ~HostMirror()
    {
        if (p && gettid() != getpid()) (void)hipHostFree(p);
    }
};
thread_local HostMirror t_mirror;

}  // namespace

void fine_coef_planes(const lbm_params &p, char *ws, char **coef, char **force)
{
    const Layout L = layout_of(&p);
    *coef = ws + L.off_coef;
    *force = ws + L.off_force;
}

// The steps of the next check interval are queued (up to kAhead of them) before
// the host waits for the result of the last check, so the device does not idle
// while the host reads it.
lbm_status run_to_steady_field(const FieldRun &f, long long result[2])
{
    constexpr int64_t kAhead = 64;
    lbm_handle h{};
    h.p = f.p;
    h.L = layout_of(&f.p);
    h.stream = f.stream;
    h.ws = f.ws;
    h.has_force = true;
    h.plan = plan_launches(h.p, true, std::max(1, device_cu_count()));
    const bool f64 = h.p.pop_dtype == LBM_F64;
    if (!t_mirror.p)
        LBM_HIP(hipHostMalloc((void **)&t_mirror.p, 4 * sizeof(long long), hipHostMallocPortable | hipHostMallocCoherent));
    long long *host = t_mirror.p;
    host[0] = host[1] = host[2] = 0;
    hipError_t e = hipSuccess;
    const int n = h.p.nx * h.p.ny, nb = (n + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, f.stream, reinterpret_cast<int *>(f.done), 2);
    if (f64)
        hipLaunchKernelGGL(k_rest<double>, dim3(nb), dim3(kBlock), 0, f.stream,
                           reinterpret_cast<double *>(h.ws + h.L.off_a), (int)h.L.stride, n);
    else
        hipLaunchKernelGGL(k_rest<float>, dim3(nb), dim3(kBlock), 0, f.stream,
                           reinterpret_cast<float *>(h.ws + h.L.off_a), (int)h.L.stride, n);
    int64_t steps = 0, ahead = 0;  // ahead: steps of the current interval already queued
    while (e == hipSuccess) {
        queue_steps(&h, f.check_every - ahead, f.check_every);
        steps += f.check_every;
        if (f64)
            field_check<double>(h, f, steps, steps == f.check_every, host);
        else
            field_check<float>(h, f, steps, steps == f.check_every, host);
        ahead = steps < f.max_steps ? queue_steps(&h, f.check_every, kAhead) : 0;
        e = hipGetLastError();
        if (e == hipSuccess) e = wait_value(host, (unsigned long long)steps, f.stream);
        if (e != hipSuccess || host[2] != 0) break;
    }
    // what was queued ahead uses the workspace and the host's mirror
    const hipError_t es = hipStreamSynchronize(f.stream);
    if (e == hipSuccess) e = es;
    result[0] = host[0];
    result[1] = host[1];
    if (e == hipSuccess) return LBM_OK;
    t_mirror.p = nullptr;  // a kernel of the failed solve may still store to it
    return hip_check(e, "lbm_coarse_solve");
}

}  // namespace lbm

using namespace lbm;

extern "C" size_t lbm_workspace_bytes(const lbm_params *p)
{
    std::string why;
    if (!params_ok(p, why)) return 0;
    return layout_of(p).total;
}

extern "C" lbm_status lbm_plan_of(const lbm_params *p, int32_t force, int32_t cus, int64_t steps, int32_t out[4],
                                  double *us)
{
    std::string why;
    if (!out || !us || cus < 1 || steps < 1 || !params_ok(p, why))
        return set_error(LBM_EINVAL, "lbm_plan_of: " + why);
    const Plan pl = plan_launches(*p, force != 0, cus);
    const int d = launch_depth(pl, steps);
    out[0] = d;
    out[1] = d == 1 ? -1 : pl.at[d].shape;
    out[2] = d == 1 ? 0 : pl.at[d].tx;
    out[3] = d == 1 ? 0 : pl.at[d].ty;
    *us = pl.at[d].us;
    return LBM_OK;
}

extern "C" lbm_status lbm_init(lbm_handle **out, const lbm_params *p, const double *d_perm,
                               const double *d_force, void *d_ws, size_t ws_bytes,
                               hipStream_t stream)
{
    if (!out) return set_error(LBM_EINVAL, "lbm_init: handle pointer is NULL");
    *out = nullptr;
    std::string why;
    if (!params_ok(p, why)) return set_error(LBM_EINVAL, "lbm_init: " + why);
    if (!d_perm) return set_error(LBM_EINVAL, "lbm_init: permeability pointer is NULL");
    const Layout L = layout_of(p);
    if (!d_ws || ((uintptr_t)d_ws % kAlign) != 0)
        return set_error(LBM_EWORKSPACE, "lbm_init: workspace is NULL or not 256-byte aligned");
    if (ws_bytes < L.total)
        return set_error(LBM_EWORKSPACE, "lbm_init: workspace too small (need " +
                                             std::to_string(L.total) + " bytes)");
    lbm_handle *h = new (std::nothrow) lbm_handle{};
    if (!h) return set_error(LBM_EINVAL, "lbm_init: out of host memory");
    h->p = *p;
    h->L = L;
    h->stream = stream;
    h->ws = static_cast<char *>(d_ws);
    h->cur = 0;
    h->has_force = d_force != nullptr;
    h->plan = plan_launches(*p, h->has_force, std::max(1, device_cu_count()));
    if (hipHostMalloc((void **)&h->host_res, 4 * sizeof(double), hipHostMallocDefault) != hipSuccess) {
        delete h;
        return set_error(LBM_EDEVICE, "lbm_init: hipHostMalloc failed");
    }
    int *flag = reinterpret_cast<int *>(h->ws + L.off_flag);
    const int n = p->nx * p->ny;
    const int nb = (n + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, stream, flag, 1);
    reinterpret_cast<unsigned long long *>(h->host_res)[2] = 0;
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        if (p->pop_dtype == LBM_F64) {
            double *coef = reinterpret_cast<double *>(h->ws + L.off_coef);
            double *hf = reinterpret_cast<double *>(h->ws + L.off_force);
            double *pa = reinterpret_cast<double *>(h->ws + L.off_a);
            if (p->scheme == LBM_SCHEME_GUO)
                hipLaunchKernelGGL((k_init<double, 0>), dim3(nb), dim3(kBlock), 0, stream, d_perm, d_force, n,
                                   p->eps, p->nu, coef, hf, (int)L.cstride, pa, (int)L.stride, flag);
            else if (p->perm_kind == LBM_PERM_SCALAR)
                hipLaunchKernelGGL((k_init<double, 1>), dim3(nb), dim3(kBlock), 0, stream, d_perm, d_force, n,
                                   p->eps, p->nu, coef, hf, (int)L.cstride, pa, (int)L.stride, flag);
            else
                hipLaunchKernelGGL((k_init<double, 4>), dim3(nb), dim3(kBlock), 0, stream, d_perm, d_force, n,
                                   p->eps, p->nu, coef, hf, (int)L.cstride, pa, (int)L.stride, flag);
        } else {
            float *coef = reinterpret_cast<float *>(h->ws + L.off_coef);
            float *hf = reinterpret_cast<float *>(h->ws + L.off_force);
            float *pa = reinterpret_cast<float *>(h->ws + L.off_a);
            if (p->scheme == LBM_SCHEME_GUO)
                hipLaunchKernelGGL((k_init<float, 0>), dim3(nb), dim3(kBlock), 0, stream, d_perm, d_force, n,
                                   p->eps, p->nu, coef, hf, (int)L.cstride, pa, (int)L.stride, flag);
            else if (p->perm_kind == LBM_PERM_SCALAR)
                hipLaunchKernelGGL((k_init<float, 1>), dim3(nb), dim3(kBlock), 0, stream, d_perm, d_force, n,
                                   p->eps, p->nu, coef, hf, (int)L.cstride, pa, (int)L.stride, flag);
            else
                hipLaunchKernelGGL((k_init<float, 4>), dim3(nb), dim3(kBlock), 0, stream, d_perm, d_force, n,
                                   p->eps, p->nu, coef, hf, (int)L.cstride, pa, (int)L.stride, flag);
        }
        e = hipGetLastError();
    }
    int bad = 0;
    if (e == hipSuccess) e = hipMemcpyAsync(&bad, flag, sizeof(int), hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) {
        (void)hipHostFree(h->host_res);
        delete h;
        return hip_check(e, "lbm_init");
    }
    if (bad) {
        (void)hipHostFree(h->host_res);
        delete h;
        return set_error(LBM_EINVAL, (bad & 1) ? "lbm_init: permeability must be > 0 (or +inf) and "
                                                 "tensors invertible"
                                               : "lbm_init: force field has non-finite values");
    }
    *out = h;
    return LBM_OK;
}

extern "C" lbm_status lbm_step(lbm_handle *h, int64_t max_steps, double tol, int32_t check_every,
                               int64_t *steps_done, double mean_u[2])
{
    if (!h) return set_error(LBM_EINVAL, "lbm_step: handle is NULL");
    if (max_steps < 0) return set_error(LBM_EINVAL, "lbm_step: max_steps must be >= 0");
    if (check_every < 0) return set_error(LBM_EINVAL, "lbm_step: check_every must be >= 0");
    if (tol > 0.0 && check_every == 0)
        return set_error(LBM_EINVAL, "lbm_step: a tolerance needs check_every > 0");
    if (steps_done) *steps_done = 0;
    lbm_status st = (tol > 0.0) ? LBM_ENOTCONV : LBM_OK;
    int64_t done = 0;
    bool last_checked = false;
    double u[2] = {0.0, 0.0};
    // Several steps per launch unless a check or the end falls in between. The
    // first launch after a check is queued before the host waits for the
    // check's result: it writes the buffer that the state is not in, so it
    // counts only once the run is known to go on. That saves the kIdle us for
    // which the device waits for the host. With a tolerance any check may be the
    // last, and the launch is then waited for in vain, so it is queued once the
    // call's checks together have idled for as long as it takes: at once where a
    // launch takes 7 us (64 x 64 cells), not within the first 42 checks at
    // 4096 x 4096 (0.43 ms). So a run never pays more for its end than its checks
    // have cost it; two intervals of 12 steps that end in convergence take
    // 2050 us at 4096 x 4096, and took 2440 with the launch always queued.
    auto depth = [&] {
        const int64_t to_check = check_every > 0 ? check_every - done % check_every : max_steps - done;
        return launch_depth(h->plan, std::min<int64_t>(to_check, max_steps - done));
    };
    auto launch = [&](int n) {
        if (n >= 2)
            dispatch<StepDFn>(h, n);
        else
            dispatch<StepFn>(h);
        return n;
    };
    constexpr double kIdle = 10.0;
    double idled = 0.0;
    int ahead = 0;  // steps of a launch that is queued and not counted yet
    while (done < max_steps) {
        const int n = ahead ? ahead : launch(depth());
        ahead = 0;
        h->cur ^= 1;
        done += n;
        h->steps_total += n;
        last_checked = false;
        if (check_every > 0 && done % check_every == 0) {
            queue_mean(h);
            idled += kIdle;
            if (done < max_steps) {
                const int d = depth();
                if (!(tol > 0.0) || h->plan.at[d].us <= idled) ahead = launch(d);
            }
            lbm_status s = wait_mean(h, ahead > 0, u);
            if (s != LBM_OK) return s;
            last_checked = true;
            if (!std::isfinite(u[0]) || !std::isfinite(u[1])) {
                st = LBM_ENONFINITE;
                break;
            }
            if (tol > 0.0 && h->have_prev) {
                const double dx = u[0] - h->prev_u[0], dy = u[1] - h->prev_u[1];
                if (std::sqrt(dx * dx + dy * dy) <= tol * std::sqrt(u[0] * u[0] + u[1] * u[1])) {
                    h->prev_u[0] = u[0];
                    h->prev_u[1] = u[1];
                    st = LBM_OK;
                    break;
                }
            }
            h->prev_u[0] = u[0];
            h->prev_u[1] = u[1];
            h->have_prev = true;
        }
    }
    LBM_HIP(hipGetLastError());
    if (ahead) LBM_HIP(hipStreamSynchronize(h->stream));  // not needed, but it uses the workspace
    if (steps_done) *steps_done = done;
    if (mean_u) {
        if (!last_checked) {
            lbm_status s = mean_velocity(h, u);
            if (s != LBM_OK) return s;
        }
        mean_u[0] = u[0];
        mean_u[1] = u[1];
        if (st == LBM_OK && (!std::isfinite(u[0]) || !std::isfinite(u[1]))) st = LBM_ENONFINITE;
    }
    if (st == LBM_ENOTCONV) return set_error(st, "lbm_step: tolerance not reached within max_steps");
    if (st == LBM_ENONFINITE) return set_error(st, "lbm_step: non-finite mean velocity");
    return LBM_OK;
}

extern "C" lbm_status lbm_fields(lbm_handle *h, double *d_u, double *d_rho)
{
    if (!h) return set_error(LBM_EINVAL, "lbm_fields: handle is NULL");
    if (!d_u && !d_rho) return set_error(LBM_EINVAL, "lbm_fields: no output given");
    if (d_u) {
        dispatch<FieldsFn>(h, d_u, d_rho, (double *)nullptr);
    } else {
        // density only: velocities are still computed, into nowhere
        dispatch<FieldsFn>(h, (double *)nullptr, d_rho, (double *)nullptr);
    }
    LBM_HIP(hipGetLastError());
    return LBM_OK;
}

extern "C" lbm_status lbm_get_populations(lbm_handle *h, double *d_f)
{
    if (!h || !d_f) return set_error(LBM_EINVAL, "lbm_get_populations: NULL argument");
    const dim3 grid(h->L.nbx, h->L.nby);
    const char *cur = h->ws + (h->cur ? h->L.off_b : h->L.off_a);
    const int S = (int)h->L.stride;
    const bool w = h->p.walls_y != 0;
    if (h->p.pop_dtype == LBM_F64) {
        auto *fin = reinterpret_cast<const double *>(cur);
        if (w) hipLaunchKernelGGL((k_get_pops<double, true>), grid, dim3(kBlock), 0, h->stream, fin, S, h->p.nx, h->p.ny, h->p.rho0, d_f);
        else   hipLaunchKernelGGL((k_get_pops<double, false>), grid, dim3(kBlock), 0, h->stream, fin, S, h->p.nx, h->p.ny, h->p.rho0, d_f);
    } else {
        auto *fin = reinterpret_cast<const float *>(cur);
        if (w) hipLaunchKernelGGL((k_get_pops<float, true>), grid, dim3(kBlock), 0, h->stream, fin, S, h->p.nx, h->p.ny, h->p.rho0, d_f);
        else   hipLaunchKernelGGL((k_get_pops<float, false>), grid, dim3(kBlock), 0, h->stream, fin, S, h->p.nx, h->p.ny, h->p.rho0, d_f);
    }
    LBM_HIP(hipGetLastError());
    return LBM_OK;
}

extern "C" lbm_status lbm_set_populations(lbm_handle *h, const double *d_f)
{
    if (!h || !d_f) return set_error(LBM_EINVAL, "lbm_set_populations: NULL argument");
    const dim3 grid(h->L.nbx, h->L.nby);
    char *cur = h->ws + (h->cur ? h->L.off_b : h->L.off_a);
    const int S = (int)h->L.stride;
    const bool w = h->p.walls_y != 0;
    if (h->p.pop_dtype == LBM_F64) {
        auto *fo = reinterpret_cast<double *>(cur);
        if (w) hipLaunchKernelGGL((k_set_pops<double, true>), grid, dim3(kBlock), 0, h->stream, d_f, h->p.nx, h->p.ny, h->p.rho0, fo, S);
        else   hipLaunchKernelGGL((k_set_pops<double, false>), grid, dim3(kBlock), 0, h->stream, d_f, h->p.nx, h->p.ny, h->p.rho0, fo, S);
    } else {
        auto *fo = reinterpret_cast<float *>(cur);
        if (w) hipLaunchKernelGGL((k_set_pops<float, true>), grid, dim3(kBlock), 0, h->stream, d_f, h->p.nx, h->p.ny, h->p.rho0, fo, S);
        else   hipLaunchKernelGGL((k_set_pops<float, false>), grid, dim3(kBlock), 0, h->stream, d_f, h->p.nx, h->p.ny, h->p.rho0, fo, S);
    }
    h->have_prev = false;
    LBM_HIP(hipGetLastError());
    return LBM_OK;
}

extern "C" int64_t lbm_steps_total(const lbm_handle *h) { return h ? h->steps_total : -1; }

extern "C" void lbm_destroy(lbm_handle *h)
{
    if (!h) return;
    if (h->host_res) (void)hipHostFree(h->host_res);
    delete h;
}
