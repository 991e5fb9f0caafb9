// Per-element model arithmetic shared by the ring and lattice kernels: the
// stage value, the coupling map and the local right-hand side.
#pragma once

#include "nd_dev.h"

namespace nd {


// ------------------------------------------------------------------ models
// Flip the sign of v where bit 31 of m is set.
__device__ __forceinline__ double flip_sign(double v, uint32_t m) {
    return __longlong_as_double(__double_as_longlong(v) ^ ((long long)(m & 0x80000000u) << 32));
}

// A double constant, with SC held in a scalar register pair the FMA reads it from.
// Left to itself the compiler keeps polynomial coefficients in vector registers:
// about 20 of them, which the kernels at the 128-register limit do not have (ball
// P = 6: spills, 90 against 82 us per stage; the cube's plane loop). Elsewhere the
// scalar moves cost more than the registers (ball P = 8 63 against 67 us, one ring
// of 1024 0.93 against 0.97 us per stage).
template <bool SC>
__device__ __forceinline__ double sconst(double c) {
    if constexpr (SC) asm("" : "+s"(c));
    return c;
}

// sin and cos of one double: Cody-Waite reduction by pi/2 (two-part constant,
// each part subtracted with one fused multiply-add), then minimax polynomials of
// sin and cos on [-pi/4, pi/4] of degrees 13 and 14 (fitted by the Remez
// exchange on (sin r - r)/r^3 and (cos r - 1 + r^2/2)/r^4, coefficients rounded
// one after the other; approximation error 1.6e-18 and 4.8e-20) by Horner in
// r^2, and the quadrant swap.  The quadrant q mod 4 is read from the bits of
// frac(q / 4), which is 0, 1/4, 1/2 or 3/4 for any integer q: high words 0,
// 0x3fd00000, 0x3fe00000 and 0x3fe80000, so bits 19 and 20 give the swap, bit 21
// the sign of the sine and bit 21 after adding 0x180000 that of the cosine.
// The reduced argument carries the rounding of the first subtraction (up to
// half an ulp of r, about 5.5e-17 near pi/4) and the neglected third part of pi/2
// (grows with |x|); over 6e6 arguments up to 3e13 the largest error against
// 113-bit values was 1.30e-16 and the rms error 3.17e-17 (Taylor series of two
// degrees more: 1.44e-16 and 3.20e-17).  Bound: FP64 issue of the callers; this
// form takes 20 FP64 operations, the Taylor form with the quadrant by floor and
// conversion took 24.  Inf and NaN give NaN.
template <bool SC = false>
__device__ __forceinline__ void sincos_cw(double x, double* sp, double* cp) {
    const double q = rint(x * 0.63661977236758134308);          // x / (pi/2), nearest
    const double r1 = fma(-q, 1.5707963267948966192, x);        // pi/2 rounded to double
    const double r = fma(-q, 6.123233995736766036e-17, r1);     // pi/2 minus that
    const double r2 = r * r;
    double ps = fma(sconst<SC>(1.588805743874414e-10), r2, sconst<SC>(-2.5050590858861764e-08));
    ps = fma(ps, r2, sconst<SC>(2.7557312482336066e-06));
    ps = fma(ps, r2, sconst<SC>(-0.00019841269825742673));
    ps = fma(ps, r2, sconst<SC>(0.008333333333316218));
    ps = fma(ps, r2, sconst<SC>(-0.166666666666666));
    const double sn = fma(r * r2, ps, r);
    double pc = fma(sconst<SC>(-1.1359934247561652e-11), r2, sconst<SC>(2.087572928127532e-09));
    pc = fma(pc, r2, sconst<SC>(-2.75573144010307e-07));
    pc = fma(pc, r2, sconst<SC>(2.4801587289671537e-05));
    pc = fma(pc, r2, sconst<SC>(-0.0013888888888874474));
    pc = fma(pc, r2, sconst<SC>(0.0416666666666666));
    pc = fma(pc, r2, -0.5);
    const double cs = fma(r2, pc, 1.0);
    const uint32_t f = (uint32_t)((unsigned long long)__double_as_longlong(__builtin_amdgcn_fract(q * 0.25)) >> 32);
    const bool swap = (f & 0x180000u) != 0;
    *sp = flip_sign(swap ? cs : sn, f << 10);
    *cp = flip_sign(swap ? sn : cs, (f + 0x180000u) << 10);
}

// The descriptor fields of a step loop that stays in one workgroup.
struct ModelConst {
    double p[7], dt3, dt6;
    __device__ __forceinline__ explicit ModelConst(const NetDesc& d) : dt3(d.dt3), dt6(d.dt6) {
#pragma unroll
        for (int q = 0; q < 7; ++q) p[q] = d.p[q];
    }
};

// The right-hand sides read the model constants as d.p[], d a NetDesc or a ModelConst.
template <int MODEL, class KT>
struct RingModel;

// Kuramoto-Sakaguchi, Eq. (3) with m = 0, eps = 1:
//   k_i = omega + mu/(2P) sum_j sin(z_j - z_i - alpha)
//       = omega + mu/(2P) [cos(z_i + alpha) S_i - sin(z_i + alpha) C_i]
// with (C_i, S_i) the window sums of (cos z_j, sin z_j).
// p = {omega, mu/(2P), cos alpha, sin alpha}
template <class KT>
struct RingModel<ND_KURAMOTO, KT> {
    static constexpr int V = 1;
    template <bool SC = false>
    __device__ static __forceinline__ double2 map(const double* z) {
        double s, c;
        if constexpr (sizeof(KT) == 8) {
            sincos_cw<SC>(z[0], &s, &c);
        } else {
            // bulk float: reduce to revolutions in double, then the hardware
            // sin/cos (their argument is in revolutions)
            double r = z[0] * 0.15915494309189535;  // 1 / (2 pi)
            r -= rint(r);
            float rf = (float)r;
            s = (double)__builtin_amdgcn_sinf(rf);
            c = (double)__builtin_amdgcn_cosf(rf);
        }
        return make_double2(c, s);
    }
    template <class D>
    __device__ static __forceinline__ void rhs(const D& d, const double* z, double2 xo, double2 W, double* k) {
        (void)z;
        if constexpr (sizeof(KT) == 8) {
            const double ca = fma(xo.x, d.p[2], -(xo.y * d.p[3]));
            const double sa = fma(xo.y, d.p[2], xo.x * d.p[3]);
            k[0] = fma(d.p[1], fma(ca, W.y, -(sa * W.x)), d.p[0]);
        } else {
            const float cf = (float)xo.x, sf = (float)xo.y;
            const float ca = cf * (float)d.p[2] - sf * (float)d.p[3];
            const float sa = sf * (float)d.p[2] + cf * (float)d.p[3];
            k[0] = d.p[0] + d.p[1] * ((double)ca * W.y - (double)sa * W.x);
        }
    }
};

// Kuramoto-Sakaguchi with inertia, Eq. (3) with m != 0, as a first-order
// system in (phi, psi = dphi/dt); the coupling is the Kuramoto one on phi:
//   dphi = psi,  dpsi = (omega - eps psi + mu/L [cos(phi+alpha) S - sin(phi+alpha) C]) / m
// p = {omega, mu/L, cos alpha, sin alpha, eps, 1/m}
template <class KT>
struct RingModel<ND_KURAMOTO_INERTIA, KT> {
    static constexpr int V = 2;
    template <bool SC = false>
    __device__ static __forceinline__ double2 map(const double* z) {
        return RingModel<ND_KURAMOTO, KT>::template map<SC>(z);
    }
    template <class D>
    __device__ static __forceinline__ void rhs(const D& d, const double* z, double2 xo, double2 W, double* k) {
        double force[1];
        RingModel<ND_KURAMOTO, KT>::rhs(d, z, xo, W, force);  // omega + coupling, as first-order Kuramoto
        k[0] = z[1];
        if constexpr (sizeof(KT) == 8) {
            k[1] = fma(-d.p[4], z[1], force[0]) * d.p[5];
        } else {
            k[1] = (double)(((float)force[0] - (float)d.p[4] * (float)z[1]) * (float)d.p[5]);
        }
    }
};

// FitzHugh-Nagumo, Eq. (2) (tau = 0, D = 0, I_app = 0) with the rotational
// coupling B(phi) on (u_j - u_i, v_j - v_i), kappa = sigma / 2P:
//   eps du = u - u^3/3 - v + kappa ( cos phi Du + sin phi Dv)
//       dv = u + a         + kappa (-sin phi Du + cos phi Dv)
// Du = sum_j u_j - 2P u_i, Dv likewise (double, before any rounding to float).
// The divisions by 3 and eps are multiplications by the rounded reciprocals
// (a last-bit difference from the division; no division sequence per element).
// p = {eps, a, kappa, cos phi, sin phi, 2P, 1/eps}
template <class KT>
struct RingModel<ND_FHN, KT> {
    static constexpr int V = 2;
    template <bool SC = false>
    __device__ static __forceinline__ double2 map(const double* z) {
        return make_double2(z[0], z[1]);
    }
    template <class D>
    __device__ static __forceinline__ void rhs(const D& d, const double* z, double2 xo, double2 W, double* k) {
        (void)xo;
        const double u = z[0], v = z[1];
        const double Du = W.x - d.p[5] * u;
        const double Dv = W.y - d.p[5] * v;
        if constexpr (sizeof(KT) == 8) {
            const double cu = fma(d.p[3], Du, d.p[4] * Dv);
            const double cv = fma(d.p[3], Dv, -(d.p[4] * Du));
            const double cubic = fma(u * u * u, -1.0 / 3.0, u);
            k[0] = fma(d.p[2], cu, cubic - v) * d.p[6];
            k[1] = fma(d.p[2], cv, u + d.p[1]);
        } else {
            const float uf = (float)u, vf = (float)v, duf = (float)Du, dvf = (float)Dv;
            const float kap = (float)d.p[2], cph = (float)d.p[3], sph = (float)d.p[4];
            const float cu = kap * (cph * duf + sph * dvf);
            const float cv = kap * (cph * dvf - sph * duf);
            k[0] = (double)((uf - uf * uf * uf * (1.0f / 3.0f) - vf + cu) * (float)d.p[6]);
            k[1] = (double)(uf + (float)d.p[1] + cv);
        }
    }
};

template <class KT>
__device__ __forceinline__ double kq(double k) {
    return (double)(KT)k;  // the value that is stored (and that every reader sees)
}

// Lattice stage kernels, FP64: the three buffers d.k hold the stage values z2, z3,
// z4 instead of the slopes.  A halo element is then one load in every stage (with
// the slopes it is y and k_prev in stages 2 to 4), and the step is completed from
// the differences to y:
//   stage 1: reads y             writes z2 = y + dt/2 k1
//   stage 2: reads y, z2         writes z3 = y + dt/2 k2, acc = (z2 - y) + 2 (z3 - y)
//   stage 3: reads y, z3         writes z4 = y + dt k3
//   stage 4: reads y, z4, acc    writes y' = y + dt/6 k4 + (acc + (z4 - y)) / 3
// the same 13 accesses per element and step.  The differences are exact or small,
// so y' has one rounding at the scale of y besides those of z2 .. z4 (weights 1/3,
// 2/3, 1/3), fewer than the slope form's four.  FP32-bulk keeps slopes: stored
// in float they are half the bytes of a stage value.
template <class KT>
constexpr bool kStageValues = sizeof(KT) == 8;

// Value read for the stage input at an element: v the d.k entry (stages 2 to 4), y the state.
template <int STAGE, class KT>
__device__ __forceinline__ double lattice_z(double y, double v, double cdt) {
    if (STAGE == 1) return y;
    return kStageValues<KT> ? v : fma(cdt, v, y);
}

// What stage STAGE writes for one variable of one element: slope kk, own state y,
// own d.k entry v (stages 2 and 4), own acc (stage 4); q the element, `off` the
// variable's offset.  Returns the new state in stage 4.
template <int STAGE, class KT>
__device__ __forceinline__ double lattice_write(const NetDesc& d, int par, int64_t off, uint32_t q, double kk, double y,
                                                double v, double acc) {
    if constexpr (kStageValues<KT>) {
        if (STAGE <= 3) {
            const double z = fma(STAGE == 3 ? d.dt : 0.5 * d.dt, kk, y);
            st32(gp((double*)d.k[STAGE - 1 < 3 ? STAGE - 1 : 0]) + off, q, z);
            if (STAGE == 2) st32(gp(d.acc) + off, q, fma(2.0, z - y, v - y));
            return 0.0;
        }
        const double yo = y + fma(d.dt6, kk, (acc + (v - y)) * (1.0 / 3.0));
        st32(gp(d.y[par ^ 1]) + off, q, yo);
        flag_nonfinite(d, yo);
        return yo;
    } else {
        if (STAGE <= 3) st32(gp((KT*)d.k[STAGE - 1 < 3 ? STAGE - 1 : 0]) + off, q, (KT)kk);
        if (STAGE == 2) st32(gp(d.acc) + off, q, fma(d.dt3, kk, fma(d.dt6, v, y)));
        if (STAGE <= 3) return 0.0;
        const double yo = fma(d.dt6, kk, fma(d.dt3, v, acc));
        st32(gp(d.y[par ^ 1]) + off, q, yo);
        flag_nonfinite(d, yo);
        return yo;
    }
}

// Stage value z_v(idx) = y + c dt k_prev (stage 1: y).  Written once here so the
// producer of the tile sums and every reader of the window ends agree bitwise.
template <int V, class KT, class YP, class KP>
__device__ __forceinline__ void stage_z(YP y, KP kp, double cdt, int64_t n, int64_t idx, double* z) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const double yy = y[v * n + idx];
        z[v] = kp ? fma(cdt, (double)kp[v * n + idx], yy) : yy;
    }
}

}  // namespace nd
