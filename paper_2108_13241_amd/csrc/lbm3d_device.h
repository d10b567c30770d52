// Device-side pieces of the D3Q19 kernels (one step per launch in
// lbm3d_kernels.hip, two in lbm3d_pair.hip): lattice constants, storage codecs,
// the collision and column offsets.
#pragma once

#include "lbm3d_launch.h"
#include "lbm_device.h"

namespace lbm3 {
namespace {

using lbm::kChunk;
using lbm::store_nt;
using lbm::xcd_remap;
using lbm::wrap_dec;
using lbm::wrap_inc;
constexpr int kBlock = 256;
constexpr int Q = 19;

// Velocities: rest; axes +x, -x, +y, -y, +z, -z; edges as opposite pairs
// (+x+y, -x-y), (+x-y, -x+y), (+x+z, -x-z), (+x-z, -x+z), (+y+z, -y-z),
// (+y-z, -y+z).  opp(i) = i + 1 for odd i, i - 1 for even i > 0.
__device__ constexpr int kCx[Q] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
__device__ constexpr int kCy[Q] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
__device__ constexpr int kCz[Q] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
__device__ constexpr int kOpp[Q] = {0, 2, 1, 4, 3, 6, 5, 8, 7, 10, 9, 12, 11, 14, 13, 16, 15, 18, 17};
// Weights of Eq. 6 for D3Q19: 1/3 at rest, 1/18 on the axes, 1/36 on the edges.
__device__ constexpr double kW[Q] = {1.0 / 3.0,  1.0 / 18.0, 1.0 / 18.0, 1.0 / 18.0, 1.0 / 18.0,
                                     1.0 / 18.0, 1.0 / 18.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0,
                                     1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0,
                                     1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0, 1.0 / 36.0};

enum : uint8_t { kFluid = 0, kSolid = 1, kBoundary = 2 };

// Storage codecs: FP64 stores f_i; the narrow formats store the deviation
// h_i = f_i - w_i (rho0 = 1) and the collision works on h_i (FP32 arithmetic).
struct F64 {
    using mem = double;
    using real = double;
    static constexpr bool kShift = false;
    static __device__ __forceinline__ real ld(mem v, int) { return v; }
    static __device__ __forceinline__ mem st(real v, int) { return v; }
    static __device__ __forceinline__ double canon(real v, int) { return v; }
    static __device__ __forceinline__ mem from_canon(double f, int) { return f; }
};
template <class M>
struct Shifted {
    using mem = M;
    using real = float;
    static constexpr bool kShift = true;
    static __device__ __forceinline__ real ld(mem v, int) { return (float)v; }
    static __device__ __forceinline__ mem st(real v, int)
    {
        if constexpr (sizeof(M) == 2)
            asm volatile("" : "+v"(v));  // round to FP32 first, identically everywhere
        return (mem)v;
    }
    static __device__ __forceinline__ double canon(real v, int i) { return (double)v + kW[i]; }
    static __device__ __forceinline__ mem from_canon(double f, int i)
    {
        return (mem)(float)(f - kW[i]);
    }
};

__device__ __forceinline__ double recip(double v) { return 1.0 / v; }
__device__ __forceinline__ float recip(float v)
{
    const float r = __builtin_amdgcn_rcpf(v);
    return __builtin_fmaf(__builtin_fmaf(-v, r, 1.0f), r, r);
}

// c . v for the first direction of pair k: (1,0,0), (0,1,0), (0,0,1), (1,1,0),
// (1,-1,0), (1,0,1), (1,0,-1), (0,1,1), (0,1,-1), without multiplications.
template <class R>
__device__ __forceinline__ R pair_dot(int k, R vx, R vy, R vz)
{
    switch (k) {
    case 0: return vx;
    case 1: return vy;
    case 2: return vz;
    case 3: return vx + vy;
    case 4: return vx - vy;
    case 5: return vx + vz;
    case 6: return vx - vz;
    case 7: return vy + vz;
    default: return vy - vz;
    }
}

// BGK collision with Guo forcing (F = rho g) at one node, in place:
//   f_i <- f_i - omega (f_i - f^eq_i) + (1 - omega/2) S_i,
// u = m / rho + g / 2, f^eq of Eq. 6 with the D3Q19 weights,
// S_i = w_i [3 (c_i - u) . F + 9 (c_i . u)(c_i . F)].  Opposite directions
// share everything but the terms odd in c, so they are updated as a pair; with
// SHIFT, f holds deviations and rho = 1 + sum is never rounded (rho v = v + sum v).
// TRT: the pair's symmetric part P = (f_i + f_opp)/2 relaxes with omega and its
// antisymmetric part M = (f_i - f_opp)/2 with omega_m (forcing split alike);
// f_i = P + M, f_opp = P - M.
// MRT: multiple-relaxation-time collision in the D3Q19 moment basis of
// d'Humieres et al. (rows, as polynomials of c: rho 1; e 19|c|^2 - 30;
// eps (21|c|^4 - 53|c|^2 + 24)/2; j c; q (5|c|^2 - 9) c; 3p_xx 3c_x^2 - |c|^2;
// 3pi_xx (3|c|^2 - 5)(3c_x^2 - |c|^2); p_ww c_y^2 - c_z^2; pi_ww (3|c|^2 - 5)
// (c_y^2 - c_z^2); p_xy, p_yz, p_xz; m_x (c_y^2 - c_z^2) c_x, m_y (c_z^2 - c_x^2)
// c_y, m_z (c_x^2 - c_y^2) c_z; orthogonal, squared norms kMrt3Norm).  The
// moments of d = f - f^eq and of the forcing term relax as
//   Delta_k = s_k d_k - (1 - s_k / 2) S_k,  f_i <- f_i - sum_k M_ki Delta_k / |M_k|^2,
// with s_e, s_eps, s_q, s_pi, s_m and omega on the shear moments (3p_xx, p_ww,
// p_xy, p_yz, p_xz); Delta_rho = 0 and Delta_j = -F (the conserved moments).
template <class R>
struct Rates3 {
    R omega_m;                         // TRT: antisymmetric rate
    R s_e, s_eps, s_q, s_pi, s_m;      // MRT
};

// Row k of the D3Q19 MRT matrix at direction i (small integers); with the
// loops unrolled every coefficient folds to a constant.
__device__ __forceinline__ constexpr int mrt3_coef(int k, int i)
{
    const int cx = kCx[i], cy = kCy[i], cz = kCz[i], c2 = cx * cx + cy * cy + cz * cz;
    switch (k) {
    case 0: return 1;
    case 1: return 19 * c2 - 30;
    case 2: return (21 * c2 * c2 - 53 * c2 + 24) / 2;
    case 3: return cx;
    case 4: return (5 * c2 - 9) * cx;
    case 5: return cy;
    case 6: return (5 * c2 - 9) * cy;
    case 7: return cz;
    case 8: return (5 * c2 - 9) * cz;
    case 9: return 3 * cx * cx - c2;
    case 10: return (3 * c2 - 5) * (3 * cx * cx - c2);
    case 11: return cy * cy - cz * cz;
    case 12: return (3 * c2 - 5) * (cy * cy - cz * cz);
    case 13: return cx * cy;
    case 14: return cy * cz;
    case 15: return cx * cz;
    case 16: return (cy * cy - cz * cz) * cx;
    case 17: return (cz * cz - cx * cx) * cy;
    default: return (cx * cx - cy * cy) * cz;
    }
}
__device__ constexpr int kMrt3Norm[Q] = {19, 2394, 252, 10, 40, 10, 40, 10, 40, 36,
                                         72, 12,   24,  4,  4,  4,  8,  8,  8};

template <class R, bool SHIFT, bool FORCE, bool TRT = false, bool MRT = false>
__device__ __forceinline__ void collide3(R (&f)[Q], R omega, R gx, R gy, R gz,
                                         const Rates3<R> &rt = Rates3<R>{})
{
    const R omega_m = rt.omega_m;
    R sum = f[0];
#pragma unroll
    for (int i = 1; i < Q; ++i)
        sum += f[i];
    R mx = R(0), my = R(0), mz = R(0);
#pragma unroll
    for (int i = 1; i < Q; i += 2) {
        const R d = f[i] - f[i + 1];
        if (kCx[i] > 0) mx += d; else if (kCx[i] < 0) mx -= d;
        if (kCy[i] > 0) my += d; else if (kCy[i] < 0) my -= d;
        if (kCz[i] > 0) mz += d; else if (kCz[i] < 0) mz -= d;
    }
    auto rho_times = [&](R v) -> R {
        if constexpr (SHIFT)
            return v + sum * v;
        else
            return sum * v;
    };
    R ux, uy, uz;
    if constexpr (SHIFT) {
        const R q = sum * recip(R(1) + sum);
        ux = mx - mx * q;
        uy = my - my * q;
        uz = mz - mz * q;
    } else {
        const R inv = recip(sum);
        ux = mx * inv;
        uy = my * inv;
        uz = mz * inv;
    }
    R Fx = R(0), Fy = R(0), Fz = R(0);
    if constexpr (FORCE) {
        ux += R(0.5) * gx;
        uy += R(0.5) * gy;
        uz += R(0.5) * gz;
        Fx = rho_times(gx);
        Fy = rho_times(gy);
        Fz = rho_times(gz);
    }
    const R usq = R(1.5) * (ux * ux + uy * uy + uz * uz);
    const R C0 = SHIFT ? sum - rho_times(usq) : rho_times(R(1) - usq);
    const R keep = R(1) - omega, guo = R(1) - R(0.5) * omega;
    const R uF = ux * Fx + uy * Fy + uz * Fz;
    if constexpr (MRT) {
        R d[Q], sg[Q];
        d[0] = f[0] - R(kW[0]) * C0;
        sg[0] = FORCE ? R(kW[0]) * (R(-3) * uF) : R(0);
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const int i = 2 * k + 1, j = i + 1;
            const R w = R(kW[i]);
            const R cu = pair_dot(k, ux, uy, uz);
            const R even = w * (C0 + rho_times(R(4.5) * (cu * cu)));
            const R odd = w * rho_times(R(3) * cu);
            d[i] = f[i] - (even + odd);
            d[j] = f[j] - (even - odd);
            if constexpr (FORCE) {
                const R cF = pair_dot(k, Fx, Fy, Fz);
                const R se = w * (R(9) * cu * cF - R(3) * uF);
                const R so = R(3) * w * cF;
                sg[i] = se + so;
                sg[j] = se - so;
            } else {
                sg[i] = sg[j] = R(0);
            }
        }
        // Delta_k / |M_k|^2 for every row (conserved rows set directly)
        R del[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            if (k == 0) {
                del[k] = R(0);
                continue;
            }
            if (k == 3 || k == 5 || k == 7) {
                const R Fk = k == 3 ? Fx : k == 5 ? Fy : Fz;
                del[k] = FORCE ? -Fk * R(1.0 / kMrt3Norm[k]) : R(0);
                continue;
            }
            R dk = R(0), sk = R(0);
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const int c = mrt3_coef(k, i);
                if (c == 1) {
                    dk += d[i];
                    if constexpr (FORCE) sk += sg[i];
                } else if (c == -1) {
                    dk -= d[i];
                    if constexpr (FORCE) sk -= sg[i];
                } else if (c != 0) {
                    dk += R(c) * d[i];
                    if constexpr (FORCE) sk += R(c) * sg[i];
                }
            }
            const R sr = k == 1 ? rt.s_e : k == 2 ? rt.s_eps
                       : (k == 4 || k == 6 || k == 8) ? rt.s_q
                       : (k == 10 || k == 12) ? rt.s_pi
                       : (k >= 16) ? rt.s_m : omega;
            R dl = sr * dk;
            if constexpr (FORCE)
                dl -= (R(1) - R(0.5) * sr) * sk;
            del[k] = dl * R(1.0 / kMrt3Norm[k]);
        }
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            R acc = R(0);
#pragma unroll
            for (int k = 1; k < Q; ++k) {
                const int c = mrt3_coef(k, i);
                if (c == 1)
                    acc += del[k];
                else if (c == -1)
                    acc -= del[k];
                else if (c != 0)
                    acc += R(c) * del[k];
            }
            f[i] -= acc;
        }
        return;
    }
    {
        R s = keep * f[0] + omega * (R(kW[0]) * C0);
        if constexpr (FORCE)
            s += guo * (R(kW[0]) * (R(-3) * uF));
        f[0] = s;
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int i = 2 * k + 1, j = i + 1;
        const R w = R(kW[i]);
        const R cu = pair_dot(k, ux, uy, uz);
        const R even = w * (C0 + rho_times(R(4.5) * (cu * cu)));
        const R odd = w * rho_times(R(3) * cu);
        if constexpr (TRT) {
            R P = keep * (R(0.5) * (f[i] + f[j])) + omega * even;
            R M = (R(1) - omega_m) * (R(0.5) * (f[i] - f[j])) + omega_m * odd;
            if constexpr (FORCE) {
                const R cF = pair_dot(k, Fx, Fy, Fz);
                P += guo * (w * (R(9) * cu * cF - R(3) * uF));
                M += (R(1) - R(0.5) * omega_m) * (R(3) * w * cF);
            }
            f[i] = P + M;
            f[j] = P - M;
        } else {
            R a = keep * f[i] + omega * (even + odd);
            R b = keep * f[j] + omega * (even - odd);
            if constexpr (FORCE) {
                const R cF = pair_dot(k, Fx, Fy, Fz);
                const R se = w * (R(9) * cu * cF - R(3) * uF);
                const R so = R(3) * w * cF;
                a += guo * (se + so);
                b += guo * (se - so);
            }
            f[i] = a;
            f[j] = b;
        }
    }
}

// Element offset of column x inside a row of 64-node chunks.
__device__ __forceinline__ uint32_t col_off(int x)
{
    return ((((uint32_t)x >> 6) * (uint32_t)(Q * kChunk)) | ((uint32_t)x & 63u)) & 0x0FFFFFFFu;
}

}  // namespace
}  // namespace lbm3
