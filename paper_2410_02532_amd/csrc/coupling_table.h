// coupling_table.h -- the RK4 half-steps of launches that take their coupling
// coefficients from a table filled ahead of them (FP64 phasors once per step boundary
// and instance, instead of in every tile).
#pragma once
#include "ssfm_kernels.h"

namespace opo {

// *p, for p the same in every lane and *p not written during the kernel: a scalar load.
template <typename T> __device__ __forceinline__ T uload(const T *p)
{
    using Q = const __attribute__((address_space(4))) unsigned;
    static_assert(sizeof(T) % 4 == 0, "whole dwords");
    const unsigned long long b = reinterpret_cast<unsigned long long>(p);
    Q *q = reinterpret_cast<Q *>(static_cast<unsigned long long>(__builtin_amdgcn_readfirstlane(static_cast<unsigned>(b >> 32))) << 32 |
                                 static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<unsigned>(b))));
    unsigned w[sizeof(T) / 4];
#pragma unroll
    for (unsigned k = 0; k < sizeof(T) / 4; ++k) w[k] = q[k];
    T v;
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

// Triple-jump coefficients of the fourth-order composition: a = 1/(2 - 2^(1/3)),
// b = 1 - 2a (a + b + a = 1, 2a^3 + b^3 = 0).
constexpr double kTjA = 1.35120719195965763405;
constexpr double kTjB = -1.70241438391931526810;

// Step i of a pass in units of dz: start z, size tau, and the propagator table it uses.
// Symmetrized steps are the steps; the fourth-order composition runs three per step, of
// a, b and a times dz.
__host__ __device__ inline void substep(int order, int i, double &z, double &tau, int &sel)
{
    if (order != 4) {
        z = i;
        tau = 1.0;
        sel = 0;
        return;
    }
    const int j = i >= 0 ? i / 3 : -1, s = i - 3 * j;
    z = j + (s == 0 ? 0.0 : s == 1 ? kTjA : kTjA + kTjB);
    tau = s == 1 ? kTjB : kTjA;
    sel = s == 1 ? 1 : 0;
}

// Couplings of the column launches at step boundaries s0 .. s0 + count - 1 of a pass:
// entry (s - s0) n + i is boundary s of instance i, with the second half-step of step
// s - 1 and the first of step s, formed as in coupling_tile. Six threads an entry. Clears
// `cleared` ints at `clear` too (what a launch behind it starts from).
template <typename R>
__global__ __launch_bounds__(kThreads) void coupling_table(const InstDesc *inst, int n, int order, double dz_arg,
                                                           double zbase, int nz, int s0, int count, Coupling<R> *out,
                                                           int *clear, int cleared)
{
    using V = cplx<R>;
    const int id = blockIdx.x * kThreads + threadIdx.x, e = id / 6, q = id - 6 * e;
    for (int w = id; w < cleared; w += gridDim.x * kThreads) clear[w] = 0;
    if (e >= count * n) return;
    const int s = s0 + e / n, which = q / 3, st = q - 3 * which;
    const InstDesc &d = inst[e % n];
    const double dz = dz_arg > 0.0 ? dz_arg : d.length_mm / nz, zb = dz_arg > 0.0 ? zbase : 0.0;
    double z, tau;
    int sel;
    substep(order, which ? s : s - 1, z, tau, sel);
    if (!which) z += 0.5 * tau;
    const double h = 0.5 * tau * dz, hh = 0.5 * h;
    const double r = d.dk_rev * (zb + z * dz + 0.5 * h * st);
    double sn, cs;
    sincospi(2.0 * (r - rint(r)), &sn, &cs);
    const double kp = d.kappa[0] * hh, ks = d.kappa[1] * hh, ki = d.kappa[2] * hh;
    V *c = out[e].c[which][st];
    c[0] = mk<V>(static_cast<R>(kp * sn), static_cast<R>(kp * cs));
    c[1] = mk<V>(static_cast<R>(-ks * sn), static_cast<R>(ks * cs));
    c[2] = mk<V>(static_cast<R>(-ki * sn), static_cast<R>(ki * cs));
    out[e].g[which][st] = static_cast<R>(d.gamma[st] * hh);
}

// The couplings of kind 0 (dk = 0: i c, the same at every stage) of both half-steps, for
// kernels that read them with their first loads.
template <typename R> struct ImagCoupling {
    cplx<R> c[2][3];
    __device__ __forceinline__ explicit ImagCoupling(const Coupling<R> *coef)
    {
#pragma unroll
        for (int which = 0; which < 2; ++which)
#pragma unroll
            for (int x = 0; x < 3; ++x) c[which][x] = uload(&coef->c[which][0][x]);
    }
};

// Half-step `which` (0: the second of the step before, 1: the first of this step) of PF
// samples of NF waves. kind 0: dk = 0, 1: general couplings, 2: Kerr terms.
template <typename R, int NF, int PF>
__device__ __forceinline__ void half_step(cplx<R> (&v)[NF][PF], int kind, const ImagCoupling<R> &imag,
                                          const Coupling<R> *coef, int which)
{
    using V = cplx<R>;
    if (kind == 0) {
        V k[3][3];
#pragma unroll
        for (int x = 0; x < 3; ++x) k[0][x] = imag.c[which][x];
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            if constexpr (NF == 3) rk4_point_imag<R>(k, v[0][m], v[1][m], v[NF - 1][m]);
            else rk4_point2_imag<R>(k, v[0][m], v[1][m]);
        }
    } else {
        Coupling<R> cp;
#pragma unroll
        for (int st = 0; st < 3; ++st) {
#pragma unroll
            for (int x = 0; x < 3; ++x) cp.c[which][st][x] = uload(&coef->c[which][st][x]);
            cp.g[which][st] = uload(&coef->g[which][st]);
        }
#pragma unroll
        for (int m = 0; m < PF; ++m)
            rk4_fields<R, NF>(cp, which, false, kind == 2, v[0][m], v[1][m], v[NF - 1][m]);
    }
}

} // namespace opo
