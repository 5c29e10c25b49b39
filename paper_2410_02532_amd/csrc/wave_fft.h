// wave_fft.h -- FFT across the lanes of one wave, without LDS.
//
// N = RS M points of a column lie in PF registers of T = N/PF lanes. The forward
// transform is decimation in frequency: a radix-RS butterfly over the register index
// (the top digit of the position), the twiddles W_M^{r q} (q the rest of the
// position, held by the lanes), then the register digit changes places with the next
// digit of the lane index, so that it becomes the top digit of what is left. The
// inverse transform runs the same steps backwards. Changing places costs one
// v_permlane swap (lane distance 16, 32) or two DPP moves (4, 8) per pair of
// registers, where an exchange through LDS waits on a write, a barrier and a read.
#pragma once
#include "fft_tile.h"

namespace opo {

// Swaps lanes whose bit D is set of a with lanes whose bit D is clear of b.
template <int D> __device__ __forceinline__ void lane_swap32(unsigned &a, unsigned &b)
{
    if constexpr (D == 32 || D == 16) {
        const auto r = D == 32 ? __builtin_amdgcn_permlane32_swap(a, b, false, false)
                               : __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else if constexpr (D == 2) {
        // within quads: lanes 2, 3 take lanes 0, 1 of b, lanes 0, 1 take lanes 2, 3 of a
        const bool hi = (threadIdx.x & 2) != 0;
        const unsigned fb = __builtin_amdgcn_mov_dpp(b, 0x44, 0xf, 0xf, false);   // quad_perm 0 1 0 1
        const unsigned fa = __builtin_amdgcn_mov_dpp(a, 0xee, 0xf, 0xf, false);   // quad_perm 2 3 2 3
        a = hi ? fb : a;
        b = hi ? b : fa;
    } else {
        static_assert(D == 8 || D == 4, "lane distance");
        constexpr int shr = 0x110 + D, shl = 0x100 + D;                 // row_shr:D, row_shl:D
        constexpr int hi = D == 8 ? 0xc : 0xa, lo = D == 8 ? 0x3 : 0x5;   // banks with bit D set / clear
        const unsigned na = __builtin_amdgcn_update_dpp(a, b, shr, 0xf, hi, false);
        b = __builtin_amdgcn_update_dpp(b, a, shl, 0xf, lo, false);
        a = na;
    }
}
template <int D> __device__ __forceinline__ void lane_swap(float &a, float &b)
{
    unsigned x = __float_as_uint(a), y = __float_as_uint(b);
    lane_swap32<D>(x, y);
    a = __uint_as_float(x);
    b = __uint_as_float(y);
}
template <int D> __device__ __forceinline__ void lane_swap(double &a, double &b)
{
    unsigned long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    unsigned xl = static_cast<unsigned>(x), xh = static_cast<unsigned>(x >> 32);
    unsigned yl = static_cast<unsigned>(y), yh = static_cast<unsigned>(y >> 32);
    lane_swap32<D>(xl, yl);
    lane_swap32<D>(xh, yh);
    a = __longlong_as_double(static_cast<long long>(static_cast<unsigned long long>(xh) << 32 | xl));
    b = __longlong_as_double(static_cast<long long>(static_cast<unsigned long long>(yh) << 32 | yl));
}

constexpr int wave_log2(int v) { return v <= 1 ? 0 : 1 + wave_log2(v / 2); }

// Digit swap after a stage: register bits RB-1.. (NB of them, from the top) change
// places with the lane bits at distances D, D/2, ...
template <typename V, int PF, int RBIT, int NB, int D> __device__ __forceinline__ void digit_swap(V (&v)[PF])
{
    if constexpr (NB > 0) {
#pragma unroll
        for (int m = 0; m < PF; ++m)
            if (!(m & RBIT)) {
                lane_swap<D>(v[m].x, v[m | RBIT].x);
                lane_swap<D>(v[m].y, v[m | RBIT].y);
            }
        digit_swap<V, PF, RBIT / 2, NB - 1, D / 2>(v);
    }
}

// A stage over sub-transforms of M points: radix RS = min(PF, M) over the top bits
// of the register index, PF/RS of them per thread; TB lane bits are still to come,
// the next at lane distance D.
template <int PF, int M> constexpr int wave_radix() { return M < PF ? M : PF; }
// Twiddles held per thread: RS - 1 for every stage but the last.
template <int N, int PF> __host__ __device__ constexpr int wave_tw_regs()
{
    int n = 0;
    for (int m = N; m > PF; m /= PF) n += PF - 1;
    return n;
}

template <typename R, int N, int PF, int M, int AT, int TOT>
__device__ __forceinline__ void wave_tw_load(Phasor<R> (&w)[TOT], int t, const Phasor<R> *__restrict__ tw)
{
    if constexpr (M > PF) {
        const int q = t & (M / PF - 1);
#pragma unroll
        for (int r = 1; r < PF; ++r) w[AT + r - 1] = tw[tw_index(PF, M / PF, q) + r - 1];
        wave_tw_load<R, N, PF, M / PF, AT + PF - 1>(w, t, tw);
    }
}

// Digits of the final position: register index m of lane t holds bin wave_bin(t) + ...
// The last stage has radix RL = M <= PF over the top register bits; the low
// register bits (PF/RL of them) then still hold the digit that came from the lanes.
template <typename R, int N, int PF, int M, int AT, int D, int TOT>
__device__ __forceinline__ void wave_fwd(cplx<R> (&v)[PF], const Phasor<R> (&w)[TOT])
{
    using V = cplx<R>;
    if constexpr (M > PF) {
        dft<PF, -1>(v);
#pragma unroll
        for (int r = 1; r < PF; ++r) v[r] = pmul(v[r], w[AT + r - 1]);
        constexpr int NB = wave_log2(M / PF < PF ? M / PF : PF);
        digit_swap<V, PF, PF / 2, NB, D>(v);
        wave_fwd<R, N, PF, M / PF, AT + PF - 1, (D >> NB)>(v, w);
    } else {
        // radix M over the top register bits, PF/M butterflies
#pragma unroll
        for (int u = 0; u < PF / M; ++u) {
            V x[M];
#pragma unroll
            for (int r = 0; r < M; ++r) x[r] = v[u + r * (PF / M)];
            dft<M, -1>(x);
#pragma unroll
            for (int r = 0; r < M; ++r) v[u + r * (PF / M)] = x[r];
        }
    }
}

template <typename R, int N, int PF, int M, int AT, int D, int TOT>
__device__ __forceinline__ void wave_inv(cplx<R> (&v)[PF], const Phasor<R> (&w)[TOT])
{
    using V = cplx<R>;
    if constexpr (M > PF) {
        constexpr int NB = wave_log2(M / PF < PF ? M / PF : PF);
        wave_inv<R, N, PF, M / PF, AT + PF - 1, (D >> NB)>(v, w);
        digit_swap<V, PF, PF / 2, NB, D>(v);
#pragma unroll
        for (int r = 1; r < PF; ++r) v[r] = pmul<true>(v[r], w[AT + r - 1]);
        dft<PF, +1>(v);
    } else {
#pragma unroll
        for (int u = 0; u < PF / M; ++u) {
            V x[M];
#pragma unroll
            for (int r = 0; r < M; ++r) x[r] = v[u + r * (PF / M)];
            dft<M, +1>(x);
#pragma unroll
            for (int r = 0; r < M; ++r) v[u + r * (PF / M)] = x[r];
        }
    }
}

// Bin held by register m of lane index t (0 <= t < N/PF) after wave_fwd.
template <int N, int PF, int M = N> __device__ __forceinline__ int wave_bin(int t, int m)
{
    if constexpr (M > PF) {
        // the first stage's output digit now sits in the lane bits it was swapped into,
        // and, where fewer than log2 PF lane bits were left, in the low register bits
        constexpr int rest = M / PF;
        constexpr int NB = wave_log2(rest < PF ? rest : PF), PB = wave_log2(PF);
        const int top = t / (rest >> NB) & ((1 << NB) - 1);
        const int digit = top << (PB - NB) | (m & ((1 << (PB - NB)) - 1));
        return digit + PF * wave_bin<N, PF, rest>(t & ((rest >> NB) - 1), m);
    } else {
        return m >> (wave_log2(PF) - wave_log2(M));
    }
}

} // namespace opo
