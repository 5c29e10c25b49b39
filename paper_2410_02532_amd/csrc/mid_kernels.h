// mid_kernels.h -- the z-steps of batches that fill the chip, inside a pass.
//
// mixed_pass without what only the ends of a pass and the round-trip boundary need.
// Those launches are bound by VALU issue (73 % of the cycles at 791 lane-instructions
// per field-point-step on the batched sweep) and, in FP64, by the three workgroups a CU
// holds at 152 registers. Here the column transforms exchange between the lanes of one
// wave (no LDS, no barrier), the flags of the boundary, the bounds checks and the FP64
// coupling phasors are gone (the couplings of every step come from a table), and one
// map entry names a workgroup's instance and tile (two dependent loads before the
// fields instead of three).
//
// Measured (MI355X, ms per round trip of the 256-instance sweeps of 2^12..2^16, with the
// launch order and the row shapes that followed, both timed in turn on one card): FP32
// 18.6 -> 17.2, two waves 13.9 -> 12.1, FP64 37.3 -> 29.9 (another card 17.0, 11.8, 29.7
// after; cards differ by some percent in FP32). The FP32 launch takes 3.70e7 wave instructions (742
// lane-instructions) and issues VALU 75 % of its cycles at four workgroups per CU (five
// changed nothing); about 9 us of it are its ramp and tail. The FP64 launch issues VALU
// 37 % of its cycles and moves its fields at 4.3 TB/s (a large copy: 4.85): memory bound.
#pragma once
#include "coupling_table.h"
#include "wave_fft.h"

namespace opo {

struct MidInst {
    long long off;        // first sample of the instance
    long long w4_off;     // its four-step twiddle table
    long long disp_off;   // its propagator table
    int nt, n1;
    int log2n1, log2n2;
    int rows;             // rows of all fields (nf n2), contiguous
    int kind;             // 0: dk = 0 (couplings i c); 1: general couplings; 2: Kerr terms
};

// A workgroup's tile: instance (-1: none), and column tile (>= 0) or row tile -1-code.
struct MidTile {
    int inst, code;
};

template <typename R> struct MidArgs {
    cplx<R> *state;
    const Phasor<R> *tw, *w4tab, *disp;
    const int *counter;       // [2] stop flag, see StepArgs
    const MidInst *inst;
    const Coupling<R> *coef;  // couplings of this launch's column tiles, per instance
    const MidTile *map;
    int flags;                // column tiles: A_INV | A_RK_PREV, A_RK_THIS | A_FWD, or both
    int disp_sel;             // row tiles: propagator table of this step size (0 or 1)
};

// ---- column tile: four waves of 64/T columns each (T = N/PF lanes a column)
constexpr int kMidMinLog2N2 = 4, kMidMinLog2N1 = 5;
constexpr int mid_col_pf(int ln2) { return ln2 <= 5 ? 2 : 4; }
// FP32 rows of 1024 and 2048 points take 16 samples a thread (radix-16 stages, one stage
// and one exchange less): the batched sweep 16.7 -> 16.4 ms, two waves 12.0 -> 11.7. The
// kernel then holds 128 registers (four workgroups per CU) instead of 92, which costs
// nothing here (mixed_pass lost 2.5 % with it). Rows of 256 with 16 lost 0.6 %, columns of
// 2^6 with 8 samples (168 registers, spills) 8 %.
template <typename R> constexpr int mid_row_pf(int ln1)
{
    return sizeof(R) == 4 && (ln1 == 10 || ln1 == 11) ? 16 : row_pf<R>(ln1);
}
template <typename R> constexpr int mid_rows(int ln1) { return kThreads * mid_row_pf<R>(ln1) >> ln1; }
template <typename R> constexpr int mid_cols(int ln2)
{
    return ln2 <= 6 ? kThreads * mid_col_pf(ln2) >> ln2 : col_cols<R>(ln2);
}

template <typename R, int LN2, int NF>
__device__ __forceinline__ void mid_column_tile(const MidArgs<R> &a, const MidInst &d, const Coupling<R> &cp, int tile)
{
    using V = cplx<R>;
    constexpr int N = 1 << LN2, PF = mid_col_pf(LN2), T = N / PF, COLS = 64 / T;
    constexpr int TW = wave_tw_regs<N, PF>();
    const int flags = a.flags;
    const int lane = threadIdx.x & 63, c = lane % COLS, t = lane / COLS;
    const unsigned n1 = d.n1, nt = d.nt;
    const unsigned j1 = tile * mid_cols<R>(LN2) + (threadIdx.x >> 6) * COLS + c;
    const int kind = d.kind;
    V *g = a.state + d.off;
    const Phasor<R> *w4t = a.w4tab + d.w4_off;
    const bool stopped = a.counter[2] != 0;   // see column_tile
    V v[NF][PF];
    // register m: row wave_bin(t, m) of the transform where a row pass left it or will
    // take it, sample t + m T otherwise
    auto at = [&](bool freq, int m) {
        return j1 + n1 * (freq ? wave_bin<N, PF>(t, m) : t + m * T);
    };
#pragma unroll
    for (int m = 0; m < PF; ++m) {
        const unsigned q = at(flags & A_INV, m);
#pragma unroll
        for (int f = 0; f < NF; ++f) v[f][m] = el32(g, q + f * nt);
    }
    Phasor<R> w[TW];
    wave_tw_load<R, N, PF, N, 0>(w, t, a.tw);
    if (flags & A_INV) {
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            const Phasor<R> w4 = el32(w4t, at(true, m));
#pragma unroll
            for (int f = 0; f < NF; ++f) v[f][m] = pmul<true>(v[f][m], w4);
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) wave_inv<R, N, PF, N, 0, 32>(v[f], w);
    }
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        if (!(flags & (which ? A_RK_THIS : A_RK_PREV))) continue;
#pragma unroll
        for (int m = 0; m < PF; ++m)
            rk4_fields<R, NF>(cp, which, kind == 0, kind == 2, v[0][m], v[1][m], v[NF - 1][m]);
    }
    if (flags & A_FWD) {
        // the twiddles again from L1 (the opaque index keeps them from being held across
        // the RK4: 92 registers instead of 116 in FP32, 164 instead of 188 in FP64)
        int tz = t;
        asm volatile("" : "+v"(tz));
        wave_tw_load<R, N, PF, N, 0>(w, tz, a.tw);
#pragma unroll
        for (int f = 0; f < NF; ++f) wave_fwd<R, N, PF, N, 0, 32>(v[f], w);
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            const Phasor<R> w4 = el32(w4t, at(true, m));
#pragma unroll
            for (int f = 0; f < NF; ++f) v[f][m] = pmul(v[f][m], w4);
        }
    }
    if (stopped) return;
#pragma unroll
    for (int m = 0; m < PF; ++m) {
        const unsigned q = at(flags & A_FWD, m);
#pragma unroll
        for (int f = 0; f < NF; ++f) el32(g, q + f * nt) = v[f][m];
    }
}

// Longer columns (2^7 and 2^8 points, of grids whose rows are at their longest): the
// tile of column_tile, exchanging through LDS, without its flags and checks (186 registers,
// two workgroups per CU: 8 x 2^20 in FP32 31.7 -> 30.9 ms a round trip; held to 168 for
// three it spills and took 31.6).
template <typename R, int LN2, int NF>
__device__ __forceinline__ void mid_long_column_tile(const MidArgs<R> &a, const MidInst &d, const Coupling<R> &cp,
                                                     int tile, cplx<R> *s)
{
    using V = cplx<R>;
    constexpr int N = 1 << LN2, PF = col_pf<R>(LN2), COLS = col_cols<R>(LN2), T = N / PF;
    const int flags = a.flags, kind = d.kind;
    const int c = threadIdx.x % COLS, t = threadIdx.x / COLS;
    const unsigned n1 = d.n1, nt = d.nt, q0 = tile * COLS + c + n1 * t, step = n1 * T;
    V *g = a.state + d.off;
    const Phasor<R> *w4t = a.w4tab + d.w4_off;
    const bool stopped = a.counter[2] != 0;   // see column_tile
    V v[NF][PF];
#pragma unroll
    for (int m = 0; m < PF; ++m)
#pragma unroll
        for (int f = 0; f < NF; ++f) v[f][m] = el32(g, q0 + m * step + f * nt);
    int base[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) base[f] = f * col_lds_row<R>(LN2) * N + c;
    if (flags & A_INV) {
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            const Phasor<R> w4 = el32(w4t, q0 + m * step);
#pragma unroll
            for (int f = 0; f < NF; ++f) v[f][m] = pmul<true>(v[f][m], w4);
        }
        column_fft<R, LN2, PF, NF, +1, COLS>(v, s, base, t, a.tw);
    }
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        if (!(flags & (which ? A_RK_THIS : A_RK_PREV))) continue;
#pragma unroll
        for (int m = 0; m < PF; ++m)
            rk4_fields<R, NF>(cp, which, kind == 0, kind == 2, v[0][m], v[1][m], v[NF - 1][m]);
    }
    if (flags & A_FWD) {
        column_fft<R, LN2, PF, NF, -1, COLS>(v, s, base, t, a.tw);
#pragma unroll
        for (int m = 0; m < PF; ++m) {
            const Phasor<R> w4 = el32(w4t, q0 + m * step);
#pragma unroll
            for (int f = 0; f < NF; ++f) v[f][m] = pmul(v[f][m], w4);
        }
    }
    if (stopped) return;
#pragma unroll
    for (int m = 0; m < PF; ++m)
#pragma unroll
        for (int f = 0; f < NF; ++f) el32(g, q0 + m * step + f * nt) = v[f][m];
}

// ---- row tile: row_rows whole rows
template <typename R, int LN1>
__device__ __forceinline__ void mid_row_tile(const MidArgs<R> &a, const MidInst &d, int tile, cplx<R> *s)
{
    using V = cplx<R>;
    constexpr int N = 1 << LN1, PF = mid_row_pf<R>(LN1), ROWS = mid_rows<R>(LN1), T = N / PF;
    constexpr bool WAVE = T <= OPO_ROW_WAVE_MAX;
    const int r = threadIdx.x / T, t = threadIdx.x % T;
    const int row = tile * ROWS + r;
    const bool act = row < d.rows;
    const unsigned q0 = static_cast<unsigned>(act ? row : 0) * N + t;
    V *g = a.state + d.off;
    const bool stopped = a.counter[2] != 0;
    const Phasor<R> *h = a.disp + d.disp_off + static_cast<long long>(a.disp_sel) * d.rows * N;
    V v[1][PF];
#pragma unroll
    for (int m = 0; m < PF; ++m) v[0][m] = el32(g, q0 + m * T);
    const int base[1] = {r * N};
    reg_fft<R, N, PF, 1, -1, 1, 2048, false, WAVE>(v, s, base, t, a.tw);
#pragma unroll
    for (int m = 0; m < PF; ++m) v[0][m] = pmul(v[0][m], el32(h, q0 + m * T));
    reg_fft<R, N, PF, 1, +1, 1, 2048, false, WAVE>(v, s, base, t, a.tw);
    if (stopped || !act) return;
#pragma unroll
    for (int m = 0; m < PF; ++m) el32(g, q0 + m * T) = v[0][m];
}

template <typename R, int L, int HI>
__device__ __forceinline__ void mid_row_dispatch(const MidArgs<R> &a, const MidInst &d, int tile, cplx<R> *s)
{
    if (d.log2n1 == L) mid_row_tile<R, L>(a, d, tile, s);
    else if constexpr (L < HI) mid_row_dispatch<R, L + 1, HI>(a, d, tile, s);
}

// Rows of 2^LO..2^HI points: 5..11, or 12 (FP32).
template <typename R, int HI, int CR> constexpr int mid_min_blocks() { return sizeof(R) == 4 && HI <= 11 && CR == 0 ? 4 : 1; }

// CR: columns of 2^4..2^6 points (0), 2^7 (1) or 2^8 (2).
template <typename R, int LO, int HI, int NF, int CR>
__global__ __launch_bounds__(kThreads, (mid_min_blocks<R, HI, CR>())) void mid_pass(MidArgs<R> a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const MidTile mt = a.map[blockIdx.x];
    if (mt.inst < 0) return;
    const MidInst &d = a.inst[mt.inst];
    if (mt.code >= 0) {
        const Coupling<R> &cp = a.coef[mt.inst];
        if constexpr (CR > 0)
            return mid_long_column_tile<R, 6 + CR, NF>(a, d, cp, mt.code, reinterpret_cast<cplx<R> *>(lds_raw));
        else switch (d.log2n2) {
        case 4: return mid_column_tile<R, 4, NF>(a, d, cp, mt.code);
        case 5: return mid_column_tile<R, 5, NF>(a, d, cp, mt.code);
        default: return mid_column_tile<R, 6, NF>(a, d, cp, mt.code);
        }
    }
    mid_row_dispatch<R, LO, HI>(a, d, -1 - mt.code, reinterpret_cast<cplx<R> *>(lds_raw));
}

// The mixed launches at the ends of a round trip where mid_pass's rows differ from
// mixed_pass's (FP32 rows of 1024 and 2048 points, mid_row_pf): column tiles with the
// flags of the boundary (column_tile, global tile numbers) and row tiles of mid_pass. The
// halves of a batch are a launch apart, so only one half's rows of a step fall into such a
// launch: with the same transform in both, equal members agree bit for bit whichever half
// they were dealt to.
template <typename R, int NF>
__global__ __launch_bounds__(kThreads, OPO_MIXED_MIN_BLOCKS) void edge_pass(StepArgs<R> ac, MidArgs<R> ar)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    __shared__ Coupling<R> cpl;
    __shared__ double red[3 * kThreads / 64];
    cplx<R> *s = reinterpret_cast<cplx<R> *>(lds_raw);
    const MidTile mt = ar.map[blockIdx.x];
    if (mt.inst < 0) return;
    if (mt.code >= 0)
        column_dispatch<R, kColRanges[0][0], kColRanges[0][1], NF, false>(ac, ac.inst[mt.inst], mt.code, s, &cpl, red);
    else
        mid_row_dispatch<R, 5, 11>(ar, ar.inst[mt.inst], -1 - mt.code, s);
}

} // namespace opo
