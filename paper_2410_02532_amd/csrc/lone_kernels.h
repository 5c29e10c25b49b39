// lone_kernels.h -- the z-steps of handles too small to fill the chip.
//
// A handle of one instance or a few runs two dependent launches per z-step
// (column and row pass), and each launch lasts about the serial time of one tile:
// what bounds it is the chain of dependent memory accesses and exchanges, not
// throughput. In the general column tile that chain was the tile's instance, its
// descriptor, the fields, then the four-step twiddles, the FP64 coupling phasors, and
// one twiddle load after every barrier of the transforms. Here everything a tile needs
// is issued at its start: descriptors come with the kernel arguments, coupling
// coefficients from a table, and the fields, four-step twiddles, propagator
// and the butterfly twiddles of every stage are loaded into registers together (one
// wave per SIMD has 512; nothing spills). A column tile is one wave that exchanges
// between its lanes in registers; a row tile is one row, whose exchanges alternate
// between two LDS buffers with one barrier each.
//
// Measured per z-step (MI355X, us, two launches of which an empty one costs 1.55):
// one 2^14 instance 12.7 -> 7.5 in FP32 and 13.6 -> 7.8 in FP64, three two-wave 2^12
// instances 12.5 -> 6.1 (shapes that team_pass has taken over, team_kernels.h), one 2^16
// 15.9 -> 10.8, one 2^18 28.3 -> 21.6. With the exchanges of the columns through LDS (256 threads, a barrier each) the 2^14 instance
// took 9.5: a radix-2 stage then lasted about 590 cycles, four fifths of them waiting.
#pragma once
#include "coupling_table.h"
#include "schedule.h"
#include "wave_fft.h"

namespace opo {

struct LoneColumnInst {
    long long off;        // first sample of the instance
    long long w4_off;     // its four-step twiddle table
    int n1, nt;
    int log2n2;
    int kind;             // see half_step
    int index;            // instance (couplings)
};

// Tiles of a launch over instances of uneven size, one after another along the grid:
// first[q] is the first tile of instance q, the largest value past the last. (Otherwise
// each instance takes a layer of the grid, as long as the largest one's. About 0.35 ns for
// each idle workgroup of those layers, against 0.3 to 0.8 us for the search here: with more
// than kLoneMaxIdle of them, in the column and row launch together, the search is the cheaper.
// Us a z-step, layers / search: FP32, a 2^18 and 40 2^10 instances 40.6 / 23.0, a 2^18 and
// eight 2^12 (9424 idle) 24.9 / 22.4, a 2^17 and eight 2^12 (5280) 15.8 / 16.2; FP64 the same
// two handles (6816, 5280) 31.3 / 32.2 and 19.6 / 20.4.)
constexpr unsigned kLoneMaxIdle = 7168;
struct LoneTiles {
    static_assert(kLoneMax % 8 == 0, "searched eight at a time");
    unsigned first[kLoneMax];

    // the instance of workgroup `tile`, which becomes its tile in the instance
    __device__ __forceinline__ int find(unsigned &tile) const
    {
        int q = -1;
        unsigned start = 0;
        for (int c = 0; c < kLoneMax && tile >= first[c]; c += 8) {   // the larger instances come first
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const bool past = tile >= first[c + k];
                q += past;
                start = past ? first[c + k] : start;
            }
        }
        tile -= start;
        return q;
    }
};

template <typename R> struct LoneColumnArgs {
    cplx<R> *state;
    const Phasor<R> *tw, *w4tab;
    const int *counter;   // [2] stop flag, see StepArgs
    const Coupling<R> *coef;   // couplings of this launch, per instance
    int flags;            // A_INV | A_RK_PREV, A_RK_THIS | A_FWD, or both
    int spread;           // see lone_col_pf
    LoneColumnInst inst[kLoneMax];
};

struct LoneRowInst {
    long long off;        // first sample of the instance
    long long disp_off;   // its propagator table of this step size
    int rows;             // rows of all fields (nf n2), contiguous
    int log2n1;
};

template <typename R> struct LoneRowArgs {
    cplx<R> *state;
    const Phasor<R> *tw, *disp;
    const int *counter;
    LoneRowInst inst[kLoneMax];
};

// ---- FFT on preloaded twiddles
template <int N, int PF, int P = 1> __host__ __device__ constexpr int tw_regs()
{
    if constexpr (P >= N) return 0;
    else {
        constexpr int RS = stage_radix<N, PF, P, N>();
        return (P > 1 ? PF / RS * (RS - 1) : 0) + tw_regs<N, PF, P * RS>();
    }
}

template <typename R, int N, int PF, int P, int AT, int TOT>
__device__ __forceinline__ void tw_load(Phasor<R> (&w)[TOT], int t, const Phasor<R> *__restrict__ tw)
{
    if constexpr (P < N) {
        constexpr int RS = stage_radix<N, PF, P, N>();
        constexpr int NBT = PF / RS, STRIDE = N / PF;
        if constexpr (P > 1) {
#pragma unroll
            for (int u = 0; u < NBT; ++u) {
                const int k = (t + u * STRIDE) & (P - 1);
                const Phasor<R> *q = tw + tw_index(RS, P, k);
#pragma unroll
                for (int r = 1; r < RS; ++r) w[AT + u * (RS - 1) + r - 1] = q[r - 1];
            }
        }
        tw_load<R, N, PF, P * RS, AT + (P > 1 ? NBT * (RS - 1) : 0)>(w, t, tw);
    }
}

// reg_fft of one transform with the twiddles of every stage in w. Exchange e of a tile
// uses LDS buffer e mod 2 (lds and lds + half): its writes follow the barrier of
// exchange e - 1, which every thread reaches after its reads of exchange e - 2 from the
// same buffer. E counts the exchanges of the tile before this transform. The positions
// of a thread differ in disjoint bit fields, so lds_index splits into the thread's part
// and a constant.
template <typename R, int N, int PF, int DIR, bool WAVE, int E, int P, int AT, int TOT>
__device__ __forceinline__ void fft_pre_from(cplx<R> (&v)[PF], cplx<R> *lds, int half, int t, const Phasor<R> (&w)[TOT])
{
    if constexpr (P < N) {
        using V = cplx<R>;
        constexpr int RS = stage_radix<N, PF, P, N>();
        constexpr int NBT = PF / RS, STRIDE = N / PF;
        constexpr bool LAST = P * RS == N;
        V *s = lds + (E & 1) * half;
#pragma unroll
        for (int u = 0; u < NBT; ++u) {
            V x[RS];
#pragma unroll
            for (int r = 0; r < RS; ++r) x[r] = v[u + r * NBT];
            if constexpr (P > 1) {
#pragma unroll
                for (int r = 1; r < RS; ++r) x[r] = pmul<(DIR > 0)>(x[r], w[AT + u * (RS - 1) + r - 1]);
            }
            dft<RS, DIR>(x);
            if constexpr (LAST) {
#pragma unroll
                for (int r = 0; r < RS; ++r) v[u + r * NBT] = x[r];
            } else {
                const int i = t + u * STRIDE;
                const int k = i & (P - 1);
                V *o = s + lds_index<R>((i - k) * RS + k);
#pragma unroll
                for (int r = 0; r < RS; ++r) o[lds_index<R>(r * P)] = x[r];
            }
        }
        if constexpr (!LAST) {
            if constexpr (WAVE) wave_lds_sync(); else lds_sync();
            const V *q = s + lds_index<R>(t);
#pragma unroll
            for (int m = 0; m < PF; ++m) v[m] = q[lds_index<R>(m * STRIDE)];
            if constexpr (WAVE) wave_lds_sync();
        }
        fft_pre_from<R, N, PF, DIR, WAVE, E + 1, P * RS, AT + (P > 1 ? NBT * (RS - 1) : 0)>(v, lds, half, t, w);
    }
}

// Exchanges of one transform.
template <int N, int PF, int P = 1> __host__ __device__ constexpr int fft_exchanges()
{
    if constexpr (P >= N) return -1;
    else return 1 + fft_exchanges<N, PF, P * stage_radix<N, PF, P, N>()>();
}

// ---- column tile: one wave, 64/T columns with T = N/PF lanes each
constexpr int kLoneMinLog2N2 = 4, kLoneMaxLog2N2 = 7;
// Samples per thread: 2 (radix 2) up to columns of 2^5, and for columns of 2^6 while
// the launch then has at most one wave per SIMD of the chip (`spread`): the RK4 of two
// points instead of four is 1700 cycles less to wait for than the three more radix-2
// stages (one 2^16 instance 12.1 -> 11.5 us a z-step, FP64 14.6 -> 13.8); with more waves
// the extra stages cost more (rows of 2^12, 2048 waves, 22.5 -> 23.0; five 2^16 instances
// in FP64 31.7 -> 35.4).
constexpr int kLoneSpreadWaves = 1024;
constexpr int lone_col_pf(int ln2, bool spread) { return ln2 <= 5 ? 2 : ln2 == 6 ? (spread ? 2 : 4) : 8; }
constexpr int lone_cols(int ln2, bool spread) { return 64 * lone_col_pf(ln2, spread) >> ln2; }

// What a column tile computes, from its samples and four-step and stage twiddles.
// (flags stay a run-time value in every kernel, so that all of them run, and round in,
// the same instructions.)
template <typename R, int N, int PF, int NF, int TW>
__device__ __forceinline__ void lone_column_math(cplx<R> (&v)[NF][PF], const Phasor<R> (&w4)[PF],
                                                 const Phasor<R> (&w)[TW], int kind, const ImagCoupling<R> &imag,
                                                 const Coupling<R> *coef, int flags)
{
    if (flags & A_INV) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
#pragma unroll
            for (int m = 0; m < PF; ++m) v[f][m] = pmul<true>(v[f][m], w4[m]);
            wave_inv<R, N, PF, N, 0, 32>(v[f], w);
        }
    }
    if (flags & A_RK_PREV) half_step<R, NF, PF>(v, kind, imag, coef, 0);
    if (flags & A_RK_THIS) half_step<R, NF, PF>(v, kind, imag, coef, 1);
    if (flags & A_FWD) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            wave_fwd<R, N, PF, N, 0, 32>(v[f], w);
#pragma unroll
            for (int m = 0; m < PF; ++m) v[f][m] = pmul(v[f][m], w4[m]);
        }
    }
}

template <typename R, int LN2, int NF, int PF>
__device__ __forceinline__ void lone_column_tile(const LoneColumnArgs<R> &a, const LoneColumnInst &d, unsigned b)
{
    using V = cplx<R>;
    constexpr int N = 1 << LN2, T = N / PF, COLS = 64 / T;
    constexpr int TW = wave_tw_regs<N, PF>();
    const int flags = a.flags;
    const int c = threadIdx.x % COLS, t = threadIdx.x / COLS;
    const unsigned n1 = d.n1, nt = d.nt, tiles = n1 / COLS;
    if (b >= tiles) return;          // a layer longer than this instance
    // workgroups are dealt to the eight XCDs in turn: neighbouring tiles, which share
    // the cache lines of their columns, go to the same one
    const unsigned tile = tiles >= 8 ? (b & 7) * (tiles >> 3) + (b >> 3) : b;
    const int kind = d.kind;
    const Coupling<R> *coef = a.coef + d.index;
    V *g = a.state + d.off;
    const Phasor<R> *w4t = a.w4tab + d.w4_off;
    V v[NF][PF];
    Phasor<R> w4[PF], w[TW];
    // register m: row wave_bin(t, m) of the transform where a row pass left it or will
    // take it, sample t + m T otherwise
    unsigned q[PF], qo[PF];
#pragma unroll
    for (int m = 0; m < PF; ++m) {
        const unsigned bin = tile * COLS + c + n1 * wave_bin<N, PF>(t, m), smp = tile * COLS + c + n1 * (t + m * T);
        q[m] = flags & A_INV ? bin : smp;
        qo[m] = flags & A_FWD ? bin : smp;
    }
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int m = 0; m < PF; ++m) v[f][m] = el32(g, q[m] + f * nt);
#pragma unroll
    for (int m = 0; m < PF; ++m) w4[m] = el32(w4t, flags & A_FWD ? qo[m] : q[m]);
    wave_tw_load<R, N, PF, N, 0>(w, t, a.tw);
    const bool stopped = a.counter[2] != 0;   // see column_tile
    const ImagCoupling<R> imag(coef);
    lone_column_math<R, N, PF, NF>(v, w4, w, kind, imag, coef, flags);
    if (stopped) return;
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int m = 0; m < PF; ++m) el32(g, qo[m] + f * nt) = v[f][m];
}

template <typename R, int NF>
__device__ __forceinline__ void lone_column_dispatch(const LoneColumnArgs<R> &a, const LoneColumnInst &d, unsigned b)
{
    switch (d.log2n2) {
    case 4: return lone_column_tile<R, 4, NF, 2>(a, d, b);
    case 5: return lone_column_tile<R, 5, NF, 2>(a, d, b);
    case 6: return a.spread ? lone_column_tile<R, 6, NF, 2>(a, d, b) : lone_column_tile<R, 6, NF, 4>(a, d, b);
    default: return lone_column_tile<R, 7, NF, 8>(a, d, b);
    }
}

template <typename R, int NF> __global__ __launch_bounds__(64) void lone_column(LoneColumnArgs<R> a)
{
    lone_column_dispatch<R, NF>(a, a.inst[blockIdx.y], blockIdx.x);
}
template <typename R, int NF> __global__ __launch_bounds__(64) void lone_column_uneven(LoneColumnArgs<R> a, LoneTiles t)
{
    unsigned b = blockIdx.x;
    const int q = t.find(b);
    lone_column_dispatch<R, NF>(a, a.inst[q], b);
}

// ---- row tile: whole rows, PF samples per thread. A workgroup holds one row where it
// takes 64 threads or more, else as many as fill a wave: the loads of a row (field,
// propagator and twiddles, 26 KB at 512 points) are bound by the CU's L1, so fewer
// rows per CU are faster as long as CUs are idle.
constexpr int kLoneMinLog2N1 = 5;
// 1024 points take 4 samples and 256 threads (five radix-4 stages) instead of 8 and 128:
// one 2^16 instance 12.4 -> 12.1 us a z-step; 4096 points 8 and 512 threads instead of 16
// (radix 16) and 256: one 2^18 instance 23.7 -> 22.5. 2048 points with 4 were no faster.
constexpr int lone_row_pf(int ln1) { return ln1 <= 7 || ln1 == 10 ? 4 : 8; }
constexpr int lone_row_threads(int ln1) { return (1 << ln1) / lone_row_pf(ln1); }

template <typename R, int LN1>
__device__ __forceinline__ void lone_row_tile(const LoneRowArgs<R> &a, const LoneRowInst &d, unsigned b, cplx<R> *s)
{
    using V = cplx<R>;
    constexpr int N = 1 << LN1, PF = lone_row_pf(LN1), T = N / PF;
    constexpr int TW = tw_regs<N, PF>(), X = fft_exchanges<N, PF>();
    constexpr bool WAVE = T <= 64;   // a row's threads lie within one wavefront
    const int rows = blockDim.x / T, r = threadIdx.x / T, t = threadIdx.x % T;
    if (static_cast<int>(b) * rows >= d.rows) return;   // a layer longer than this instance
    const int row = b * rows + r;
    const bool act = row < d.rows;
    const unsigned q0 = static_cast<unsigned>(act ? row : 0) * N + t;
    V *g = a.state + d.off;
    const Phasor<R> *h = a.disp + d.disp_off;
    V v[PF];
    Phasor<R> hr[PF], w[TW];
#pragma unroll
    for (int m = 0; m < PF; ++m) v[m] = el32(g, q0 + m * T);
    tw_load<R, N, PF, 1, 0>(w, t, a.tw);
#pragma unroll
    for (int m = 0; m < PF; ++m) hr[m] = el32(h, q0 + m * T);
    const bool stopped = a.counter[2] != 0;
    s += lds_index<R>(r * N);         // rows of a workgroup side by side
    const int half = lds_elems<R>(static_cast<int>(blockDim.x) * PF);
    fft_pre_from<R, N, PF, -1, WAVE, 0, 1, 0>(v, s, half, t, w);
#pragma unroll
    for (int m = 0; m < PF; ++m) v[m] = pmul(v[m], hr[m]);
    fft_pre_from<R, N, PF, +1, WAVE, X, 1, 0>(v, s, half, t, w);
    if (stopped || !act) return;
#pragma unroll
    for (int m = 0; m < PF; ++m) el32(g, q0 + m * T) = v[m];
}

// Rows of 2^5..2^HI points: HI = 9, or 12 (the longer rows hold more samples and
// twiddles per thread, one wave per SIMD).
template <typename R, int HI>
__device__ __forceinline__ void lone_row_dispatch(const LoneRowArgs<R> &a, const LoneRowInst &d, unsigned b, cplx<R> *s)
{
    switch (d.log2n1) {
    case 5: return lone_row_tile<R, 5>(a, d, b, s);
    case 6: return lone_row_tile<R, 6>(a, d, b, s);
    case 7: return lone_row_tile<R, 7>(a, d, b, s);
    case 8: return lone_row_tile<R, 8>(a, d, b, s);
    case 9: return lone_row_tile<R, 9>(a, d, b, s);
    }
    if constexpr (HI > 9) {
        switch (d.log2n1) {
        case 10: return lone_row_tile<R, 10>(a, d, b, s);
        case 11: return lone_row_tile<R, 11>(a, d, b, s);
        case 12:
            if constexpr (kMaxLog2N1<R> >= 12) return lone_row_tile<R, 12>(a, d, b, s);
        }
    }
}

template <typename R, int HI> __global__ __launch_bounds__(HI > 9 ? 512 : 256) void lone_row(LoneRowArgs<R> a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    lone_row_dispatch<R, HI>(a, a.inst[blockIdx.y], blockIdx.x, reinterpret_cast<cplx<R> *>(lds_raw));
}
template <typename R, int HI>
__global__ __launch_bounds__(HI > 9 ? 512 : 256) void lone_row_uneven(LoneRowArgs<R> a, LoneTiles t)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    unsigned b = blockIdx.x;
    const int q = t.find(b);
    lone_row_dispatch<R, HI>(a, a.inst[q], b, reinterpret_cast<cplx<R> *>(lds_raw));
}

} // namespace opo
