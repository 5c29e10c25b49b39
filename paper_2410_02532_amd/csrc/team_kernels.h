// team_kernels.h -- the z-steps of small instances in one launch: teams of waves.
//
// The lone kernels spend 3.1 of the 7.5 us of a z-step of one 2^14 instance on two
// launch boundaries, and load the same twiddles and propagator again in every launch.
// team_pass runs all interior phases of a pass in one launch instead: up to kTeamMax
// waves of one XCD form a team for an instance, every wave keeps its column tile's and
// its row tile's tables in registers for the whole pass, and a phase begins when every
// member has flagged the phase before.
//
// Waiting only for waves that run: the members of a team are the waves that have
// arrived when its first wave (the leader) closes it, at the latest kTeamWait after the
// leader came. A member never waits for a wave that may not have started, so a team
// makes progress whatever else the GPU runs; one that closes early is only slower (its
// members then share the tiles out among fewer). The results do not depend on the
// team's size. Workgroups are dealt to the XCDs in turn: those of one class (their number
// modulo eight) share one, and the lists are dealt to the classes. A wave joins the first
// list of its class that nobody has claimed, or that its XCD has and where a place is left.
// A class has as many waves as its lists have places together, so every list gets some,
// wherever its workgroups run. A wait that makes kTeamSpin polls gives up: it raises a flag,
// which the host reads when it has waited for the stream, and the launch ends with fields
// that are not those of the pass.
//
// Coherent without fences: a team's waves share the L2 of the XCD they run on (XCC_ID)
// and the L1 is write-through. Stores are waited for (vmcnt) before the flag is set;
// field and flag loads bypass the L1 (agent scope). Only the claim of a list is a matter
// between XCDs. A device-scope barrier (release and acquire fences) costs 3.9 us among 32
// workgroups (microbench/launch_vs_barrier.hip); an exchange of 12 KB per workgroup
// through flags in one XCD's L2 costs 1.3 us (microbench/flag_exchange.hip).
#pragma once
#include "lone_kernels.h"

namespace opo {

constexpr int kTeamMax = 128;             // waves of a team: one per SIMD of an XCD
constexpr int kTeamWait = 2000;           // ticks of 10 ns the leader waits for members
constexpr int kTeamSpin = 1 << 24;        // polls of a wait before it gives up (about ten seconds)
constexpr int kTeamSealed = 1 << 30;

// Shapes: columns of 2^5 points with rows of 2^5..2^9, columns of 2^6 with rows of 2^9,
// where a full team holds every tile (three waves of 2^15 points have 192 row tiles: in
// turns of 128 waves they ran 9.9 us a z-step against 8.8 of the lone kernels).
// Measured (MI355X, us per z-step of one instance, FP32 / FP64, three waves): before the
// lone kernels, lone kernels, team
//   2^10  10.7 / 9.7  6.1 / 6.3  4.2 / 4.3      2^13  11.7 / 12.3  7.9 / 8.4  5.0 / 5.4
//   2^12  11.5 / 12.0  6.2 / 6.5  4.6 / 4.9     2^14  12.5 / 13.6  7.4 / 7.8  5.7 / 6.1
// eight of 2^14 at once 17.9 / 22.3, 10.9 / 15.3, 5.8 / 6.4; one of 2^15, two waves,
// 13.2 / 13.4, 7.9 / 8.7, 6.3 / 6.8.
constexpr bool team_shape(int log2n2, int log2n1, int nf)
{
    return (log2n2 == 5 && log2n1 >= 5 && log2n1 <= 9) || (log2n2 == 6 && log2n1 == 9 && nf == 2);
}
// A launch of teams has its price: claims, the members' arrival, and with more lists than
// places at once the wait for members that do not come (about 8 us with one list, 16 with
// 16, 40 to 60 with 32 to 48). A pass of at most 2 team_short_steps phases takes a launch a
// phase instead, which gives the same results (a round trip of nz steps has 2 nz - 1 phases,
// an nz-step call of ssfm_propagate 2 nz + 1). `waves` are the places of the fullest class's
// lists. Measured (us a round trip, teams / a launch a phase): FP32, one 2^10, nz 1 27.1 /
// 25.3, nz 2 31.8 / 34.3; one 2^14, nz 2 46.5 / 40.0, nz 4 55.3 / 58.5; 16 of 2^13, nz 2 55.8 /
// 47.1, nz 4 69.1 / 73.8; 32 of 2^12, nz 3 64.5 / 58.9, nz 6 85 / 100; 48 of 2^10, nz 3 53.4 /
// 50.4, nz 4 56.2 / 60.2; 48 of 2^12, whose class fills its second turn of 256 places to an
// eighth, nz 8 178 / 170, nz 12 222 / 253. FP64, one 2^14, nz 2 50.8 / 41.6; 32 of 2^13, nz 3
// 131 / 120, nz 4 150 / 160; 48 of 2^12, nz 3 107 / 108, nz 4 118 / 140. Over 378 such shapes
// and step counts the faster of the two is missed by 0.3 % on average. (Before the lone kernels
// such round trips took as long or longer, but for many FP64 instances and two or three steps:
// 48 of 2^10 35.9 and 45.3, now 43.2 and 55.0; 32 of 2^13 80.4, now 89.0.)
constexpr int team_short_steps(bool f64, int n, int waves)
{
    const int steps = 1 + (waves > kTeamMax ? 1 : 0) + (n <= 4 && waves >= 96 ? 1 : 0);
    if (f64) return steps + n / 32;
    const int places = 2 * kTeamMax, lists = (n + 7) / 8;   // FP32: two waves a SIMD
    int tail = 0;
    if (waves > places) {
        const int at_once = places * lists / waves > 1 ? places * lists / waves : 1;
        const int turns = (lists + at_once - 1) / at_once;
        if (2 * turns * places > 3 * waves) tail = 4;       // the last one mostly empty
    }
    return steps + n / 16 + tail;
}
constexpr int kTeamCols = 4;              // columns per wave: 2^5 points on 16 lanes of 2, 2^6 of 4
constexpr int team_row_pf(int ln1) { return ln1 <= 8 ? 4 : 8; }
constexpr int team_rows(int ln1) { return 64 * team_row_pf(ln1) >> ln1; }   // rows per wave
// Waves of a full team: one for every tile, up to an XCD's.
constexpr int team_want(int n1, int log2n1, int rows)
{
    const int c = n1 / kTeamCols, r = (rows + team_rows(log2n1) - 1) / team_rows(log2n1), w = c > r ? c : r;
    return w < kTeamMax ? w : kTeamMax;
}

// Device memory of a list's team, zeroed before the launch.
struct alignas(128) TeamSync {
    int owner;            // 1 + XCC_ID of the XCD that works on the list
    int join;             // waves arrived, and kTeamSealed
    int size;             // members, once closed
    int pad[29];
    int flag[kTeamMax];   // per member: phases done
};

// Samples of an instance that other waves of the XCD write during the kernel: loads that
// miss the L1 and are served by the XCD's L2.
template <typename R> struct FieldLoad {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ FieldLoad(const cplx<R> *p, unsigned count)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<cplx<R> *>(p), 0, count * sizeof(cplx<R>), 0x00027000))
    {
    }
    __device__ __forceinline__ cplx<R> operator()(unsigned q) const
    {
        constexpr int sc1 = 16;   // agent scope: served by the L2
        cplx<R> v;
        if constexpr (sizeof(R) == 4) {
            const auto u = __builtin_amdgcn_raw_buffer_load_b64(rsrc, q * 8, 0, sc1);
            __builtin_memcpy(&v, &u, 8);
        } else {
            const auto u = __builtin_amdgcn_raw_buffer_load_b128(rsrc, q * 16, 0, sc1);
            __builtin_memcpy(&v, &u, 16);
        }
        return v;
    }
};
struct TeamInst {
    long long off, w4_off, disp_off;
    int nt, n1, log2n1, log2n2;
    int rows;             // rows of all fields
    int kind;             // as LoneColumnInst
    int index;            // instance (couplings)
    int want;             // waves of a full team
};

template <typename R> struct TeamArgs {
    cplx<R> *state;
    const Phasor<R> *tw, *w4tab, *disp;
    const int *counter;       // [2] stop flag, see StepArgs
    const Coupling<R> *coef;  // couplings of step boundary s0 + b at b n + index
    TeamSync *sync;           // per list
    int *failed;              // set when a wait gave up (pinned host memory)
    int n;                    // instances of the handle
    int count;                // lists
    // phases begin .. end - 1: 2 j are the columns at step boundary s0 + j, 2 j + 1 the
    // rows of step s0 + j. The first and the last boundary of a pass (open, close) have
    // only the half-step and the transform on their inner side
    int begin, end, open, close;
    int s0, order;
    int first[9];         // lists first[c] .. first[c + 1] - 1 are dealt to class c
    TeamInst inst[kLoneMax];
};

__device__ __forceinline__ int xcc_id()
{
    return __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 0xf;   // HW_REG_XCC_ID, bits 0..3
}

__device__ __forceinline__ int team_load(const int *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Counts a poll; true when the wait has to be given up.
__device__ __forceinline__ bool team_give_up(int &polls, int *failed)
{
    if ((++polls & 1023) != 0) return false;
    if (polls < kTeamSpin && team_load(failed) == 0) return false;
    __hip_atomic_store(failed, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return true;
}

template <typename R, int LN2, int LN1, int NF>
__device__ __forceinline__ void team_run(const TeamArgs<R> &a, const TeamInst &d, TeamSync *sync, int rank, int size,
                                         cplx<R> *s)
{
    using V = cplx<R>;
    // columns: as lone_column_tile
    constexpr int CN = 1 << LN2, CPF = LN2 == 6 ? 4 : 2, CT = CN / CPF, COLS = 64 / CT;
    // rows: whole rows, RT lanes each
    constexpr int RN = 1 << LN1, RPF = team_row_pf(LN1), RT = RN / RPF, ROWS = 64 / RT;
    constexpr int CTW = wave_tw_regs<CN, CPF>(), RTW = tw_regs<RN, RPF>(), X = fft_exchanges<RN, RPF>();
    const int lane = threadIdx.x;
    const int c = lane % COLS, ct = lane / COLS, r = lane / RT, rt = lane % RT;
    const int tiles_c = d.n1 / COLS, tiles_r = (d.rows + ROWS - 1) / ROWS;
    const unsigned n1 = d.n1, nt = d.nt;
    V *g = a.state + d.off;
    const FieldLoad<R> in(g, NF * nt);
    const Phasor<R> *w4t = a.w4tab + d.w4_off;
    Phasor<R> cw[CTW], w4[CPF], rw[RTW], hr[RPF];
    wave_tw_load<R, CN, CPF, CN, 0>(cw, ct, a.tw);
    tw_load<R, RN, RPF, 1, 0>(rw, rt, a.tw);
    int have_c = -1, have_r = -1;   // tiles whose tables are in registers
    s += lds_index<R>(r * RN);

    // every member has done the phases before ph
    bool gave_up = false;           // then this wave stores NaN
    auto ready = [&](int ph) {
        if (ph == a.begin) return;
        int polls = 0;
        for (;;) {
            const int f0 = lane < size ? team_load(&sync->flag[lane]) : ph;
            const int f1 = size > 64 && lane + 64 < size ? team_load(&sync->flag[lane + 64]) : ph;
            if (__all(f0 >= ph && f1 >= ph)) break;
            if (team_give_up(polls, a.failed)) {
                gave_up = true;
                break;
            }
        }
        asm volatile("" ::: "memory");
    };
    for (int ph = a.begin; ph < a.end; ++ph) {
        const int j = ph >> 1;
        if (ph & 1) {
            const int sel = a.order == 4 && (a.s0 + j) % 3 == 1 ? 1 : 0;
            for (int tile = rank; tile < tiles_r; tile += size) {
                const int row = tile * ROWS + r;
                const bool act = row < d.rows;
                const unsigned q0 = static_cast<unsigned>(act ? row : 0) * RN + rt;
                if (have_r != 2 * tile + sel) {
                    have_r = 2 * tile + sel;
                    const Phasor<R> *h = a.disp + d.disp_off + static_cast<long long>(sel) * NF * d.nt;
#pragma unroll
                    for (int m = 0; m < RPF; ++m) hr[m] = el32(h, q0 + m * RT);
                }
                if (tile == rank) ready(ph);
                V v[RPF];
#pragma unroll
                for (int m = 0; m < RPF; ++m) v[m] = in(q0 + m * RT);
                fft_pre_from<R, RN, RPF, -1, true, 0, 1, 0>(v, s, 0, rt, rw);
#pragma unroll
                for (int m = 0; m < RPF; ++m) v[m] = pmul(v[m], hr[m]);
                fft_pre_from<R, RN, RPF, +1, true, X, 1, 0>(v, s, 0, rt, rw);
                if (gave_up) v[0].x = static_cast<R>(NAN);
                if (act)
#pragma unroll
                    for (int m = 0; m < RPF; ++m) el32(g, q0 + m * RT) = v[m];
            }
        } else {
            const Coupling<R> *coef = a.coef + static_cast<size_t>(j) * a.n + d.index;
            const int flags = (ph == a.open ? 0 : A_INV | A_RK_PREV) | (ph == a.close ? 0 : A_RK_THIS | A_FWD);
            for (int tile = rank; tile < tiles_c; tile += size) {
                // register m: row wave_bin(t, m) of the transform, sample t + m T without one
                unsigned q[CPF], qo[CPF];
#pragma unroll
                for (int m = 0; m < CPF; ++m) {
                    const unsigned bin = tile * COLS + c + n1 * wave_bin<CN, CPF>(ct, m);
                    const unsigned smp = tile * COLS + c + n1 * (ct + m * CT);
                    q[m] = flags & A_INV ? bin : smp;
                    qo[m] = flags & A_FWD ? bin : smp;
                }
                if (have_c != tile) {
                    have_c = tile;
#pragma unroll
                    for (int m = 0; m < CPF; ++m) w4[m] = el32(w4t, flags & A_FWD ? qo[m] : q[m]);
                }
                const ImagCoupling<R> imag(coef);
                if (tile == rank) ready(ph);
                V v[NF][CPF];
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int m = 0; m < CPF; ++m) v[f][m] = in(q[m] + f * nt);
                lone_column_math<R, CN, CPF, NF>(v, w4, cw, d.kind, imag, coef, flags);
                if (gave_up) v[0][0].x = static_cast<R>(NAN);
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int m = 0; m < CPF; ++m) el32(g, qo[m] + f * nt) = v[f][m];
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's stores are in the L2
        if (lane == 0) __hip_atomic_store(&sync->flag[rank], ph + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

template <typename R, int NF>
__device__ __forceinline__ void team_dispatch(const TeamArgs<R> &a, int list, int rank, int size, cplx<R> *s)
{
    const TeamInst &d = a.inst[list];
    TeamSync *sync = a.sync + list;
    if (d.log2n2 == 6) team_run<R, 6, 9, NF>(a, d, sync, rank, size, s);
    else if (d.log2n1 == 5) team_run<R, 5, 5, NF>(a, d, sync, rank, size, s);
    else if (d.log2n1 == 6) team_run<R, 5, 6, NF>(a, d, sync, rank, size, s);
    else if (d.log2n1 == 7) team_run<R, 5, 7, NF>(a, d, sync, rank, size, s);
    else if (d.log2n1 == 8) team_run<R, 5, 8, NF>(a, d, sync, rank, size, s);
    else team_run<R, 5, 9, NF>(a, d, sync, rank, size, s);
}

// AGAIN: a wave that has done with its list joins a further one. FP64 handles whose lists
// have more places than an XCD has SIMDs run it: 40 of 2^12 points, round trips of 20 steps,
// 358 us with a workgroup for every place, the later ones started as SIMDs come free, 240
// so. FP32 without it holds two waves a SIMD (247 -> 180).
template <typename R, int NF, bool AGAIN> __global__ __launch_bounds__(64) void team_pass(TeamArgs<R> a)
{
    __shared__ __align__(16) cplx<R> s[lds_elems<R>(512)];
    if (a.counter[2] != 0) return;   // a round trip of this call was not finite: store nothing
    // (a class without lists has no part: a claim contended by all waves costs 80 ns a wave)
    const int xcc = xcc_id(), cls = blockIdx.x & 7;
    const bool first_lane = threadIdx.x == 0;
    int list = a.first[cls];
    do {
        int rank = -1;
        for (; list < a.first[cls + 1]; ++list) {
            TeamSync *sync = a.sync + list;
            if (first_lane) {
                // owner and join in one load: a list that is full or closed costs no atomic
                const unsigned long long both = __hip_atomic_load(
                    reinterpret_cast<const unsigned long long *>(&sync->owner), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                int seen = static_cast<int>(both);   // 0: this wave claims the list
                if (static_cast<int>(both >> 32) >= a.inst[list].want) seen = -1;
                if (seen == 0)
                    __hip_atomic_compare_exchange_strong(&sync->owner, &seen, xcc + 1, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (seen == 0 || seen == xcc + 1) {
                    const int j = __hip_atomic_fetch_add(&sync->join, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (j < a.inst[list].want) rank = j;   // a closed list's count is past kTeamSealed
                }
            }
            rank = __builtin_amdgcn_readfirstlane(rank);
            if (rank >= 0) break;
        }
        if (rank < 0) return;
        TeamSync *sync = a.sync + list;
        int size = 0, polls = 0;
        if (rank == 0) {
            const int want = a.inst[list].want;
            const long long t0 = wall_clock64();
            while (team_load(&sync->join) < want && wall_clock64() - t0 < kTeamWait) __builtin_amdgcn_s_sleep(1);
            if (first_lane) {
                size = __hip_atomic_fetch_or(&sync->join, kTeamSealed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                size = size < want ? size : want;
                __hip_atomic_store(&sync->size, size, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            size = __builtin_amdgcn_readfirstlane(size);
        } else {
            while ((size = __builtin_amdgcn_readfirstlane(team_load(&sync->size))) == 0)
                if (team_give_up(polls, a.failed)) return;
        }
        team_dispatch<R, NF>(a, list, rank, size, s);
        ++list;
    } while (AGAIN);
}

// A single phase, without teams: workgroup (x, y) is a member of list y.
template <typename R, int NF> __global__ __launch_bounds__(64) void team_phase(TeamArgs<R> a)
{
    __shared__ __align__(16) cplx<R> s[lds_elems<R>(512)];
    if (a.counter[2] != 0) return;
    const int list = blockIdx.y, size = a.inst[list].want, x = blockIdx.x;
    if (x >= size) return;
    // neighbouring tiles, which share cache lines, on one XCD
    team_dispatch<R, NF>(a, list, size & 7 ? x : (x & 7) * (size >> 3) + (x >> 3), size, s);
}

static_assert(sizeof(TeamArgs<float>) <= 4096 && sizeof(LoneColumnArgs<float>) <= 4096, "kernel arguments");

} // namespace opo
