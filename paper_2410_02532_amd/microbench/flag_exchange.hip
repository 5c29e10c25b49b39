// flag_exchange.hip -- what an exchange among waiting workgroups costs without fences
// and without a common counter: every workgroup writes 12 KB, waits for its own stores,
// sets a flag of its own, waits until the flags of all members are set, and reads 12 KB
// that other members wrote. (launch_vs_barrier.hip has the same exchange behind a
// device-scope barrier and behind a launch boundary.)
//
//   one XCD    members are the workgroups 0, 8, 16 ... (workgroups are dealt to the eight
//              XCDs in turn): plain stores, loads that miss the L1 and are served by the
//              XCD's L2
//   all XCDs   members are all workgroups: stores and loads at agent scope
//
// Every value read is checked. A wait is bounded: after 2^15 polls the workgroup records
// a time-out and ends, and the members that wait for it do the same. At most one
// workgroup per CU runs, so all members are resident.
//
// Build and run (one GPU):
//   hipcc --offload-arch=gfx950 -O3 -Xclang -target-feature -Xclang -packed-fp32-ops \
//         -o flag_exchange paper_2410_02532_amd/microbench/flag_exchange.hip
//   ./flag_exchange
#include <hip/hip_runtime.h>
#include <cstdio>

#define CK(x) do { hipError_t e_ = (x); if (e_ != hipSuccess) { \
    std::printf("HIP error %s at line %d\n", hipGetErrorString(e_), __LINE__); return 1; } } while (0)

using u64 = unsigned long long;
constexpr int kThreadsMb = 256;
constexpr int kPer = 6;              // values per thread and step (12 KB per workgroup)
constexpr int kMaxGroup = 256;
constexpr int kSpinLimit = 1 << 15;

__device__ inline u64 value(int it, int member, int q) { return static_cast<u64>(it) * 100000 + member * 100 + q; }

template <bool ONE_XCD>
__global__ __launch_bounds__(kThreadsMb) void exchange(u64 *buf, int *flags, int *err, int G, int steps)
{
    constexpr int kStride = ONE_XCD ? 8 : 1;
    constexpr int kFlagScope = ONE_XCD ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT;
    if (blockIdx.x % kStride) return;
    const int r = blockIdx.x / kStride, t = threadIdx.x;
    int bad = 0;
    for (int it = 0; it < steps; ++it) {
        u64 *step = buf + static_cast<size_t>(it & 1) * G * (kThreadsMb * kPer);
        u64 *mine = step + static_cast<size_t>(r) * (kThreadsMb * kPer);
        for (int q = 0; q < kPer; ++q) {
            if constexpr (ONE_XCD) mine[t + kThreadsMb * q] = value(it, r, q);
            else __hip_atomic_store(mine + t + kThreadsMb * q, value(it, r, q), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (t == 0) __hip_atomic_store(flags + r, it + 1, __ATOMIC_RELAXED, kFlagScope);
        int polls = 0, ready = 0;
        do {
            const int f = t < G ? __hip_atomic_load(flags + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : it + 1;
            ready = __syncthreads_and(f >= it + 1);
        } while (!ready && ++polls < kSpinLimit);
        if (!ready) {
            if (t == 0) atomicAdd(err, 1);
            break;
        }
        for (int q = 0; q < kPer; ++q) {
            const int g = (r + 1 + q + (t >> 5)) % G;
            const u64 v = __hip_atomic_load(step + static_cast<size_t>(g) * (kThreadsMb * kPer) + t + kThreadsMb * q,
                                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bad += v != value(it, g, q);
        }
    }
    if (bad) atomicAdd(err + 1, bad);
}

int main()
{
    u64 *buf;
    int *flags, *err;
    CK(hipMalloc(&buf, sizeof(u64) * 2 * kMaxGroup * kThreadsMb * kPer));
    CK(hipMalloc(&flags, sizeof(int) * kMaxGroup));
    CK(hipMalloc(&err, 2 * sizeof(int)));
    hipEvent_t e0, e1;
    CK(hipEventCreate(&e0));
    CK(hipEventCreate(&e1));
    constexpr int kSteps = 1000;
    for (int one : {1, 0})
        for (int G : {8, 16, 24, 32, 64, 128, 256}) {
            if (one && G > 32) break;            // CUs of an XCD
            float best = 1e30f;
            int he[2] = {0, 0};
            for (int rep = 0; rep < 3 && !he[0] && !he[1]; ++rep) {
                CK(hipMemset(flags, 0, sizeof(int) * kMaxGroup));
                CK(hipMemset(err, 0, 2 * sizeof(int)));
                CK(hipDeviceSynchronize());
                CK(hipEventRecord(e0));
                if (one) exchange<true><<<8 * G, kThreadsMb>>>(buf, flags, err, G, kSteps);
                else exchange<false><<<G, kThreadsMb>>>(buf, flags, err, G, kSteps);
                CK(hipGetLastError());
                CK(hipEventRecord(e1));
                CK(hipDeviceSynchronize());
                float ms;
                CK(hipEventElapsedTime(&ms, e0, e1));
                best = ms < best ? ms : best;
                CK(hipMemcpy(he, err, sizeof(he), hipMemcpyDeviceToHost));
            }
            std::printf("%s, %3d workgroups: %.2f us a step, time-outs %d, wrong values %d\n",
                        one ? "one XCD " : "all XCDs", G, best * 1e3f / kSteps, he[0], he[1]);
            std::fflush(stdout);
            if (he[0] || he[1]) return 1;
        }
    return 0;
}
