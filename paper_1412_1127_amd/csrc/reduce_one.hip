// Reductions in one launch: the workgroup whose partial arrives last adds all
// of them, in index order as the second launch of reduce.hip does, so that
// both give the same bits.  The loops over the elements are those of
// reduce.hip's kernels (reduce_body.h).
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>

#include "kernels.h"
#include "reduce_body.h"

namespace accx {
namespace {

// Whether the caller is the last of g to arrive at `word`, which counts the
// arrivals of one call: the call's own number in the bits above ARRIVALS, the
// count below.  A workspace may hold anything before a call, so the first to
// arrive puts the number there; the last one leaves the word zero, which
// saves the next call a step.  Nothing loops or waits on another workgroup.
constexpr uint64_t ARRIVALS = 0xfff;

__device__ inline bool arrives_last_at(uint64_t *word, uint64_t number, unsigned g)
{
    uint64_t seen = 0, count = 1;
    if (!__hip_atomic_compare_exchange_strong(word, &seen, number + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT)) {
        if ((seen & ~ARRIVALS) != number)
            __hip_atomic_compare_exchange_strong(word, &seen, number, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        count = (__hip_atomic_fetch_add(word, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ARRIVALS) + 1;
    }
    if (count != g) return false;
    __hip_atomic_store(word, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// Whether this workgroup is the last of g; called by one thread of each, after
// its stores of partials.  No device-scope fence is needed, which would write
// back the XCD's L2 (18 us over 1 GiB): the partials are device-scope stores,
// written through to the level that the XCDs share, and s_waitcnt holds the
// arrival back until they are there.  Atomics on one word take about 20 ns
// each, one after the other (768 arrivals: 30 us for a sum and sum of squares
// that takes 16), so a grid beyond ONE_WORD arrives at WORD_GROUPS words, each
// 256 bytes from the next, and the last at each of them at a common one.
constexpr unsigned WORD_GROUPS = 32, WORD_STRIDE = 32, ONE_WORD = 64;
static_assert((int)ONE_WORD >= (int)WORD_GROUPS && MAX_BLOCKS <= (int)ARRIVALS &&
                  8 * (1 + WORD_GROUPS) * WORD_STRIDE <= 4 * (4096 - MAX_BLOCKS) &&
                  RED_MAX_VARS * MAX_BLOCKS + (1 + WORD_GROUPS) * WORD_STRIDE <= RED_MAX_VARS * 4096,
              "no empty group, the count in a word, and room for the words");

__device__ inline bool arrives_last(uint64_t *words, uint64_t number, unsigned g)
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((15 << 8) | (7 << 4));  // vmcnt(0)
    asm volatile("" ::: "memory");
    bool last = true;
    unsigned here = g;
    if (g > ONE_WORD) {
        const unsigned k = blockIdx.x % WORD_GROUPS;
        last = arrives_last_at(words + (1 + k) * WORD_STRIDE, number, (g - k + WORD_GROUPS - 1) / WORD_GROUPS);
        here = WORD_GROUPS;
    }
    last = last && arrives_last_at(words, number, here);
    asm volatile("" ::: "memory");
    return last;
}

// The partials and their sum in one launch.
template <typename L>
__global__ __launch_bounds__(RT) void reduce_fast_one(const L *__restrict__ x, int64_t n, uint32_t *partials,
                                                      uint64_t *words, uint64_t number, L init, L *__restrict__ result)
{
    __shared__ L lds4[4];
    __shared__ bool last;
    L s = fast_partial(x, n, lds4);
    const unsigned g = gridDim.x;
    if (g > 1) {
        if (threadIdx.x == 0) {
            __hip_atomic_store(partials + blockIdx.x, to_bits(s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last = arrives_last(words, number, g);
        }
        __syncthreads();
        if (!last) return;
        s = 0;
        for (unsigned k = threadIdx.x; k < g; k += RT)
            s = s + from_bits<L>(__hip_atomic_load(partials + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        s = block_sum(s, lds4);
    }
    if (threadIdx.x == 0) result[0] = init + s;
}

// The partials, folded and combined with the initial values in one launch.
template <typename E, int NV, uint32_t SIG>
__global__ __launch_bounds__(RT) void reduce_vars_one(const E *__restrict__ x, int64_t n, RedVars vars,
                                                      uint64_t *partials, uint64_t *words, uint64_t number,
                                                      E *__restrict__ result)
{
    __shared__ E lds4[4];
    __shared__ bool last;
    int op[NV];
    E acc[NV];
    const unsigned g = gridDim.x;
    vars_partials<E, NV, SIG>(x, n, vars, lds4, [&](int v, int o, E b) {
        op[v] = o;
        acc[v] = b;
        if (g > 1 && threadIdx.x == 0)
            __hip_atomic_store(partials + (size_t)v * g + blockIdx.x, as_bits<E>(b), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    });
    if (g > 1) {
        if (threadIdx.x == 0) last = arrives_last(words, number, g);
        __syncthreads();
        if (!last) return;
        // folds the g partials of each variable in index order
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] = red_identity<E>(op[v]);
        for (unsigned k = threadIdx.x; k < g; k += RT)
#pragma unroll
            for (int v = 0; v < NV; ++v)
                acc[v] = red_apply<E>(op[v], acc[v],
                                      bits_as<E>(__hip_atomic_load(partials + (size_t)v * g + k, __ATOMIC_RELAXED,
                                                                   __HIP_MEMORY_SCOPE_AGENT)));
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] = block_apply<E>(op[v], acc[v], lds4);
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) result[v] = red_apply<E>(op[v], bits_as<E>(vars.init[v]), acc[v]);
    }
}

// A number of one call's own, ARRIVALS and below zero, never 0: a counter,
// mixed (splitmix64's finalizer), so that nothing that a workspace can hold by
// chance looks like it.  It starts from the clock and from where this process
// was loaded, so that numbers an earlier process left in memory differ too;
// std::random_device may throw, which no C entry may.
uint64_t call_number() noexcept
{
    static std::atomic<uint64_t> next{
        (uint64_t)std::chrono::system_clock::now().time_since_epoch().count() * 0x9e3779b97f4a7c15ull +
        (uint64_t)(uintptr_t)&next};
    uint64_t z;
    do {
        z = next.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed);
        z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
        z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
        z = (z ^ (z >> 31)) & ~(uint64_t)0xfff;
    } while (z == 0);
    return z;
}

}  // namespace

bool reduce_in_one_launch(int64_t g, int64_t limit, hipStream_t s)
{
    // A capture is replayed with one number, so that arrivals left over from
    // replays that overlapped would spoil all later ones: two launches.  The
    // null stream cannot be captured, and is not asked: while a blocking
    // stream is under capture the query itself fails there, and its error
    // would be taken for the launch's.
    if (g == 1) return true;
    if (g > limit) return false;
    if (s == nullptr) return true;
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st == hipStreamCaptureStatusNone;
}

template <typename L>
void launch_reduce_one(const L *x, int64_t n, L init, L *result, uint32_t *partials, unsigned g, hipStream_t s)
{
    hipLaunchKernelGGL(reduce_fast_one<L>, dim3(g), dim3(RT), 0, s, x, n, partials,
                       reinterpret_cast<uint64_t *>(partials + MAX_BLOCKS), call_number(), init, result);
}
template void launch_reduce_one<float>(const float *, int64_t, float, float *, uint32_t *, unsigned, hipStream_t);
template void launch_reduce_one<uint32_t>(const uint32_t *, int64_t, uint32_t, uint32_t *, uint32_t *, unsigned,
                                          hipStream_t);

template <typename E>
void launch_reduce_vars_one(const E *x, int64_t n, const RedVars &vars, E *result, uint64_t *partials, unsigned g,
                            hipStream_t s)
{
    auto run = [&](auto nv) {
        constexpr int NV = decltype(nv)::value;
        with_operators<NV>(vars, [&](auto sig) {
            hipLaunchKernelGGL((reduce_vars_one<E, NV, decltype(sig)::value>), dim3(g), dim3(RT), 0, s, x, n, vars,
                               partials, partials + RED_MAX_VARS * MAX_BLOCKS, call_number(), result);
        });
    };
    switch (vars.nvars) {  // 1..RED_MAX_VARS, as the callers have checked
    case 1: return run(std::integral_constant<int, 1>{});
    case 2: return run(std::integral_constant<int, 2>{});
    case 3: return run(std::integral_constant<int, 3>{});
    default: return run(std::integral_constant<int, 4>{});
    }
}
template void launch_reduce_vars_one<float>(const float *, int64_t, const RedVars &, float *, uint64_t *, unsigned,
                                            hipStream_t);
template void launch_reduce_vars_one<int32_t>(const int32_t *, int64_t, const RedVars &, int32_t *, uint64_t *,
                                              unsigned, hipStream_t);
template void launch_reduce_vars_one<double>(const double *, int64_t, const RedVars &, double *, uint64_t *, unsigned,
                                             hipStream_t);
template void launch_reduce_vars_one<int64_t>(const int64_t *, int64_t, const RedVars &, int64_t *, uint64_t *,
                                              unsigned, hipStream_t);

}  // namespace accx
