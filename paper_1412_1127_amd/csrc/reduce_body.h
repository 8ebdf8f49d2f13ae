// What the streaming reductions of one and of two launches share: the loop
// over the elements, the combination of values over a workgroup, the operators
// and element types.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"

namespace accx {
namespace {

constexpr int RT = 256;          // threads per workgroup
constexpr int RU = 8;            // 16-byte loads in flight per thread
constexpr int MAX_BLOCKS = 1024; // fast kernels: upper bound on workgroups

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

template <typename L> struct Vec;
template <> struct Vec<float> { using T = f4; };
template <> struct Vec<uint32_t> { using T = u4; };

template <typename L> __device__ inline L hsum(typename Vec<L>::T v) { return (v.x + v.y) + (v.z + v.w); }

template <typename L> __device__ inline L wave_sum(L v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = v + __shfl_xor(v, o, 64);
    return v;
}

// Sum over the 256 threads of a workgroup, fixed order; valid in thread 0.
template <typename L> __device__ inline L block_sum(L v, L *lds4)
{
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) lds4[w] = v;
    __syncthreads();
    L r = 0;
    if (threadIdx.x == 0) r = (lds4[0] + lds4[1]) + (lds4[2] + lds4[3]);
    return r;
}

__device__ inline uint32_t to_bits(float v) { return __float_as_uint(v); }
__device__ inline uint32_t to_bits(uint32_t v) { return v; }
template <typename L> __device__ inline L from_bits(uint32_t b);
template <> __device__ inline float from_bits<float>(uint32_t b) { return __uint_as_float(b); }
template <> __device__ inline uint32_t from_bits<uint32_t>(uint32_t b) { return b; }

// A workgroup's partial of the sum over its grid-stride slice; valid in
// thread 0.
template <typename L> __device__ inline L fast_partial(const L *__restrict__ x, int64_t n, L *lds4)
{
    using V = typename Vec<L>::T;

    // Aligned body of 16-byte vectors, with up to 3 leading and 3 trailing
    // scalars (x may start at any 4-byte boundary).
    const uintptr_t addr = (uintptr_t)x;
    int64_t head = (int64_t)(((16u - (unsigned)(addr & 15u)) & 15u) >> 2);
    if (head > n) head = n;
    const int64_t nvec = (n - head) >> 2;
    const int64_t tail0 = head + (nvec << 2);
    const V *__restrict__ xv = reinterpret_cast<const V *>(x + head);

    const int64_t stride = (int64_t)gridDim.x * RT;
    int64_t v = (int64_t)blockIdx.x * RT + threadIdx.x;
    V acc[RU];
#pragma unroll
    for (int u = 0; u < RU; ++u) acc[u] = (V)0;
    for (; v + (RU - 1) * stride < nvec; v += RU * stride) {
        V t[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) t[u] = __builtin_nontemporal_load(xv + v + u * stride);
#pragma unroll
        for (int u = 0; u < RU; ++u) acc[u] += t[u];
    }
    for (; v < nvec; v += stride) acc[0] += __builtin_nontemporal_load(xv + v);
    // fixed pairwise combination of the accumulators
#pragma unroll
    for (int w = RU / 2; w > 0; w >>= 1)
#pragma unroll
        for (int u = 0; u < w; ++u) acc[u] += acc[u + w];
    L s = hsum<L>(acc[0]);
    if (blockIdx.x == 0) {
        if (threadIdx.x < head) s = s + x[threadIdx.x];
        if ((int64_t)threadIdx.x < n - tail0) s = s + x[tail0 + threadIdx.x];
    }
    return block_sum(s, lds4);
}

// ---- reduction variables of any operator and type --------------------------
//
// Up to four reduction variables over one array in one pass (the SRAD loop
// keeps a sum and a sum of squares of the same image): variable v combines
// f_v(x[k]) with operator op_v, where f_v(x) = x or x*x in the element type.
// Operators: + (integers wrap around), max, min (floats: a NaN operand is
// ignored, as fmax/fmin do).  Each thread folds its grid-stride slice into
// one accumulator per variable in a fixed order, the workgroup combines its
// threads in a fixed tree and stores one partial per variable, and the
// workgroup that arrives last, or a second launch, folds the partials in
// index order and then the initial value: result_v = init_v (op_v) (partial_0 (op_v) partial_1 ...).

template <typename E> struct Red;
template <> struct Red<float> {
    using V = f4;
    using Bits = uint32_t;
    static constexpr int W = 4;
    __device__ static float lowest() { return -__builtin_inff(); }
    __device__ static float highest() { return __builtin_inff(); }
    __device__ static float add(float a, float b) { return a + b; }
    __device__ static float mul(float a, float b) { return a * b; }
    __device__ static float max(float a, float b) { return __builtin_fmaxf(a, b); }
    __device__ static float min(float a, float b) { return __builtin_fminf(a, b); }
    __device__ static bool nonzero(float a) { return a != 0.0f; }
};
typedef double d2 __attribute__((ext_vector_type(2)));
template <> struct Red<double> {
    using V = d2;
    using Bits = uint64_t;
    static constexpr int W = 2;
    __device__ static double lowest() { return -__builtin_inf(); }
    __device__ static double highest() { return __builtin_inf(); }
    __device__ static double add(double a, double b) { return a + b; }
    __device__ static double mul(double a, double b) { return a * b; }
    __device__ static double max(double a, double b) { return __builtin_fmax(a, b); }
    __device__ static double min(double a, double b) { return __builtin_fmin(a, b); }
    __device__ static bool nonzero(double a) { return a != 0.0; }
};
typedef int32_t i4 __attribute__((ext_vector_type(4)));
template <> struct Red<int32_t> {
    using V = i4;
    using Bits = uint32_t;
    static constexpr int W = 4;
    __device__ static int32_t lowest() { return INT32_MIN; }
    __device__ static int32_t highest() { return INT32_MAX; }
    __device__ static int32_t add(int32_t a, int32_t b) { return (int32_t)((uint32_t)a + (uint32_t)b); }
    __device__ static int32_t mul(int32_t a, int32_t b) { return (int32_t)((uint32_t)a * (uint32_t)b); }
    __device__ static int32_t max(int32_t a, int32_t b) { return a > b ? a : b; }
    __device__ static int32_t min(int32_t a, int32_t b) { return a < b ? a : b; }
    __device__ static bool nonzero(int32_t a) { return a != 0; }
};
typedef int64_t l2 __attribute__((ext_vector_type(2)));
template <> struct Red<int64_t> {
    using V = l2;
    using Bits = uint64_t;
    static constexpr int W = 2;
    __device__ static int64_t lowest() { return INT64_MIN; }
    __device__ static int64_t highest() { return INT64_MAX; }
    __device__ static int64_t add(int64_t a, int64_t b) { return (int64_t)((uint64_t)a + (uint64_t)b); }
    __device__ static int64_t mul(int64_t a, int64_t b) { return (int64_t)((uint64_t)a * (uint64_t)b); }
    __device__ static int64_t max(int64_t a, int64_t b) { return a > b ? a : b; }
    __device__ static int64_t min(int64_t a, int64_t b) { return a < b ? a : b; }
    __device__ static bool nonzero(int64_t a) { return a != 0; }
};

template <typename E> __device__ inline E red_identity(int op)
{
    return op == RED_SUM ? (E)0 : op == RED_MAX ? Red<E>::lowest() : Red<E>::highest();
}

template <typename E> __device__ inline E red_apply(int op, E a, E b)
{
    return op == RED_SUM ? Red<E>::add(a, b) : op == RED_MAX ? Red<E>::max(a, b) : Red<E>::min(a, b);
}

template <typename E> __device__ inline E bits_as(uint64_t b)
{
    typename Red<E>::Bits t = (typename Red<E>::Bits)b;
    return __builtin_bit_cast(E, t);
}
template <typename E> __device__ inline uint64_t as_bits(E v)
{
    return (uint64_t)__builtin_bit_cast(typename Red<E>::Bits, v);
}

// Combine v over the workgroup in a fixed order; valid in thread 0.
template <typename E> __device__ inline E block_apply(int op, E v, E *lds4)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = red_apply<E>(op, v, __shfl_xor(v, o, 64));
    if ((threadIdx.x & 63) == 0) lds4[threadIdx.x >> 6] = v;
    __syncthreads();
    E r = v;
    if (threadIdx.x == 0) r = red_apply<E>(op, red_apply<E>(op, lds4[0], lds4[1]), red_apply<E>(op, lds4[2], lds4[3]));
    __syncthreads();
    return r;
}

// Operators fixed at compile time: SIG holds (op | square << 2) of variable v
// in bits 4v..4v+3; SIG_RUNTIME reads them from `vars` (any combination, but
// the per-element operator selection then costs more VALU work than the
// element's load: about 4.5 instead of 6.9 TB/s over 1 GiB).
constexpr uint32_t SIG_RUNTIME = 0xffffffffu;

// Hands a workgroup's partial of each variable over its grid-stride slice to
// put(v, operator, partial), which stores thread 0's.
template <typename E, int NV, uint32_t SIG, typename Put>
__device__ inline void vars_partials(const E *__restrict__ x, int64_t n, const RedVars &vars, E *lds4, Put put)
{
    using R = Red<E>;
    using V = typename R::V;
    constexpr int W = R::W;

    int op[NV], sq[NV];
    E acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        op[v] = SIG == SIG_RUNTIME ? vars.op[v] : (int)((SIG >> (4 * v)) & 3u);
        sq[v] = SIG == SIG_RUNTIME ? vars.square[v] : (int)((SIG >> (4 * v + 2)) & 1u);
        acc[v] = red_identity<E>(op[v]);
    }
    auto fold = [&](E t) {
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] = red_apply<E>(op[v], acc[v], sq[v] ? R::mul(t, t) : t);
    };

    // Aligned body of 16-byte vectors, up to W-1 leading and trailing scalars.
    const uintptr_t addr = (uintptr_t)x;
    int64_t head = (int64_t)(((16u - (unsigned)(addr & 15u)) & 15u) / sizeof(E));
    if (head > n) head = n;
    const int64_t nvec = (n - head) / W;
    const int64_t tail0 = head + nvec * W;
    const V *__restrict__ xv = reinterpret_cast<const V *>(x + head);
    const int64_t stride = (int64_t)gridDim.x * RT;
    int64_t i = (int64_t)blockIdx.x * RT + threadIdx.x;
    for (; i + (RU - 1) * stride < nvec; i += RU * stride) {
        V t[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) t[u] = __builtin_nontemporal_load(xv + i + u * stride);
#pragma unroll
        for (int u = 0; u < RU; ++u)
#pragma unroll
            for (int e = 0; e < W; ++e) fold(t[u][e]);
    }
    for (; i < nvec; i += stride) {
        const V t = __builtin_nontemporal_load(xv + i);
#pragma unroll
        for (int e = 0; e < W; ++e) fold(t[e]);
    }
    if (blockIdx.x == 0) {
        if ((int64_t)threadIdx.x < head) fold(x[threadIdx.x]);
        if ((int64_t)threadIdx.x < n - tail0) fold(x[tail0 + threadIdx.x]);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) put(v, op[v], block_apply<E>(op[v], acc[v], lds4));
}

// Operator sets that are compiled: one variable (+, max, min; x or x*x), and
// the pairs the paper's reduction loops use (SRAD's sum and sum of squares)
// or that come as one (max and min); anything else decodes at run time.
// Calls launch with the set as an integral constant.
template <int NV, typename Launch> void with_operators(const RedVars &vars, Launch launch)
{
    uint32_t sig = 0;
    for (int v = 0; v < NV; ++v) sig |= (uint32_t)(vars.op[v] | (vars.square[v] ? 4 : 0)) << (4 * v);
    if constexpr (NV == 1) {
        switch (sig) {
        case 0x0: return launch(std::integral_constant<uint32_t, 0x0>{});
        case 0x1: return launch(std::integral_constant<uint32_t, 0x1>{});
        case 0x2: return launch(std::integral_constant<uint32_t, 0x2>{});
        case 0x4: return launch(std::integral_constant<uint32_t, 0x4>{});
        case 0x5: return launch(std::integral_constant<uint32_t, 0x5>{});
        case 0x6: return launch(std::integral_constant<uint32_t, 0x6>{});
        }
    } else if constexpr (NV == 2) {
        switch (sig) {
        case 0x40: return launch(std::integral_constant<uint32_t, 0x40>{});  // sum, sum of squares
        case 0x04: return launch(std::integral_constant<uint32_t, 0x04>{});  // sum of squares, sum
        case 0x21: return launch(std::integral_constant<uint32_t, 0x21>{});  // max, min
        case 0x12: return launch(std::integral_constant<uint32_t, 0x12>{});  // min, max
        }
    }
    launch(std::integral_constant<uint32_t, SIG_RUNTIME>{});
}

}  // namespace

// One launch instead of two (reduce_one.hip), for a grid of g workgroups:
// whether it is taken, and the launches.  `partials`: the workspace.  The
// limits: arrivals cost more the more there are, and a second launch costs
// what it costs.  us a call, two launches / one: a float32 or int32 sum
// (whose second launch adds plain words) 8.2 / 5.6 at 13 workgroups, 8.3 /
// 5.7 at 86 to 184, 8.3 / 8.1 at 245, 8.4 / 7.8 at 367 to 489, but 9.7 / 10.3
// at 733 and 11.6 / 12.5 at 768; other variables, whose second launch takes
// longer, at every size: float64 sum 8.9 / 5.9 at 98, 9.0 / 7.1 at 391, 8.9 /
// 8.5 at 489, float32 sum and sum of squares 9.2 / 6.2 at 98, 11.2 / 10.4 at
// 733, 16.6 / 15.7 over 2^24 elements, max and min 9.3 / 8.4 at 367.
constexpr int64_t ONE_LAUNCH_SUM = 512, ONE_LAUNCH_VARS = MAX_BLOCKS;
bool reduce_in_one_launch(int64_t g, int64_t limit, hipStream_t s);
template <typename L>
void launch_reduce_one(const L *x, int64_t n, L init, L *result, uint32_t *partials, unsigned g, hipStream_t s);
template <typename E>
void launch_reduce_vars_one(const E *x, int64_t n, const RedVars &vars, E *result, uint64_t *partials, unsigned g,
                            hipStream_t s);

}  // namespace accx
