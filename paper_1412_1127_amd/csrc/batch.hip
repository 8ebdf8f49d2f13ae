// Batched offload: many independent loop-nest matmuls (Listing 1a,
// section 1.3) and reduction(+) clauses (section 2.3; SRAD paragraph of
// section 4.2) run as one graph of two kernels:
//
//  1. batch_prologue: zeroes the queues' counters and the reductions' tickets,
//     and copies the matmul operands that some item of the batch overwrites;
//  2. batch_persistent: a persistent kernel (a fixed number of workgroups per
//     CU) that pulls work units from queues through atomic counters: either
//     one output tile of one matmul, straight from the float32 operands
//     (direct_tile.h) on the tile configuration chosen for that matmul's
//     size, or one chunk of one reduction.  There is one queue per XCD, and a
//     matmul's tiles all sit in one of them, so that they share an L2; a
//     workgroup whose queue is empty helps with the others.  A queue
//     interleaves matmul tiles (largest matmuls first) with reduction chunks
//     so that HBM-bound and matrix-core-bound work share the CUs.
//
// What bounds it: 512 matmuls (LEN uniform over 64, 128, ..., 1024) and 256
// sums (2^16 to 2^24 elements) take 1.49 ms, 1.28 ms with the matmuls alone
// and 0.49 ms with the sums alone (6.4 TB/s).  They took 2.54 ms while a
// prepass packed every operand (0.71 ms) for tiles fed by direct-to-LDS
// loads (1.83 ms); queues per XCD instead of one: 1.85 -> 1.80 ms; 256 x 128
// tiles beside 128 x 128: 1.80 -> 1.65 ms; a second set of loads in flight in
// the sums: 1.65 -> 1.60 ms; the probe on the float64 matrix cores: 1.60 ->
// 1.51 ms.  In the tile loop (128 x 128, LEN = 4096) the matrix cores are busy
// 44 % of the cycles, the vector units 34 % (the split is two thirds of that)
// and the LDS 38 %: with two wavefronts per SIMD their times add up more than
// they overlap.  Without the split the tile would run 13 % faster, without its
// loads 30 %; three workgroups per CU of 16-element stages gained 5 % on 128 x
// 128, less than the larger tile, which they leave no registers for.
//
// A reduction's chunk partials are combined by the workgroup that finishes
// its last chunk (atomic ticket), in chunk order, so results do not depend
// on which workgroup ran what.  A matmul tile is computed by one workgroup in
// fixed K order, bitwise as by the standalone kernel in the same tile
// configuration when that one runs unsplit (no split K).
//
// Precision: six products (FULL6), or AUTO: the three-product pass of the
// tile, then the same workgroup probes that tile in float64 (probe_direct:
// the standalone probe's samples) and, if the tile is marked, adds the three
// correction products over it -- the standalone AUTO path's steps for that
// tile, done in place, so no other workgroup and no other launch is involved.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "direct_tile.h"

namespace accx {
namespace {

using namespace dev;

constexpr int BT = 256;              // threads per workgroup (both kernels)
// Persistent workgroups per CU (LDS: 2 x 72 KB).  They leave a lane 256
// registers; the AUTO kernel's 256 x 128 branch needs 28 more, which it keeps
// in 116 bytes of scratch (3 and 16 bytes without that branch, none with six
// products).
constexpr int WG_PER_CU = 2;
constexpr uint32_t UNIT_RED = 0x80000000u;

// K elements per LDS stage: a stage holds 24 matrix instructions per
// wavefront on 256 x 128 and 128 x 128 with either product list, 12 on 64 x
// 64, and two workgroups' stages fit a CU.

constexpr int cmax(int a, int b) { return a > b ? a : b; }
constexpr int LDS_MAX = cmax(cmax(direct_lds_bytes<256, 128, 16, 3, PL_CHEAP3>(), direct_lds_bytes<128, 128, 16, 3, PL_CORR3>()),
                        cmax(cmax(direct_lds_bytes<128, 128, 32, 3, PL_CHEAP3>(), direct_lds_bytes<64, 64, 64, 3, PL_CHEAP3>()),
                             cmax(direct_lds_bytes<128, 128, 16, 6, PL_FULL6>(), direct_lds_bytes<64, 64, 32, 6, PL_FULL6>())));
static_assert(LDS_MAX * WG_PER_CU <= 160 * 1024 && sizeof(DirectProbeLds) <= LDS_MAX, "persistent kernel LDS");

constexpr int COPY_WGS = 256;  // prologue workgroups per operand copy

// Makes the queue ready for one run of the persistent kernel: workgroup 0
// zeroes the counters, the others make the operand copies.
__global__ __launch_bounds__(BT) void batch_prologue(BatchQueue q)
{
    if (blockIdx.x == 0) {
        if (threadIdx.x < BATCH_QUEUES) q.counters[threadIdx.x * BATCH_COUNTER_STRIDE] = 0u;
        for (uint32_t k = threadIdx.x; k < q.nreds; k += BT) *q.reds[k].ticket = 0u;
        return;
    }
    const BatchCopy c = q.copies[(blockIdx.x - 1) / COPY_WGS];
    const int64_t step = (int64_t)COPY_WGS * BT;
    for (int64_t k = (int64_t)((blockIdx.x - 1) % COPY_WGS) * BT + threadIdx.x; k < c.n; k += step) c.dst[k] = c.src[k];
}

__device__ inline float wave_sum_f(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Sum over the workgroup in fixed order; valid in thread 0.
__device__ inline float block_sum_f(float v, float *red4)
{
    v = wave_sum_f(v);
    if ((threadIdx.x & 63) == 0) red4[threadIdx.x >> 6] = v;
    __syncthreads();
    const float r = (threadIdx.x == 0) ? (red4[0] + red4[1]) + (red4[2] + red4[3]) : 0.0f;
    __syncthreads();
    return r;
}

typedef float f4v __attribute__((ext_vector_type(4)));

__device__ __attribute__((always_inline)) inline void reduce_chunk(const BatchRed &r, uint32_t chunk, float *red4, int *is_last)
{
    const int64_t b0 = (int64_t)chunk * r.chunk;
    const int64_t b1 = b0 + r.chunk < r.n ? b0 + r.chunk : r.n;
    const float *__restrict__ x = r.x;
    float s = 0.0f;
    if ((((uintptr_t)(x + b0)) & 15u) == 0) {
        const int64_t nv = (b1 - b0) >> 2;
        const f4v *__restrict__ xv = reinterpret_cast<const f4v *>(x + b0);
        // two sets of eight 16-byte loads: one in flight while the other is added
        f4v acc[8], t[2][8];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[u] = (f4v)0;
        int64_t v = threadIdx.x;
        auto load = [&](int64_t at, f4v(&w)[8]) {
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u] = __builtin_nontemporal_load(xv + at + u * BT);
        };
        auto add = [&](const f4v(&w)[8]) {
#pragma unroll
            for (int u = 0; u < 8; ++u) acc[u] += w[u];
        };
        if (v + 15 * BT < nv) {
            load(v, t[0]);
            load(v + 8 * BT, t[1]);
            for (v += 16 * BT; v + 15 * BT < nv; v += 16 * BT) {
                add(t[0]);
                load(v, t[0]);
                add(t[1]);
                load(v + 8 * BT, t[1]);
            }
            add(t[0]);
            add(t[1]);
        }
        for (; v < nv; v += BT) acc[0] += xv[v];
#pragma unroll
        for (int w = 4; w > 0; w >>= 1)
#pragma unroll
            for (int u = 0; u < w; ++u) acc[u] += acc[u + w];
        s = (acc[0].x + acc[0].y) + (acc[0].z + acc[0].w);
        for (int64_t e = b0 + (nv << 2) + threadIdx.x; e < b1; e += BT) s += x[e];
    } else {
        for (int64_t e = b0 + threadIdx.x; e < b1; e += BT) s += x[e];
    }
    s = block_sum_f(s, red4);
    if (threadIdx.x == 0) {
        // The partial goes out as a device-scope store (through to the
        // level the XCDs share) and counts as done before the ticket; the
        // last chunk reads the partials with device-scope loads.  No fence:
        // a device-scope fence writes back and invalidates this XCD's whole
        // L2 under the matmul tiles that share it, once per chunk.
        __hip_atomic_store(r.partials + chunk, __float_as_uint(s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(vmcnt_imm<0>());
        asm volatile("" ::: "memory");
        *is_last = (atomicAdd(r.ticket, 1u) == (uint32_t)r.nchunks - 1);
    }
    __syncthreads();
    if (!*is_last) return;
    float t = 0.0f;
    for (int k = threadIdx.x; k < r.nchunks; k += BT)
        t += __uint_as_float(__hip_atomic_load(r.partials + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    t = block_sum_f(t, red4);
    if (threadIdx.x == 0) {
        *r.result = r.init + t;
        __hip_atomic_store(r.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <int BM, int BN, int KS, int NPROD, uint64_t PL>
__device__ __attribute__((always_inline)) inline void matmul_pass(const DirectArgs &g, int tm, int tn, char *lds,
                                                                   bool accumulate)
{
    f32x16 acc[BM / 64][BN / 64];
    direct_acc<BM, BN, KS, 2, 2, NPROD, PL>(g, tm, tn, 0, g.K, threadIdx.x, 0, lds, acc);
    direct_store<BM, BN, 2, 2>(g, tm, tn, threadIdx.x, acc, accumulate);
}

// The three-product pass of a tile; leaves the probe's samples of C in L.
template <int BM, int BN, int KS>
__device__ __attribute__((always_inline)) inline void cheap_pass(const DirectArgs &g, int tm, int tn, char *lds,
                                                                  uint32_t tile)
{
    f32x16 acc[BM / 64][BN / 64];
    direct_acc<BM, BN, KS, 2, 2, 3, PL_CHEAP3>(g, tm, tn, 0, g.K, threadIdx.x, 0, lds, acc);
    const int64_t row0 = (int64_t)tm * BM, col0 = (int64_t)tn * BN;
    probe_samples<BM, BN, 2, 2>(acc, threadIdx.x, probe_block(tile, (int)min<int64_t>(BM, g.M - row0), 0),
                                probe_block(tile, (int)min<int64_t>(BN, g.N - col0), 1),
                                reinterpret_cast<DirectProbeLds *>(lds)->c);
    direct_store<BM, BN, 2, 2>(g, tm, tn, threadIdx.x, acc, false);
}

template <bool AUTO>
__device__ __attribute__((always_inline)) inline void matmul_unit(const BatchMat &m, uint32_t tile, char *lds,
                                                                  double tau2)
{
    const DirectArgs g{m.a, m.b, m.c, m.len, m.len, m.len, m.len, m.len, m.len};
    const int tm = (int)(tile / (uint32_t)m.tiles_n), tn = (int)(tile % (uint32_t)m.tiles_n);
    if constexpr (!AUTO) {
        if (m.tile == GEMM_TILE_128)
            matmul_pass<128, 128, 16, 6, PL_FULL6>(g, tm, tn, lds, false);
        else
            matmul_pass<64, 64, 32, 6, PL_FULL6>(g, tm, tn, lds, false);
    } else {
        if (m.tile == GEMM_TILE_256x128)
            cheap_pass<256, 128, 16>(g, tm, tn, lds, tile);
        else if (m.tile == GEMM_TILE_128)
            cheap_pass<128, 128, 32>(g, tm, tn, lds, tile);
        else
            cheap_pass<64, 64, 64>(g, tm, tn, lds, tile);
        const int bm = m.tile == GEMM_TILE_256x128 ? 256 : m.tile == GEMM_TILE_128 ? 128 : 64;
        const int bn = m.tile == GEMM_TILE_64 ? 64 : 128;
        if (!probe_direct<BT>(g, bm, bn, tile, tm, tn, tau2, nullptr, *reinterpret_cast<DirectProbeLds *>(lds))) return;
        // Marked: C += the three correction products.  This tile of C is read
        // back only by this workgroup, so the barrier's workgroup-scope release
        // and acquire make it visible; a device-scope fence here would write
        // back the L2.  The LDS is free after the barrier too.
        __syncthreads();
        if (m.tile == GEMM_TILE_64) {
            matmul_pass<64, 64, 32, 3, PL_CORR3>(g, tm, tn, lds, true);
        } else {
            const int sub = bm / 128;
            for (int q = 0; q < sub; ++q)
                if ((int64_t)(tm * sub + q) * 128 < g.M)
                    matmul_pass<128, 128, 16, 3, PL_CORR3>(g, tm * sub + q, tn, lds, true);
        }
    }
}

template <bool AUTO>
__global__ __launch_bounds__(BT, WG_PER_CU) void batch_persistent(BatchQueue q)
{
    __shared__ __attribute__((aligned(1024))) char lds[LDS_MAX];
    __shared__ uint32_t cur;
    __shared__ float red4[4];
    __shared__ int is_last;
    // This XCD's queue first; once it is empty, the others' in turn.  A queue
    // that has run out stays empty, so every workgroup leaves after at most
    // BATCH_QUEUES failed pulls.
    for (int tries = 0; tries < BATCH_QUEUES;) {
        const int x = (int)((blockIdx.x + tries) % BATCH_QUEUES);
        if (threadIdx.x == 0) cur = atomicAdd(q.counters + x * BATCH_COUNTER_STRIDE, 1u);
        lds_barrier();
        const uint32_t u = q.first[x] + __builtin_amdgcn_readfirstlane(cur);
        lds_barrier();  // every thread has read `cur` before it is rewritten
        if (u >= q.first[x + 1]) {
            ++tries;
            continue;
        }
        const BatchUnit w = q.units[u];
        if (w.item & UNIT_RED)
            reduce_chunk(q.reds[w.item & ~UNIT_RED], w.sub, red4, &is_last);
        else
            matmul_unit<AUTO>(q.mats[w.item], w.sub, lds, q.tau2);
        lds_barrier();  // LDS and shared scalars are reused by the next unit
    }
}

}  // namespace

int batch_tile_supported(int tile) { return tile == GEMM_TILE_128 || tile == GEMM_TILE_64; }

int batch_workgroups() { return device_cu_count() * WG_PER_CU; }

hipError_t launch_batch_prologue(const BatchQueue &q, hipStream_t s)
{
    tmark("batch_prologue", s, true);
    hipLaunchKernelGGL(batch_prologue, dim3(1 + q.ncopies * COPY_WGS), dim3(BT), 0, s, q);
    tmark("batch_prologue", s, false);
    return hipGetLastError();
}

hipError_t launch_batch_persistent(const BatchQueue &q, hipStream_t s)
{
    tmark("batch_persistent", s, true);
    if (q.auto_prec)
        hipLaunchKernelGGL(batch_persistent<true>, dim3((unsigned)batch_workgroups()), dim3(BT), 0, s, q);
    else
        hipLaunchKernelGGL(batch_persistent<false>, dim3((unsigned)batch_workgroups()), dim3(BT), 0, s, q);
    tmark("batch_persistent", s, false);
    return hipGetLastError();
}

}  // namespace accx
