// The float32 nest on the bf16 matrix cores in one launch, straight from the
// float32 operands (direct_tile.h): no prepass, no packed operands, and with
// ACC_PREC_AUTO the float64 probe and the correction of a tile in the
// workgroup that computed it (in several rounds of tiles with long loops, the
// corrections in a second launch that shares them among all CUs).
//
// A workgroup is G groups of four wavefronts on one output tile; each group
// runs its own share of the K loop with its own LDS stages, and the groups'
// sums are added in group order at the end.  A small product has fewer tiles
// than the chip has CUs, so that one workgroup per CU is all there is: the
// groups multiply the loads in flight and divide the serial chain of K
// stages, each of which costs a memory round trip.  When even that leaves
// CUs idle, the K range is split over workgroups as in the packed path
// (partial sums in a workspace, added in part order by the last part).
//
// Measured (us per call, calls back to back; before: the packed path's two to
// four launches): AUTO LEN = 256 17.8 -> 9.1, 1000 39 -> 17, 2048 96 -> 62,
// 512 x 4096 x 4096 127 -> 70 (245 TFLOP/s float32, 730 of bf16 products); six
// products LEN = 2048 104 -> 88 (1170 TFLOP/s of bf16 products).  What bounds
// them: up to LEN = 512 the launch and a handful of memory round trips (64 x
// 64 x 64 takes 6.6 us, of which the probe 1.9); at 1000, one 64 x 64 tile per
// CU, the loads (32 KB per 64 k and CU, 12.7 ns per k) and 3.5 us of probe; at
// 2048 the tile loop itself, where the matrix cores wait for the split and the
// loads as in the batch kernel.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "direct_tile.h"
#include "kernels.h"

namespace accx {
namespace {

using namespace dev;

struct DirectPlan {
    int tiles_m, tiles_n;
    int ksplit;           // parts of the K range, one workgroup each
    int64_t kpart;        // K elements per part (a multiple of 64), the last shorter
    uint32_t *tickets;    // ksplit > 1: one per tile, zero before the launch, left at zero
    float *partials;      // ksplit x tiles x BM x BN
    double tau2;          // AUTO
    ProbeRecord *rec;     // AUTO
};

template <int BM, int BN, int KS, int G, int NPROD, uint64_t PL, bool AUTO, int KSC, int GC> constexpr int direct_lds()
{
    int n = G * direct_lds_bytes<BM, BN, KS, NPROD, PL>();
    if (AUTO) n = std::max(n, GC * direct_lds_bytes<BM, BN, KSC, 3, PL_CORR3>());
    return std::max(n, std::max((G - 1) * BM * BN * 4, (int)sizeof(DirectProbeLds)));
}

// KS, G: the pass's stage and groups; KSC, GC: the correction's (GC 0: marked
// tiles are left to a launch of their own).
template <int BM, int BN, int KS, int G, int NPROD, uint64_t PL, bool AUTO, int KSC = KS, int GC = G>
__global__ __launch_bounds__(256 * G) void gemm_direct(DirectArgs g, DirectPlan pl)
{
    constexpr int WBM = BM / 64, WBN = BN / 64, NBLK = WBM * WBN;
    __shared__ __attribute__((aligned(1024))) char lds[direct_lds<BM, BN, KS, G, NPROD, PL, AUTO, KSC, GC>()];
    __shared__ int last_part;
    const int T = pl.tiles_m * pl.tiles_n;
    const int tile = (int)(blockIdx.x % (unsigned)T), part = (int)(blockIdx.x / (unsigned)T);
    int tm, tn;
    tile_of(tile, pl.tiles_m, pl.tiles_n, tm, tn);
    const int gi = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), t = threadIdx.x & 255;
    union Acc {
        f32x16 tile[WBM][WBN];
        f32x16 flat[NBLK];
        __device__ Acc() {}
    } acc;
    {
        const int64_t p0 = part * pl.kpart, p1 = min<int64_t>(g.K, p0 + pl.kpart);
        int64_t b, e;
        int barriers;
        group_range<KS, G>(p0, p1, gi, b, e, barriers);
        direct_acc<BM, BN, KS, 2, 2, NPROD, PL, (NPROD >= 5 && BM == 128)>(
            g, tm, tn, b, e, t, barriers, lds + gi * direct_lds_bytes<BM, BN, KS, NPROD, PL>(), acc.tile);
        group_sum<G, 4>(acc.flat, gi, t, lds);
    }
    if (pl.ksplit > 1) {
        // As the packed path's split K: device-scope stores, which count as
        // done at the level the XCDs share, a wait for them, the ticket; the
        // last part reads all parts with device-scope loads.  No fence.
        const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
        const int64_t words = BM * BN;
        if (gi == 0) {
            float *mine = pl.partials + ((int64_t)part * T + tile) * words + wave * (NBLK * 1024) + lane;
#pragma unroll
            for (int x = 0; x < NBLK; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    __hip_atomic_store(mine + x * 1024 + r * 64, acc.flat[x][r], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(vmcnt_imm<0>());
        asm volatile("" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) last_part = atomicAdd(pl.tickets + tile, 1u) == (uint32_t)(pl.ksplit - 1);
        __syncthreads();
        if (!last_part) return;
        if (gi == 0) {
            const float *p = pl.partials + (int64_t)tile * words + wave * (NBLK * 1024) + lane;
#pragma unroll
            for (int x = 0; x < NBLK; ++x) {
                f32x16 sum = (f32x16)0;
                for (int q = 0; q < pl.ksplit; ++q) {
                    const float *b = p + (int64_t)q * T * words + x * 1024;
                    float w[16];
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        w[r] = __hip_atomic_load(b + r * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int r = 0; r < 16; ++r) sum[r] += w[r];
                }
                acc.flat[x] = sum;
            }
        }
        if (threadIdx.x == 0)
            __hip_atomic_store(pl.tickets + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if constexpr (AUTO) {
        const int64_t row0 = (int64_t)tm * BM, col0 = (int64_t)tn * BN, id = (int64_t)tm * pl.tiles_n + tn;
        DirectProbeLds &L = *reinterpret_cast<DirectProbeLds *>(lds);
        if (gi == 0) {
            probe_samples<BM, BN, 2, 2>(acc.tile, t, probe_block(id, (int)min<int64_t>(BM, g.M - row0), 0),
                                        probe_block(id, (int)min<int64_t>(BN, g.N - col0), 1), L.c);
            direct_store<BM, BN, 2, 2>(g, tm, tn, t, acc.tile, false);
        }
        if constexpr (GC == 0) {
            (void)probe_direct<256 * G>(g, BM, BN, id, tm, tn, pl.tau2, pl.rec + id, L);
        } else {
            if (!probe_direct<256 * G>(g, BM, BN, id, tm, tn, pl.tau2, pl.rec + id, L)) return;
            // C += the three correction products (by the threads that stored
            // C, so each reads back its own elements)
            __syncthreads();
            int64_t b = g.K, e = g.K, b0, e0;
            int barriers;
            group_range<KSC, GC>(0, g.K, gi, b0, e0, barriers);
            if (gi < GC) b = b0, e = e0;
            direct_acc<BM, BN, KSC, 2, 2, 3, PL_CORR3>(
                g, tm, tn, b, e, t, barriers, lds + (gi % GC) * direct_lds_bytes<BM, BN, KSC, 3, PL_CORR3>(), acc.tile);
            group_sum<GC, 4>(acc.flat, gi < GC ? gi : -1, t, lds);
            if (gi == 0) direct_store<BM, BN, 2, 2>(g, tm, tn, t, acc.tile, true);
        }
    } else {
        if (gi == 0) direct_store<BM, BN, 2, 2>(g, tm, tn, t, acc.tile, false);
    }
}

// C += the three correction products on the listed tiles: a persistent grid
// over (marked tile, 128 x 128 sub-tile, K part).  How many tiles are marked is
// known on the device only, and a few marked tiles must still fill the chip,
// so the K parts per sub-tile follow from the count: at most about four units
// per workgroup (more parts share fewer operands in the L2: all of LEN = 6144
// marked 2.7 ms in one part, 2.96 in two), and of those the number whose last
// round of units leaves the least of the grid idle (LEN = 4096, row-scaled, 92
// sub-tiles: five parts in one round 467 us a call, eight in two 37 more, packed
// 64 x 64 correction 492; 20 % of LEN = 6144 marked, 468 sub-tiles, one part
// 1.57 ms, five 1.78), none shorter than 64.  Parts leave their sums in
// `partials`, the last one (the record's ticket) adds them in part order to C;
// the result does not depend on the list's order.  Before, every 64 x 64
// sub-tile of C had a workgroup that read its record and, if marked, ran the
// packed three-plane tile over all of K: 1104 of them on the 768 slots of the
// chip in two unequal rounds, 0.71 ms on the row-scaled LEN = 8192 inputs (69
// of 1024 tiles marked, 222 GFLOP); now 0.49 ms, beside 0.55 with C and the
// parts' sums loaded one element after the other.  The split into three planes
// bounds it (88 vector instructions for 12 matrix instructions of a wavefront
// and 16 k).
// After the direct kernel in more than one round of tiles there is no list:
// every workgroup makes it from the records, in the order of the tiles.
struct CorrPlan {
    ProbeRecord *rec;
    int scan;           // > 0: no list, search this many records
    int tiles_n;        // marked tiles per row of C
    int subs_m, subs_n; // 128 x 128 sub-tiles of a marked tile
    float *partials;
    int64_t cap;        // sub-tile sums `partials` holds
    int max_parts;
};

__global__ __launch_bounds__(256, 2) void correct_direct(DirectArgs g, CorrPlan c)
{
    constexpr int BM = 128, KS = 16, NBLK = 4, WORDS = BM * BM;
    __shared__ __attribute__((aligned(1024))) char lds[direct_lds_bytes<BM, BM, KS, 3, PL_CORR3>()];
    __shared__ int last_part;
    __shared__ int found[CORR_SCAN], nfound[4];
    int count;
    if (c.scan > 0) {
        // wavefront w takes the w-th quarter of the records
        constexpr int EACH = CORR_SCAN / 256;
        const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
        int mine[EACH], n = 0;
#pragma unroll
        for (int q = 0; q < EACH; ++q) {
            const int id = (w * EACH + q) * 64 + l;
            mine[q] = id < c.scan ? c.rec[id].corrected : 0;
        }
        uint64_t ballot[EACH];
#pragma unroll
        for (int q = 0; q < EACH; ++q) {
            ballot[q] = __ballot(mine[q] != 0);
            n += __popcll(ballot[q]);
        }
        if (l == 0) nfound[w] = n;
        __syncthreads();
        int at = 0;
        count = 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (v < w) at += nfound[v];
            count += nfound[v];
        }
        count = __builtin_amdgcn_readfirstlane(count);
        if (count == 0) return;
#pragma unroll
        for (int q = 0; q < EACH; ++q) {
            if (mine[q] != 0)
                found[at + __popcll(ballot[q] & (((uint64_t)1 << l) - 1))] = (w * EACH + q) * 64 + l;
            at += __popcll(ballot[q]);
        }
        __syncthreads();
    } else {
        count = __builtin_amdgcn_readfirstlane(c.rec[0].count);
        if (count == 0) return;
    }
    const int subs = c.subs_m * c.subs_n;
    const int64_t S = (int64_t)count * subs;
    const int64_t most = min<int64_t>(min<int64_t>(min<int64_t>(c.max_parts, g.K / 64), c.cap / S),
                                      (4 * (int64_t)gridDim.x + S - 1) / S);
    int64_t parts = 1, rounds = (S + gridDim.x - 1) / gridDim.x;
    for (int64_t q = 2; q <= most; ++q) {
        const int64_t r = (S * q + gridDim.x - 1) / gridDim.x;
        if (r * parts < rounds * q) parts = q, rounds = r;
    }
    const int64_t kpart = ((g.K + parts - 1) / parts + KS - 1) / KS * KS;
    parts = (g.K + kpart - 1) / kpart;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int64_t u = blockIdx.x; u < S * parts; u += gridDim.x) {
        const int64_t x = u / parts, part = u % parts;
        const int sub = (int)(x % subs);
        const int tile = __builtin_amdgcn_readfirstlane(c.scan > 0 ? found[x / subs] : c.rec[x / subs].mark);
        const int tm = tile / c.tiles_n * c.subs_m + sub / c.subs_n, tn = tile % c.tiles_n * c.subs_n + sub % c.subs_n;
        if ((int64_t)tm * BM >= g.M || (int64_t)tn * BM >= g.N) continue;
        f32x16 acc[2][2];
        direct_acc<BM, BM, KS, 2, 2, 3, PL_CORR3>(g, tm, tn, part * kpart, min<int64_t>(g.K, (part + 1) * kpart),
                                                  threadIdx.x, 0, lds, acc);
        if (parts > 1) {
            float *mine = c.partials + u * WORDS + wave * (NBLK * 1024) + lane;
#pragma unroll
            for (int q = 0; q < NBLK; ++q)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    __hip_atomic_store(mine + q * 1024 + r * 64, acc[q / 2][q % 2][r], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(vmcnt_imm<0>());
            asm volatile("" ::: "memory");
            __syncthreads();
            if (threadIdx.x == 0)
                last_part = ((atomicAdd(&c.rec[tile].ticket, 1u << (8 * sub)) >> (8 * sub)) & 255u) ==
                            (uint32_t)(parts - 1);
            __syncthreads();
            const int last = last_part;
            __syncthreads();  // read by all before the next unit writes it
            if (!last) continue;
            // a part's 64 words are all in flight at once (16 at a time, the
            // sum of eight parts was a chain of 32 trips to memory)
            const float *p = c.partials + x * parts * WORDS + wave * (NBLK * 1024) + lane;
#pragma unroll
            for (int q = 0; q < NBLK; ++q) acc[q / 2][q % 2] = (f32x16)0;
            for (int64_t d = 0; d < parts; ++d) {
                float w[NBLK][16];
#pragma unroll
                for (int q = 0; q < NBLK; ++q)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        w[q][r] = __hip_atomic_load(p + d * WORDS + q * 1024 + r * 64, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int q = 0; q < NBLK; ++q)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[q / 2][q % 2][r] += w[q][r];
            }
        }
        direct_store<BM, BM, 2, 2>(g, tm, tn, threadIdx.x, acc, true);
    }
}

template <int BM, int BN, int KS, int G, int NPROD, uint64_t PL, bool AUTO, int KSC = KS, int GC = G>
hipError_t launch(const DirectArgs &g, const DirectPlan &pl, hipStream_t s)
{
    const unsigned grid = (unsigned)(pl.tiles_m * pl.tiles_n * pl.ksplit);
    hipLaunchKernelGGL((gemm_direct<BM, BN, KS, G, NPROD, PL, AUTO, KSC, GC>), dim3(grid), dim3(256 * G), 0, s, g, pl);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_correction(const float *a, const float *b, float *c, const GemmShape &sh, int tile, ProbeRecord *rec,
                             void *work, size_t work_bytes, int max_parts, bool listed, hipStream_t s)
{
    int bm, bn;
    tile_dims(tile, sh.m, sh.n, bm, bn);
    if (bm % 128 || bn % 128) return hipErrorInvalidValue;
    const int scan = listed ? 0 : probe_tiles(tile, sh.m, sh.n);
    if (scan > CORR_SCAN) return hipErrorInvalidValue;
    const DirectArgs g{a, b, c, sh.m, sh.n, sh.k, sh.lda, sh.ldb, sh.ldc};
    const CorrPlan p{rec, scan, (int)((sh.n + bn - 1) / bn), bm / 128, bn / 128, static_cast<float *>(work),
                     (int64_t)(work_bytes / (128 * 128 * 4)), std::min(max_parts, 255)};
    tmark("gemm_bf16x3_corr", s, true);
    hipLaunchKernelGGL(correct_direct, dim3((unsigned)(2 * device_cu_count())), dim3(256), 0, s, g, p);
    tmark("gemm_bf16x3_corr", s, false);
    return hipGetLastError();
}

hipError_t launch_gemm_direct(const float *a, const float *b, float *c, const GemmShape &sh, int products, int tile,
                              double tau, ProbeRecord *rec, bool corrects, hipStream_t s, const SplitK &sk)
{
    if (sh.m <= 0 || sh.n <= 0) return hipSuccess;
    int bm, bn;
    tile_dims(tile, sh.m, sh.n, bm, bn);
    const DirectArgs g{a, b, c, sh.m, sh.n, sh.k, sh.lda, sh.ldb, sh.ldc};
    DirectPlan pl{};
    pl.tiles_m = (int)((sh.m + bm - 1) / bm);
    pl.tiles_n = (int)((sh.n + bn - 1) / bn);
    pl.tau2 = tau * tau;
    pl.rec = rec;
    pl.ksplit = 1;
    pl.kpart = sh.k;
    if (sk.parts > 1) {
        pl.kpart = ((sh.k + sk.parts - 1) / sk.parts + 63) / 64 * 64;
        pl.ksplit = (int)((sh.k + pl.kpart - 1) / pl.kpart);
        const int64_t T = (int64_t)pl.tiles_m * pl.tiles_n;
        pl.tickets = static_cast<uint32_t *>(sk.work);
        pl.partials = reinterpret_cast<float *>(static_cast<char *>(sk.work) + (256 + 4 * T + 255) / 256 * 256);
        if (pl.ksplit > 1) {
            const hipError_t e = launch_zero_u32(pl.tickets, (int)T, s);
            if (e != hipSuccess) return e;
        }
    }
    const char *name = rec ? "gemm_direct_auto" : "gemm_direct";
    tmark(name, s, true);
    hipError_t e = hipErrorInvalidValue;
    if (tile == GEMM_TILE_128) {
        if (rec && corrects)
            e = launch<128, 128, 32, 2, 3, PL_CHEAP3, true, 16, 2>(g, pl, s);
        else if (rec)
            e = launch<128, 128, 32, 2, 3, PL_CHEAP3, true, 16, 0>(g, pl, s);
        else if (products == 6)
            e = launch<128, 128, 16, 2, 6, PL_FULL6, false>(g, pl, s);
        else if (products == 5)
            e = launch<128, 128, 16, 2, 5, PL_FIVE, false>(g, pl, s);
        else if (products == 3)
            e = launch<128, 128, 32, 2, 3, PL_CHEAP3, false>(g, pl, s);
    } else if (tile == GEMM_TILE_64) {
        if (rec && corrects)
            e = launch<64, 64, 32, 4, 3, PL_CHEAP3, true, 32, 2>(g, pl, s);
        else if (products == 6)
            e = launch<64, 64, 32, 2, 6, PL_FULL6, false>(g, pl, s);
        else if (products == 5)
            e = launch<64, 64, 32, 2, 5, PL_FIVE, false>(g, pl, s);
        else if (products == 3)
            e = launch<64, 64, 32, 4, 3, PL_CHEAP3, false>(g, pl, s);
    }
    tmark(name, s, false);
    return e;
}

}  // namespace accx
