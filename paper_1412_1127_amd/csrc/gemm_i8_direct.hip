// The int32 nest on the int8 matrix cores in one launch, straight from the
// int32 operands: the balanced base-256 digits of the header of gemm_mfma.hip
// are formed between the global load and LDS, and how many of them a stage of
// the K loop needs is decided from that stage's own elements.  No prepass, no
// maximum over the operands before the product can begin, no second packing
// pass and kernel that usually exit at once: the packed path's four launches
// become one.  A stage runs one product if all of its elements fit one digit,
// four if they fit two, else ten, whatever the other stages hold.
//
// Work per element and tile: two operations for all four digits (x +
// 0x00808080, with the sign bits of the lower three bytes flipped back, is the
// four digits' bytes), two byte permutes to gather a digit of four elements
// into a word, one LDS write.  So the path pays while tiles are few: each
// operand element is converted once per tile that reads it and moves four
// bytes instead of one.
//
// Measured, us per call, before and after (values in [-16, 16] / full range):
// LEN = 64 10.5 -> 4.7 / 16.7 -> 5.1; 256 12.2 -> 7.2 / 23.2 -> 8.1; 1000 17.0 ->
// 16.1 / 58 -> 21; 128 x 128 x 4096 18.8 -> 15.1 / 131 -> 16.9.  Up to 512 the
// launch and the memory round trips bound it; at 1000 (one 64 x 64 tile per CU)
// the conversion and the 32 KB a stage loads.  Before the two wavefronts of a
// SIMD took the halves of a step in opposite order, ten products on 128 x 128
// tiles took 71 us instead of 63 at 1531.
//
// Groups of wavefronts share a tile's K loop as in gemm_direct.hip; the sums
// are integers modulo 2^32, so neither groups nor parts change the result.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "direct_tile.h"
#include "kernels.h"

namespace accx {
namespace {

using namespace dev;

struct I8Args {
    const int32_t *A, *B;
    int32_t *C;
    int64_t M, N, K, lda, ldb, ldc;
    int tiles_m, tiles_n;
    int ksplit;         // parts of the K range, one workgroup each
    int64_t kpart;      // K elements per part (a multiple of 64)
    uint32_t *tickets;  // ksplit > 1: one per tile, zero before the launch, left at zero
    int32_t *partials;  // ksplit x tiles x BM x BN
};

constexpr int KS8 = 64;             // K elements per LDS stage
constexpr int CS8 = 512 + 64;       // bytes per 16-element chunk of 32 rows, padded (direct_cs)
constexpr int PLS8 = KS8 / 16 * CS8;
constexpr int UNIT8 = 4 * PLS8;     // 32 rows, four digit planes
template <int BM, int BN> constexpr int i8_stage_bytes() { return (BM / 32 + BN / 32) * UNIT8; }

// acc = the product over k in [kb, ke) on tile (tm, tn), modulo 2^32, by one
// group of WGM x WGN wavefronts (t: thread in the group; lds: its two stages;
// flags: its two rows of one word per wavefront).  As direct_acc: the operands
// of the stage after next are in flight while a stage is computed, one barrier
// of the workgroup per stage, `barriers` stages' worth in all.
template <int BM, int BN, int WGM, int WGN>
__device__ __attribute__((always_inline)) inline void i8_acc(const I8Args &g, int tm, int tn, int64_t kb, int64_t ke,
                                                             int t, int barriers, char *lds, uint32_t (*flags)[WGM * WGN],
                                                             i32x16 (&out)[BM / 32 / WGM][BN / 32 / WGN])
{
    constexpr int THREADS = WGM * WGN * 64, WAVES = WGM * WGN;
    constexpr int MB = BM / 32, WBM = MB / WGM, WBN = BN / 32 / WGN, STAGE = i8_stage_bytes<BM, BN>();
    constexpr int RPP = THREADS / 16, NA = BM / RPP, CG = THREADS / BN;
    static_assert(BM % RPP == 0 && 32 % RPP == 0 && CG == KS8 / 16, "staging divides evenly");
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int wm = wave / WGN, wn = wave % WGN;
    const int64_t row0 = (int64_t)tm * BM, col0 = (int64_t)tn * BN;
    // this thread's pieces: 4 elements of row ar + j * RPP, 16 of column bcol
    const int ar = t / 16, ak = (t % 16) * 4, bcol = t % BN, bc = t / BN;
    uint32_t offA[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j)
        offA[j] = ((uint32_t)min<int64_t>(ar + j * RPP, g.M - 1 - row0) * (uint32_t)g.lda + ak) * 4u;
    const uint32_t offB = ((uint32_t)bc * 16u * (uint32_t)g.ldb + (uint32_t)min<int64_t>(bcol, g.N - 1 - col0)) * 4u;
    const int32_t *pA = g.A + row0 * g.lda, *pB = g.B + col0;
    const int wA = (ak >> 4) * CS8 + ar * 16 + (ak & 15);
    const int wB = MB * UNIT8 + (bcol / 32) * UNIT8 + bc * CS8 + (bcol & 31) * 16;

    i32x4 ra[NA];
    int32_t rb[16];
    auto load = [&](int64_t k) {
        const auto sa = buffer_of(pA + k), sb = buffer_of(pB + k * g.ldb);
#pragma unroll
        for (int j = 0; j < NA; ++j)
            ra[j] = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(sa, offA[j], 0, 0));
#pragma unroll
        for (int e = 0; e < 16; ++e)
            rb[e] = (int32_t)__builtin_amdgcn_raw_buffer_load_b32(sb, offB, e * (int)g.ldb * 4, 0);
    };
    auto load_tail = [&](int64_t k, int n) {  // the last, shorter stage: n elements, then zeros
        const char *a = reinterpret_cast<const char *>(pA + k);
#pragma unroll
        for (int j = 0; j < NA; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                ra[j][e] = ak + e < n ? *reinterpret_cast<const int32_t *>(a + offA[j] + 4 * e) : 0;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const char *be = reinterpret_cast<const char *>(pB + (k + e) * g.ldb);
            rb[e] = bc * 16 + e < n ? *reinterpret_cast<const int32_t *>(be + offB) : 0;
        }
    };
    // Planes 1-3 are written only if this wavefront's elements of the stage
    // use them, or to put zeros back where it wrote them before (`full`: the
    // buffers whose planes 1-3 this wavefront may have left nonzero).
    uint32_t full_planes = 3;
    auto stage = [&](int buf) {
        char *s = lds + buf * STAGE;
        uint32_t oa = 0, ob = 0;  // digits 1-3 in use
#pragma unroll
        for (int j = 0; j < NA; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) oa |= digit_bytes(ra[j][e]);
#pragma unroll
        for (int e = 0; e < 16; ++e) ob |= digit_bytes(rb[e]);
        // digit planes 1-3 of A (bits 1-3) and of B (bits 5-7) in use
        uint32_t f = 0;
        if (__any(((oa | ob) >> 8) != 0)) {
#pragma unroll
            for (int p = 1; p < 4; ++p) {
                f |= __any(((oa >> (8 * p)) & 255u) != 0) ? 1u << p : 0u;
                f |= __any(((ob >> (8 * p)) & 255u) != 0) ? 16u << p : 0u;
            }
        }
        char *dB = s + wB;
        if (f || ((full_planes >> buf) & 1u)) {
            full_planes = f ? full_planes | (1u << buf) : full_planes & ~(1u << buf);
#pragma unroll
            for (int j = 0; j < NA; ++j) {
                uint32_t w[4];
                digits4(ra[j].x, ra[j].y, ra[j].z, ra[j].w, w);
                char *d = s + wA + (j * RPP / 32) * UNIT8 + (j * RPP % 32) * 16;
#pragma unroll
                for (int p = 0; p < 4; ++p) *reinterpret_cast<uint32_t *>(d + p * PLS8) = w[p];
            }
            uint32_t w[4][4];
#pragma unroll
            for (int q = 0; q < 4; ++q) digits4(rb[4 * q], rb[4 * q + 1], rb[4 * q + 2], rb[4 * q + 3], w[q]);
#pragma unroll
            for (int p = 0; p < 4; ++p)
                *reinterpret_cast<u32x4_t *>(dB + p * PLS8) = u32x4_t{w[0][p], w[1][p], w[2][p], w[3][p]};
        } else {
#pragma unroll
            for (int j = 0; j < NA; ++j)
                *reinterpret_cast<int *>(s + wA + (j * RPP / 32) * UNIT8 + (j * RPP % 32) * 16) =
                    low_bytes4(ra[j].x, ra[j].y, ra[j].z, ra[j].w);
            *reinterpret_cast<i32x4 *>(dB) =
                i32x4{low_bytes4(rb[0], rb[1], rb[2], rb[3]), low_bytes4(rb[4], rb[5], rb[6], rb[7]),
                      low_bytes4(rb[8], rb[9], rb[10], rb[11]), low_bytes4(rb[12], rb[13], rb[14], rb[15])};
        }
        if (lane == 0) flags[buf][wave] = f;
    };
    i32x16 acc[4][WBM][WBN];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int i = 0; i < WBM; ++i)
#pragma unroll
            for (int j = 0; j < WBN; ++j) acc[a][i][j] = (i32x16)0;
    const int off = (lane >> 5) * CS8 + (lane & 31) * 16;
    auto compute = [&](int buf) {
        uint32_t f = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) f |= flags[buf][w];
        f = __builtin_amdgcn_readfirstlane(f);
        const char *sA = lds + buf * STAGE + wm * WBM * UNIT8 + off;
        const char *sB = lds + buf * STAGE + (MB + wn * WBN) * UNIT8 + off;
        // The products of digit pairs (p, q), p + q <= 3, that digits below LO
        // do not have and digits below HI do.  Per 32 k: B's planes once, then
        // plane by plane of A with every product that plane takes part in (a
        // fragment read per product instead, ten products took 30 KB of LDS
        // reads a wavefront, more LDS time than matrix time; the three sets
        // below take 21).
        auto products = [&](auto lo, auto hi) {
            constexpr int LO = decltype(lo)::value, HI = decltype(hi)::value;
#pragma unroll
            for (int s = 0; s < KS8 / 32; ++s) {
                i32x4 fb[HI][WBN];
#pragma unroll
                for (int q = 0; q < HI; ++q)
#pragma unroll
                    for (int j = 0; j < WBN; ++j)
                        fb[q][j] = *reinterpret_cast<const i32x4 *>(sB + j * UNIT8 + q * PLS8 + 2 * s * CS8);
#pragma unroll
                for (int p = 0; p < HI; ++p) {
                    i32x4 fa[WBM];
#pragma unroll
                    for (int i = 0; i < WBM; ++i)
                        fa[i] = *reinterpret_cast<const i32x4 *>(sA + i * UNIT8 + p * PLS8 + 2 * s * CS8);
#pragma unroll
                    for (int q = p < LO ? LO : 0; q < HI && q + p < 4; ++q)
#pragma unroll
                        for (int i = 0; i < WBM; ++i)
#pragma unroll
                            for (int j = 0; j < WBN; ++j)
                                acc[p + q][i][j] = Mma<true>::run(fa[i], fb[q][j], acc[p + q][i][j]);
                }
            }
        };
        // uniform: one digit, two, or more.  (As nested sets: as one branch per
        // digit count the compiler kept a copy of the accumulators per branch
        // and spilled them, eight times slower.)
        using D0 = std::integral_constant<int, 0>;
        using D1 = std::integral_constant<int, 1>;
        using D2 = std::integral_constant<int, 2>;
        using D4 = std::integral_constant<int, 4>;
        products(D0(), D1());
        if (f != 0) products(D1(), D2());
        if ((f & 0xccu) != 0) products(D2(), D4());
    };
    const int64_t len = ke - kb;
    const int full = (int)(len / KS8), tail = (int)(len % KS8), steps = full + (tail ? 1 : 0);
    auto load_any = [&](int s) {
        if (s < full)
            load(kb + (int64_t)s * KS8);
        else
            load_tail(kb + (int64_t)s * KS8, tail);
    };
    // The two wavefronts of a SIMD (w and w + 4 of the workgroup) take the two
    // halves of a step in opposite order, so that one splits on the vector
    // unit while the other multiplies.
    const bool early = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) & 1;
    int s = 0;
    if (full > 2) {
        load(kb);
        stage(0);
        load(kb + KS8);
        lds_barrier();
        for (; s + 2 < full; ++s) {
            if (early) {
                stage((s + 1) & 1);
                load(kb + (int64_t)(s + 2) * KS8);
            }
            compute(s & 1);
            if (!early) {
                stage((s + 1) & 1);
                load(kb + (int64_t)(s + 2) * KS8);
            }
            lds_barrier();
        }
    } else {
        if (steps > 0) {
            load_any(0);
            stage(0);
        }
        if (steps > 1) load_any(1);
        lds_barrier();
    }
    for (; s < steps; ++s) {
        if (s + 1 < steps) stage((s + 1) & 1);
        if (s + 2 < steps) load_any(s + 2);
        compute(s & 1);
        lds_barrier();
    }
    for (; s < barriers; ++s) lds_barrier();
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int j = 0; j < WBN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                out[i][j][r] = (int)((uint32_t)acc[0][i][j][r] + ((uint32_t)acc[1][i][j][r] << 8) +
                                     ((uint32_t)acc[2][i][j][r] << 16) + ((uint32_t)acc[3][i][j][r] << 24));
}

template <int BM, int BN, int WGM, int WGN, int G>
__global__ __launch_bounds__(WGM *WGN * 64 * G) void gemm_i8_direct(I8Args g)
{
    constexpr int WAVES = WGM * WGN, TG = WAVES * 64, WBM = BM / 32 / WGM, WBN = BN / 32 / WGN, NBLK = WBM * WBN;
    constexpr int GROUP = 2 * i8_stage_bytes<BM, BN>();
    static_assert(G * GROUP >= (G - 1) * BM * BN * 4 && G * GROUP <= 156 * 1024, "LDS");
    __shared__ __attribute__((aligned(1024))) char lds[G * GROUP];
    __shared__ uint32_t flags[G][2][WAVES];
    __shared__ int last_part;
    const int T = g.tiles_m * g.tiles_n;
    const int tile = (int)(blockIdx.x % (unsigned)T), part = (int)(blockIdx.x / (unsigned)T);
    int tm, tn;
    tile_of(tile, g.tiles_m, g.tiles_n, tm, tn);
    const int gi = __builtin_amdgcn_readfirstlane(threadIdx.x / TG), t = threadIdx.x % TG;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    i32x16 acc[WBM][WBN];
    {
        const int64_t p0 = part * g.kpart, p1 = min<int64_t>(g.K, p0 + g.kpart);
        int64_t b, e;
        int barriers;
        group_range<KS8, G>(p0, p1, gi, b, e, barriers);
        i8_acc<BM, BN, WGM, WGN>(g, tm, tn, b, e, t, barriers, lds + gi * GROUP, flags[gi], acc);
    }
    if constexpr (G > 1) {  // group 0 adds the other groups' sums
        i32x4 *sum = reinterpret_cast<i32x4 *>(lds);
        lds_barrier();
#pragma unroll
        for (int x = 0; x < NBLK; ++x)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (gi > 0) {
                    const i32x16 &v = acc[x / WBN][x % WBN];
                    sum[((((gi - 1) * WAVES + wave) * NBLK + x) * 4 + r) * 64 + lane] =
                        i32x4{v[4 * r], v[4 * r + 1], v[4 * r + 2], v[4 * r + 3]};
                }
        lds_barrier();
        if (gi > 0 && g.ksplit == 1) return;
#pragma unroll
        for (int x = 0; x < NBLK; ++x)
#pragma unroll
            for (int q = 0; q < G - 1; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (gi == 0) {
                        const i32x4 v = sum[(((q * WAVES + wave) * NBLK + x) * 4 + r) * 64 + lane];
                        i32x16 &a = acc[x / WBN][x % WBN];
#pragma unroll
                        for (int e = 0; e < 4; ++e) a[4 * r + e] = (int)((uint32_t)a[4 * r + e] + (uint32_t)v[e]);
                    }
    }
    if (g.ksplit > 1) {
        // as gemm_direct's parts: device-scope stores, a wait for them, the
        // ticket; the last part adds all of them
        const int64_t words = BM * BN;
        if (gi == 0) {
            int32_t *mine = g.partials + ((int64_t)part * T + tile) * words + wave * (NBLK * 1024) + lane;
#pragma unroll
            for (int x = 0; x < NBLK; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    __hip_atomic_store(mine + x * 1024 + r * 64, acc[x / WBN][x % WBN][r], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(vmcnt_imm<0>());
        asm volatile("" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) last_part = atomicAdd(g.tickets + tile, 1u) == (uint32_t)(g.ksplit - 1);
        __syncthreads();
        if (!last_part || gi > 0) return;
        const int32_t *p = g.partials + (int64_t)tile * words + wave * (NBLK * 1024) + lane;
#pragma unroll
        for (int x = 0; x < NBLK; ++x) {
            uint32_t sum[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[r] = 0;
            for (int q = 0; q < g.ksplit; ++q)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    sum[r] += (uint32_t)__hip_atomic_load(p + (int64_t)q * T * words + x * 1024 + r * 64,
                                                          __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[x / WBN][x % WBN][r] = (int)sum[r];
        }
        if (threadIdx.x == 0) __hip_atomic_store(g.tickets + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // 32 x 32 accumulator layout as in direct_store
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int j = 0; j < WBN; ++j) {
            const int64_t col = (int64_t)tn * BN + (wave % WGN * WBN + j) * 32 + (lane & 31);
            const int64_t rowb = (int64_t)tm * BM + (wave / WGN * WBM + i) * 32 + (lane >> 5) * 4;
            if (col >= g.N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = rowb + (r >> 2) * 8 + (r & 3);
                if (row < g.M) g.C[row * g.ldc + col] = acc[i][j][r];
            }
        }
}

}  // namespace

hipError_t launch_gemm_i8_direct(const int32_t *a, const int32_t *b, int32_t *c, const GemmShape &sh, int tile,
                                 hipStream_t s, const SplitK &sk)
{
    if (sh.m <= 0 || sh.n <= 0) return hipSuccess;
    int bm, bn;
    tile_dims(tile, sh.m, sh.n, bm, bn);
    I8Args g{a, b, c, sh.m, sh.n, sh.k, sh.lda, sh.ldb, sh.ldc};
    g.tiles_m = (int)((sh.m + bm - 1) / bm);
    g.tiles_n = (int)((sh.n + bn - 1) / bn);
    g.ksplit = 1;
    g.kpart = sh.k;
    const int64_t T = (int64_t)g.tiles_m * g.tiles_n;
    if (sk.parts > 1) {
        g.kpart = ((sh.k + sk.parts - 1) / sk.parts + KS8 - 1) / KS8 * KS8;
        g.ksplit = (int)((sh.k + g.kpart - 1) / g.kpart);
        g.tickets = static_cast<uint32_t *>(sk.work);
        g.partials = reinterpret_cast<int32_t *>(static_cast<char *>(sk.work) + (256 + 4 * T + 255) / 256 * 256);
        if (g.ksplit > 1) {
            const hipError_t e = launch_zero_u32(g.tickets, (int)T, s);
            if (e != hipSuccess) return e;
        }
    }
    const unsigned grid = (unsigned)(T * g.ksplit);
    tmark("gemm_i8_direct", s, true);
    if (tile == GEMM_TILE_128)
        hipLaunchKernelGGL((gemm_i8_direct<128, 128, 2, 4, 1>), dim3(grid), dim3(512), 0, s, g);
    else
        hipLaunchKernelGGL((gemm_i8_direct<64, 64, 2, 2, 2>), dim3(grid), dim3(512), 0, s, g);
    tmark("gemm_i8_direct", s, false);
    return hipGetLastError();
}

}  // namespace accx
