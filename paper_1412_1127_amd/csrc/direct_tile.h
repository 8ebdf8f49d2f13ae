// The bf16x3 matrix-core tile straight from float32 operands: the split into
// bf16 terms runs between the global load and LDS, so that no prepass writes
// and re-reads packed operands and one launch does the whole product.
//
// What it trades.  The packed path (mfma_tile.h) splits each element once and
// moves 4 or 6 bytes of planes per element and tile through direct-to-LDS
// loads; here each tile splits its own operands (three VALU instructions per
// element for two planes, 5.5 for three) and moves the 4 bytes of the element
// itself.  The prepass (4 bytes read, 6 written per element, and a launch)
// goes away.  With 128 x 128 tiles an element's split is shared by 128
// outputs: 48 VALU instructions per 16 k beside 12 matrix instructions per
// wavefront, half of the matrix time and overlapping it.
//
// The matrix instructions see the same planes in the same order as the packed
// path (k in 16-element steps, the products of the list within each step), so
// the results are bitwise those of the packed tiles, unsplit.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"
#include "mfma_tile.h"

namespace accx {
namespace dev {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct DirectArgs {
    const float *A, *B;  // row-major M x K and K x N
    float *C;            // M x N
    int64_t M, N, K, lda, ldb, ldc;
};

// A buffer resource over all 4 GB above p (uniform): offsets are checked by
// the caller, not by the resource.
__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void *p)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, 0xffffffff, 0x00020000);
}

// The planes of two elements, packed: w[p] = plane p of x0 (low half) and x1.
// Plane p + 1 of x is RN of what plane p leaves (split3).
template <int NPL> __device__ inline void split_pair(float x0, float x1, uint32_t (&w)[NPL])
{
#pragma unroll
    for (int p = 0; p < NPL; ++p) {
        w[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x0, x1}, bf16x2));
        if (p + 1 < NPL) {
            x0 -= __uint_as_float(w[p] << 16);
            x1 -= __uint_as_float(w[p] & 0xffff0000u);
        }
    }
}

// LDS layout of one stage: units of 32 rows; per unit NPL planes of KS / 8
// chunks (8 elements of a row, 16 bytes), row r of chunk c at c * CS + r * 16.
// CS is 512 bytes plus a pad that spreads the chunks a wavefront writes at
// once (KS / 4 lanes per row of A, 8 bytes each) over all banks; fragment
// reads (32 rows x 16 bytes of one chunk) are contiguous either way.
template <int KS> constexpr int direct_cs() { return 512 + 2048 / KS; }
template <int KS, int NPL> constexpr int direct_unit() { return NPL * (KS / 8) * direct_cs<KS>(); }
template <int BM, int BN, int KS, int NPROD, uint64_t PL> constexpr int direct_lds_bytes()
{
    return 2 * (BM / 32 + BN / 32) * direct_unit<KS, planes_used(PL, NPROD)>();
}

// acc = sum over k in [kb, ke) of the product list on tile (tm, tn), by
// WGM x WGN wavefronts: a whole workgroup, or one of its groups of that many,
// each with an LDS area of its own (t: the thread's index in its group).  Two
// LDS stages of KS elements; the float32 operands of the stage after next are
// in flight in registers while a stage is computed: one barrier of the
// workgroup per stage, `barriers` stages' worth in all, so that groups with
// fewer stages keep step.  Rows past M and columns past N read the last row
// or column (their outputs are not stored); elements past ke are zero in both
// operands.
// OPP: the two wavefronts of a SIMD (w and w + 4 of the workgroup, in two
// groups) stage the next operands at opposite ends of a step, so that one
// splits while the other multiplies; without it each spreads its staging over
// the step.  Six products, LEN = 2048: 91.5 -> 88.7 us, 512 x 4096 x 4096 99 ->
// 95; three products, whose steps are half as long, 64 -> 69 us.
template <int BM, int BN, int KS, int WGM, int WGN, int NPROD, uint64_t PL, bool OPP = false>
__device__ __attribute__((always_inline)) inline void direct_acc(const DirectArgs &g, int tm, int tn, int64_t kb,
                                                                 int64_t ke, int t, int barriers, char *lds,
                                                                 f32x16 (&acc)[BM / 32 / WGM][BN / 32 / WGN])
{
    constexpr int THREADS = WGM * WGN * 64;
    constexpr int NPL = planes_used(PL, NPROD);
    constexpr int MB = BM / 32, NB = BN / 32, WBM = MB / WGM, WBN = NB / WGN;
    constexpr int CS = direct_cs<KS>(), PLS = (KS / 8) * CS, UNIT = NPL * PLS, STAGE = (MB + NB) * UNIT;
    constexpr int LA = KS / 4, RPP = THREADS / LA, NA = BM / RPP;  // A: lanes per row, rows per pass, passes
    constexpr int CG = THREADS / BN, NBC = (KS / 8) / CG;          // B: chunks per pass, passes
    static_assert(BM % RPP == 0 && THREADS % BN == 0 && (KS / 8) % CG == 0, "staging divides evenly");
    static_assert(RPP % 32 == 0 || 32 % RPP == 0, "rows per pass");
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int wm = wave / WGN, wn = wave % WGN;
    const int64_t row0 = (int64_t)tm * BM, col0 = (int64_t)tn * BN;

    // this thread's pieces: 4 elements of row ar + j * RPP, and the 8 elements
    // of chunk bc + i * CG of column bcol; byte offsets from the tile's corner
    // (below 2^32: the host admits lda, ldb <= DIRECT_MAX_LD only)
    const int ar = t / LA, ak = (t % LA) * 4;
    const int bcol = t % BN, bc = t / BN;
    uint32_t offA[NA], offB[NBC];
#pragma unroll
    for (int j = 0; j < NA; ++j)
        offA[j] = ((uint32_t)min<int64_t>(ar + j * RPP, g.M - 1 - row0) * (uint32_t)g.lda + ak) * 4u;
#pragma unroll
    for (int i = 0; i < NBC; ++i)
        offB[i] = ((uint32_t)(bc + i * CG) * 8u * (uint32_t)g.ldb + (uint32_t)min<int64_t>(bcol, g.N - 1 - col0)) * 4u;
    const float *pA = g.A + row0 * g.lda, *pB = g.B + col0;
    const int wA = (ar / 32) * UNIT + (ak >> 3) * CS + (ar & 31) * 16 + ((ak >> 2) & 1) * 8;
    const int wB = MB * UNIT + (bcol / 32) * UNIT + bc * CS + (bcol & 31) * 16;

    // Buffer loads: a scalar base per stage (and per row of B) and the
    // thread's constant 32-bit offset, so a load costs no vector address
    // arithmetic.
    f32x4 ra[NA];
    float rb[NBC][8];
    auto load_a = [&](int j, int64_t k) {
        ra[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(buffer_of(pA + k), offA[j], 0, 0));
    };
    auto load_b = [&](int i, int64_t k) {
        const auto r = buffer_of(pB + k * g.ldb);
#pragma unroll
        for (int e = 0; e < 8; ++e)
            rb[i][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, offB[i], e * (int)g.ldb * 4, 0));
    };
    auto load = [&](int64_t k) {
#pragma unroll
        for (int j = 0; j < NA; ++j) load_a(j, k);
#pragma unroll
        for (int i = 0; i < NBC; ++i) load_b(i, k);
    };
    // the last, shorter stage: n elements
    auto load_tail = [&](int64_t k, int n) {
        const char *a = reinterpret_cast<const char *>(pA + k);
#pragma unroll
        for (int j = 0; j < NA; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                ra[j][e] = ak + e < n ? *reinterpret_cast<const float *>(a + offA[j] + 4 * e) : 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const char *be = reinterpret_cast<const char *>(pB + (k + e) * g.ldb);
#pragma unroll
            for (int i = 0; i < NBC; ++i)
                rb[i][e] = (bc + i * CG) * 8 + e < n ? *reinterpret_cast<const float *>(be + offB[i]) : 0.0f;
        }
    };
    auto stage_a = [&](int j, char *s) {
        uint32_t lo[NPL], hi[NPL];
        split_pair<NPL>(ra[j].x, ra[j].y, lo);
        split_pair<NPL>(ra[j].z, ra[j].w, hi);
        char *d = s + wA + (j * RPP / 32) * UNIT + (j * RPP % 32) * 16;
#pragma unroll
        for (int p = 0; p < NPL; ++p) *reinterpret_cast<u32x2 *>(d + p * PLS) = u32x2{lo[p], hi[p]};
    };
    auto stage_b = [&](int i, char *s) {
        uint32_t w[4][NPL];
#pragma unroll
        for (int q = 0; q < 4; ++q) split_pair<NPL>(rb[i][2 * q], rb[i][2 * q + 1], w[q]);
        char *d = s + wB + i * CG * CS;
#pragma unroll
        for (int p = 0; p < NPL; ++p)
            *reinterpret_cast<u32x4_t *>(d + p * PLS) = u32x4_t{w[0][p], w[1][p], w[2][p], w[3][p]};
    };
    const int off = (lane >> 5) * CS + (lane & 31) * 16;
    bf16x8 fa[NPL][WBM], fb[NPL][WBN];
    auto frags = [&](int buf, int sub) {
        const char *sA = lds + buf * STAGE + wm * WBM * UNIT + 2 * sub * CS + off;
        const char *sB = lds + buf * STAGE + (MB + wn * WBN) * UNIT + 2 * sub * CS + off;
#pragma unroll
        for (int p = 0; p < NPL; ++p) {
#pragma unroll
            for (int i = 0; i < WBM; ++i) fa[p][i] = *reinterpret_cast<const bf16x8 *>(sA + i * UNIT + p * PLS);
#pragma unroll
            for (int j = 0; j < WBN; ++j) fb[p][j] = *reinterpret_cast<const bf16x8 *>(sB + j * UNIT + p * PLS);
        }
    };
    auto product = [&](int q) {
#pragma unroll
        for (int i = 0; i < WBM; ++i)
#pragma unroll
            for (int j = 0; j < WBN; ++j)
                acc[i][j] = Mma<false>::run(fa[prod_p(PL, q)][i], fb[prod_q(PL, q)][j], acc[i][j]);
    };
    constexpr int SUB = KS / 16;
    const int64_t len = ke - kb;
    const int full = (int)(len / KS), tail = (int)(len % KS), steps = full + (tail ? 1 : 0);
    auto load_any = [&](int s) {
        if (s < full)
            load(kb + (int64_t)s * KS);
        else
            load_tail(kb + (int64_t)s * KS, tail);
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int j = 0; j < NA; ++j) stage_a(j, lds + buf * STAGE);
#pragma unroll
        for (int i = 0; i < NBC; ++i) stage_b(i, lds + buf * STAGE);
    };

#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int j = 0; j < WBN; ++j) acc[i][j] = (f32x16)0;
    const bool early = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) & 1;
    int s = 0;
    // The step is cut into GROUPS scheduling regions, one product of one 16-k
    // sub-step each; region x also splits its share of the next stage's pieces
    // and issues the load that refills each piece's registers, so that every
    // load has a whole step to arrive.
    constexpr int GROUPS = SUB * NPROD, PIECES = NA + NBC;
    if (full > 2) {
        load(kb);
        stage(0);
        load(kb + KS);
        lds_barrier();
        for (; s + 2 < full; ++s) {
            char *next = lds + ((s + 1) & 1) * STAGE;
            const int64_t k2 = kb + (int64_t)(s + 2) * KS;
            auto pieces = [&](int z0, int z1) {
#pragma unroll
                for (int z = 0; z < PIECES; ++z) {
                    if (z < z0 || z >= z1) continue;
                    if (z < NA) {
                        stage_a(z, next);
                        load_a(z, k2);
                    } else {
                        stage_b(z - NA, next);
                        load_b(z - NA, k2);
                    }
                }
            };
            if (OPP && early) pieces(0, PIECES);
#pragma unroll
            for (int x = 0; x < GROUPS; ++x) {
                if (x % NPROD == 0) frags(s & 1, x / NPROD);
                product(x % NPROD);
                if constexpr (!OPP) {
                    pieces(x * PIECES / GROUPS, (x + 1) * PIECES / GROUPS);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (OPP && !early) pieces(0, PIECES);
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
#pragma unroll
        for (int x = 0; x < GROUPS; ++x) {
            if (x % NPROD == 0) frags(s & 1, x / NPROD);
            product(x % NPROD);
        }
        lds_barrier();
    }
    for (; s < barriers; ++s) lds_barrier();
}

// K range of group gi of G: whole KS stages, the same number for every group
// but the last ones.
template <int KS, int G>
__device__ inline void group_range(int64_t kb, int64_t ke, int gi, int64_t &b, int64_t &e, int &barriers)
{
    const int64_t stages = (ke - kb + KS - 1) / KS;
    barriers = (int)((stages + G - 1) / G);
    b = min<int64_t>(ke, kb + (int64_t)gi * barriers * KS);
    e = min<int64_t>(ke, b + (int64_t)barriers * KS);
}

// Adds the accumulators of groups 1 .. G - 1 to group 0's, in group order,
// through LDS (G - 1 groups x BM x BN floats).  Begins and ends with a barrier.
template <int G, int WAVES, int NB>
__device__ __attribute__((always_inline)) inline void group_sum(f32x16 (&acc)[NB], int gi, int t, char *lds)
{
    if constexpr (G > 1) {
        const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
        f32x4 *part = reinterpret_cast<f32x4 *>(lds);
        lds_barrier();
        if (gi > 0) {
#pragma unroll
            for (int x = 0; x < NB; ++x)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    part[((((gi - 1) * WAVES + wave) * NB + x) * 4 + r) * 64 + lane] =
                        f32x4{acc[x][4 * r], acc[x][4 * r + 1], acc[x][4 * r + 2], acc[x][4 * r + 3]};
        }
        lds_barrier();
        if (gi == 0) {
#pragma unroll
            for (int q = 0; q < G - 1; ++q)
#pragma unroll
                for (int x = 0; x < NB; ++x)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const f32x4 v = part[(((q * WAVES + wave) * NB + x) * 4 + r) * 64 + lane];
                        acc[x][4 * r] += v.x, acc[x][4 * r + 1] += v.y, acc[x][4 * r + 2] += v.z, acc[x][4 * r + 3] += v.w;
                    }
        }
        lds_barrier();
    }
}

// C = acc (or C += acc) on tile (tm, tn); a block's elements are all loaded
// before the first is stored (one after the other, 64 round trips to memory
// made a correction of K = 64 take 17 us longer).  32 x 32 accumulator layout:
// register r of lane l holds row (r / 4) * 8 + (l / 32) * 4 + r % 4, column
// l % 32 of the block.
template <int BM, int BN, int WGM, int WGN>
__device__ __attribute__((always_inline)) inline void direct_store(const DirectArgs &g, int tm, int tn, int t,
                                                                   const f32x16 (&acc)[BM / 32 / WGM][BN / 32 / WGN],
                                                                   bool accumulate)
{
    constexpr int MB = BM / 32, NB = BN / 32, WBM = MB / WGM, WBN = NB / WGN;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int wm = wave / WGN, wn = wave % WGN;
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int j = 0; j < WBN; ++j) {
            const int64_t col = ((int64_t)tn * NB + wn * WBN + j) * 32 + (lane & 31);
            const int64_t rowb = ((int64_t)tm * MB + wm * WBM + i) * 32 + (lane >> 5) * 4;
            if (col >= g.N) continue;
            f32x16 old = (f32x16)0;
            if (accumulate) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int64_t row = rowb + (r >> 2) * 8 + (r & 3);
                    if (row < g.M) old[r] = g.C[row * g.ldc + col];
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = rowb + (r >> 2) * 8 + (r & 3);
                if (row < g.M) g.C[row * g.ldc + col] = accumulate ? old[r] + acc[i][j][r] : acc[i][j][r];
            }
        }
}

struct DirectProbeLds {
    double part[16][PS * PS];  // one row per wavefront
    float c[PS * PS];
    int marked;
};

// The probe's samples of C, from the accumulators of the tile: PS consecutive
// rows and columns from tile row 8 r8 and tile column 8 c8 (both uniform).
// An aligned group of 8 rows of a 32 x 32 block is registers 4 g .. 4 g + 3 of
// both lane halves.  (Rows past M and columns past N hold the last row's and
// column's values, which is where probe_pick clamps to.)
template <int BM, int BN, int WGM, int WGN>
__device__ __attribute__((always_inline)) inline void probe_samples(const f32x16 (&acc)[BM / 32 / WGM][BN / 32 / WGN],
                                                                    int t, int r8, int c8, float *cs)
{
    constexpr int WBM = BM / 32 / WGM, WBN = BN / 32 / WGN;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int bi = r8 / 4 - wave / WGN * WBM, bj = c8 / 4 - wave % WGN * WBN;  // block within this wavefront's
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int j = 0; j < WBN; ++j)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq)
                if (i == bi && j == bj && gq == (r8 & 3) && ((lane & 31) >> 3) == (c8 & 3)) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) cs[((lane >> 5) * 4 + e) * PS + (lane & 7)] = acc[i][j][4 * gq + e];
                }
}

// probe_tile's decision and record for one tile, from the float32 operands
// themselves and on the float64 matrix cores: one v_mfma_f64_16x16x4_f64 takes
// eight k at once, rows and columns 0-7 holding the sampled rows and columns
// at k .. k + 3, rows and columns 8-15 the same ones at k + 4 .. k + 7; the two
// diagonal 8 x 8 blocks of its result are the two halves of the 64 samples'
// sums.  Operand lane l: row (column) l % 16, k l / 16; result register r of
// lane l: row 4 r + l / 16, column l % 16.  Every sampled element is loaded
// once (eight 32-byte pieces per load), and the sums need 8 registers and no
// exchange but the last one: with one float64 accumulator per sample in
// vector registers instead (64 of them a thread, then a butterfly over the
// wavefront) the probe took 10 us of a 15 us call at LEN = 64.  The tile has
// just streamed the same operands, so these reads hit the L2.  L.c holds the
// samples of C (probe_samples): the tile's stores of C need not have finished.
template <int THREADS>
__device__ __attribute__((always_inline)) inline bool probe_direct(const DirectArgs &g, int bm, int bn, int64_t tile,
                                                                   int tm, int tn, double tau2,
                                                                   ProbeRecord *__restrict__ rec, DirectProbeLds &L)
{
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    constexpr int WAVES = THREADS / 64, U = WAVES <= 4 ? 8 : 4;  // U steps of 8 k in flight per wavefront, twice
    static_assert(PS == 8 && WAVES <= 16, "8 x 8 samples");
    const int64_t row0 = (int64_t)tm * bm, col0 = (int64_t)tn * bn;
    const int rext = (int)min<int64_t>(bm, g.M - row0), cext = (int)min<int64_t>(bn, g.N - col0);
    const int l = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kq = ((l & 15) >> 3) * 4 + (l >> 4);  // this lane's k within a step
    const uint32_t offA = ((uint32_t)probe_pick(tile, l & 7, rext, 0) * (uint32_t)g.lda + kq) * 4u;
    const uint32_t colB = (uint32_t)probe_pick(tile, l & 7, cext, 1);
    const uint32_t offB = ((uint32_t)kq * (uint32_t)g.ldb + colB) * 4u;
    const float *pA = g.A + row0 * g.lda, *pB = g.B + col0;
    const uint32_t strideB = (uint32_t)(8 * WAVES * g.ldb * 4);  // bytes between a wavefront's steps
    const int K = (int)g.K;
    float xa[2][U], xb[2][U];
    // U steps from k0 on, 8 WAVES apart; elements past K read the last one and
    // count as zero
    auto load = [&](int k0, float (&va)[U], float (&vb)[U]) {
        if (k0 + (U - 1) * 8 * WAVES + 8 <= K) {
            const auto ra = buffer_of(pA + k0), rb = buffer_of(pB + k0 * g.ldb);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                va[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, offA, u * 8 * WAVES * 4, 0));
                vb[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, offB, u * strideB, 0));
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + u * 8 * WAVES + kq, kc = min(k, K - 1);
                const float x = pA[(int64_t)(offA / 4u - kq) + kc], y = pB[(int64_t)kc * g.ldb + colB];
                va[u] = k < K ? x : 0.0f;
                vb[u] = k < K ? y : 0.0f;
            }
        }
    };
    f64x4 d = {0.0, 0.0, 0.0, 0.0};
    auto sum = [&](const float (&va)[U], const float (&vb)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            d = __builtin_amdgcn_mfma_f64_16x16x4f64((double)va[u], (double)vb[u], d, 0, 0, 0);
    };
    constexpr int STEP = U * 8 * WAVES;
    if (wave * 8 < K) load(wave * 8, xa[0], xb[0]);
    for (int k0 = wave * 8; k0 < K; k0 += 2 * STEP) {
        if (k0 + STEP < K) load(k0 + STEP, xa[1], xb[1]);
        sum(xa[0], xb[0]);
        if (k0 + 2 * STEP < K) load(k0 + 2 * STEP, xa[0], xb[0]);
        if (k0 + STEP < K) sum(xa[1], xb[1]);
    }
    // lane l, column c: the sums of samples (l / 16, c % 8) and (l / 16 + 4,
    // c % 8) over its block's half of the k
    const bool hi = (l & 8) != 0;
    double s0 = hi ? d[2] : d[0], s1 = hi ? d[3] : d[1];
    s0 += __shfl_xor(s0, 8, 64);
    s1 += __shfl_xor(s1, 8, 64);
    if (!hi) {
        L.part[wave][(l >> 4) * PS + (l & 7)] = s0;
        L.part[wave][((l >> 4) + 4) * PS + (l & 7)] = s1;
    }
    return probe_decide<WAVES>(L.part, L.c, g.C, g.ldc, row0, col0, rext, cext, tile, tau2, rec, &L.marked);
}

}  // namespace dev
}  // namespace accx
