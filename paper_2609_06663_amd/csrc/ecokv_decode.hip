// ecokv_decode kernels (gfx950): attention of one new query per (layer, query
// head, sequence) over the compressed cache written by ecokv_compact -- the
// generation step that reads the kept rows (Sec. 3).
//
// Split over rows (flash-decoding): every block takes a chunk of one unit's
// rows (see DecodePlan) for query heads QG z .. QG z + QG - 1 of the unit's G;
// each of its four waves takes a quarter of the chunk.  q.k runs on the matrix
// cores, 16 rows per tile, P goes through LDS into the layout of the coalesced
// V loads (one or two heads of fp32 rows: both on the vector ALUs, in that
// layout), P.V is fp32 FMAs, and the next tile's rows load while one is used.
// The online softmax is kept in base 2.  A block merges its waves in LDS and
// writes one (max, sum, acc[D]) per query to the workspace; k_decode_merge or,
// for few chunks, k_decode_merge_few combines a query row's chunks.
#include "ecokv_internal.h"

namespace ecokv {

typedef unsigned int u32x4d __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8d __attribute__((ext_vector_type(8)));

constexpr int kDecThreads = 256;
static_assert(kDecWaves == kDecThreads / kWave && kPlanUnits == kPlanPer * kWave, "the plan's block");

// Which chunk a block takes.
//  * Fixed (a.plan == 0, and past two rounds): every unit in a.np chunks (or
//    fewer, of at least kMinWaveRows rows per wave), block b chunk b / U of
//    unit b % U, so that the blocks past the shorter units, which end at once,
//    come last.
//  * Balanced: the counts are on the device, so every wave reads them all,
//    gives every chunk of the call the same number of rows and finds its
//    block's chunk by a prefix sum.  Chunks of a fixed length leave compute
//    units idle when there are few rows, and with each unit split into the
//    same number of chunks the long ones of ragged units finish last.  About
//    one block per compute unit while its waves then take at most kOneRows
//    rows each, else two; past two rounds of kWaveRows rows the fixed chunks.
//    (us, fixed 768-row chunks -> now: one layer's 4 units of 6553 rows 16 ->
//    8.2; 16 sequences with budgets shared over 4 heads 36 -> 25; 8 packed
//    sequences 27 -> 14.5; 32 units of 2048 rows 15 -> 10.3; 4 layers of 4
//    fp32 units of 6553 rows 54 -> 27, half of it from the matrix cores.)
struct DecodePlan {
    int u, c, n, off, wave_rows;  // unit, chunk, the unit's rows and offset, rows per wave
};

__device__ __forceinline__ bool decode_plan(const DecodeArgs &a, int b, DecodePlan &p)
{
    const int U = a.L * a.Hkv * a.B;
    // the fixed chunk's, read beside the plan's so that falling back costs no round trip
    const int fixed_u = b % U;
    int fixed_n = uniform_i32(a.counts[fixed_u]), fixed_off = uniform_i32(a.offsets[fixed_u]);
    if (a.plan) {
        const int lane = threadIdx.x & 63;
        // four units' counts and offsets per lane (zero past the last unit)
        static_assert(kPlanPer == 4, "one 16-byte load");
        const auto units4 = [&](const int32_t *p) {
            const __amdgpu_buffer_rsrc_t r =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(p), (short)0, U * 4, 0x00020000);
            return __builtin_bit_cast(u32x4d, __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16, 0, 0));
        };
        const u32x4d cnt = units4(a.counts), off = units4(a.offsets);
        int n[kPlanPer];
        float sum = 0.f;
#pragma unroll
        for (int q = 0; q < kPlanPer; ++q) {
            n[q] = max(0, min((int)cnt[q], a.max_count));  // more rows than max_count: the merge writes NaN
            sum += (float)n[q];  // (a float: only the rows per wave come from it, alike in every wave)
        }
        p.wave_rows = uniform_i32(plan_wave_rows(wave_sum(sum), a.scale));
        if (p.wave_rows > 0) {
            int parts[kPlanPer], mine = 0;
#pragma unroll
            for (int q = 0; q < kPlanPer; ++q) {
                parts[q] = unit_chunks(n[q], p.wave_rows);
                mine += parts[q];
            }
            const int end = (int)wave_incl_scan((uint32_t)mine);
            const unsigned long long own = __builtin_amdgcn_ballot_w64(b < end && b >= end - mine);
            if (own == 0) return false;  // past the last chunk
            const int ol = __builtin_ctzll(own);
            int first = __builtin_amdgcn_readlane(end - mine, ol);
#pragma unroll
            for (int q = 0; q < kPlanPer; ++q) {
                const int pq = __builtin_amdgcn_readlane(parts[q], ol);
                if (b >= first && b < first + pq) {
                    p.u = kPlanPer * ol + q;
                    p.c = b - first;
                    p.n = __builtin_amdgcn_readlane(n[q], ol);
                    p.off = __builtin_amdgcn_readlane((int)off[q], ol);
                    if (p.c == 0 && threadIdx.x == 0) a.tab[p.u] = make_int2(b, pq);
                }
                first += pq;
            }
            return true;
        }
    }
    p.u = fixed_u;
    p.c = b / U;
    p.n = max(0, min(fixed_n, a.max_count));
    p.off = fixed_off;
    if (a.plan && p.c == 0 && threadIdx.x == 0) a.tab[p.u] = make_int2(0, 0);  // (fixed chunks)
    p.wave_rows = fixed_wave_rows(p.n, a.np);
    return (int64_t)p.c * (kDecWaves * p.wave_rows) < p.n;
}

template <bool BF16>
__device__ __forceinline__ void unpack(const u32x4d &x, float (&f)[BF16 ? 8 : 4])
{
    if constexpr (BF16) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            f[2 * c] = __uint_as_float(x[c] << 16);
            f[2 * c + 1] = __uint_as_float(x[c] & 0xffff0000u);
        }
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) f[c] = __uint_as_float(x[c]);
    }
}

// Q.K^T on the matrix cores, P.V on the vector ALUs in fp32.
//  * Tile of 16 rows: the rows as A (lane l: row l % 16, 16 bytes at 64 st +
//    16 (l / 16) of the row for step st, so each load instruction reads 64
//    contiguous bytes of 16 rows) and the block's query heads as B (lane l:
//    head l % 16, the same bytes; heads >= nq are zero).  Both operands take
//    dimension j of a row from the same lane group and element, so the
//    contraction is exact whatever order the instruction sums its products
//    in: v_mfma_f32_16x16x32_bf16 per step, or, for fp32 rows, four
//    v_mfma_f32_16x16x4_f32 (fp32 products and sums).  Lane l then holds the
//    logits of rows 4 (l / 16) .. +3 against head l % 16.
//  * Online softmax per head, base 2, with a lazy reference: the running
//    maximum m moves only when a batch exceeds it by more than 2^8, so the
//    fp32 P.V accumulators are rescaled rarely (one wave-uniform branch).
//  * P goes through a wave-private LDS tile into the V layout (lane l: row
//    RPI i + l / S, bytes 16 (l % S)) and P.V accumulates there.
// fp32 rows for one or two query heads (kVector) take q.k on the vector ALUs
// instead: the rows in the V layout, four products per lane and the S lanes of
// a row added by butterflies.  The 32 (16) serial fp32 matrix instructions of a
// tile cost more than that for so few heads, and without them the loads are
// whole lines and four waves share a SIMD (the call, us, 128-wide rows and one
// query head, matrix -> vector: 4 units of 1500 rows 19.8 -> 12.3, 32 of 2048
// 17.1 -> 14.5, 112 of 6553 122 -> 117; two heads 20.0 -> 17.1, 17.3 -> 14.8,
// 123 -> 119.  Four heads have the matrix form: 112 of 6553 129 against 138).
constexpr float kDecRebase = 8.f;

template <bool BF, int QG>
constexpr bool kVector = !BF && QG <= 2;

// The register budget: with bf16 rows 168, so that three waves share a SIMD.
template <bool BF, int D, int QG>
__global__ __launch_bounds__(kDecThreads, (kVector<BF, QG> ? 4 : BF ? 3 : 2)) void k_decode(DecodeArgs a)
{
    constexpr bool VEC = kVector<BF, QG>;
    constexpr int RB = D * (BF ? 2 : 4);  // row bytes
    constexpr int EL = BF ? 8 : 4;        // elements per 16 bytes
    constexpr int S = RB / 16;            // lanes per row in the V layout
    constexpr int RPI = kWave / S;        // V rows per load instruction
    constexpr int BR = VEC ? 4 * RPI : 16;  // rows per tile
    constexpr int NV = BR / RPI;          // V load instructions per tile
    constexpr int KS = VEC ? NV : RB / 64;  // K load instructions per tile
    constexpr int MS = VEC ? QG : 1;      // softmax states per lane
    constexpr int QP = QG < 4 ? 4 : QG;   // floats per row of the P tile
    typedef float f32x4d __attribute__((ext_vector_type(4)));
    __shared__ float cm[kDecWaves][QG], cl[kDecWaves][QG];
    __shared__ float cacc[kDecWaves][QG][D];
    __shared__ __attribute__((aligned(16))) float pt[VEC ? 1 : kDecWaves][BR][QP];
    const int index = blockIdx.z * kGridX + blockIdx.x;
    const DecodePlace place = QG == kDecQG && a.zg > 1 ? decode_place(index, a.zg) : DecodePlace{index, 0};
    const int block = place.block, z = place.z;
    DecodePlan pl;
    if (!decode_plan(a, block, pl)) return;  // (the whole block; those past the last too)
    const Unit un = unit_of(pl.u, a.Hkv, a.B);
    const int lane = threadIdx.x & 63, wv = uniform_i32(threadIdx.x >> 6);
    const int r16 = lane & 15, kg = lane >> 4, seg = lane % S, rg = lane / S;
    const int64_t off = pl.off;
    const int nq = min(QG, a.G - z * QG);
    // the query heads as operand B; vector form: this lane's 16 bytes of each head
    u32x4d qb[VEC ? QG : KS];
    {
        const int64_t q0 = (int64_t)un.l * a.Hq + un.h * a.G + z * QG;
        if constexpr (VEC) {
#pragma unroll
            for (int g = 0; g < QG; ++g)
                qb[g] = *reinterpret_cast<const u32x4d *>(static_cast<const char *>(a.Q) +
                                                          ((q0 + min(g, nq - 1)) * a.B + un.s) * RB + 16 * seg);
        } else {
            const char *qp = static_cast<const char *>(a.Q) + ((q0 + min(r16, nq - 1)) * a.B + un.s) * RB + 16 * kg;
#pragma unroll
            for (int st = 0; st < KS; ++st)
                qb[st] = r16 < nq ? *reinterpret_cast<const u32x4d *>(qp + 64 * st) : (u32x4d){0u, 0u, 0u, 0u};
        }
    }
    const int row0 = (pl.c * kDecWaves + wv) * pl.wave_rows;
    const int nrows = max(0, min(pl.n - row0, pl.wave_rows));

    const int64_t base = (off + row0) * RB;
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(uniform_ptr(static_cast<const char *>(a.Kc) + base)), (short)0, uniform_i32(nrows * RB),
        0x00020000);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(uniform_ptr(static_cast<const char *>(a.Vc) + base)), (short)0, uniform_i32(nrows * RB),
        0x00020000);

    // m, ls: head r16's (vector form: every head's) reference maximum and this
    // lane's part of its sum
    float m[MS], ls[MS], acc[QG][EL];
#pragma unroll
    for (int g = 0; g < MS; ++g) {
        m[g] = -INFINITY;
        ls[g] = 0.f;
    }
#pragma unroll
    for (int g = 0; g < QG; ++g)
#pragma unroll
        for (int e = 0; e < EL; ++e) acc[g][e] = 0.f;
    float *ptw = &pt[VEC ? 0 : wv][0][0];

    // every load is unconditional: rows past nrows read zero.  A Kc load
    // instruction covers 64 of a row's bytes, so two instructions share each
    // 128-byte line: those loads keep the default cache policy, and the
    // second finds the line the first brought in (nontemporal Kc loads took
    // 68 us instead of 62 on the 28-layer cache); the Vc loads, and the vector
    // form's Kc loads, cover whole lines and stream nontemporally.
    auto load = [&](u32x4d (&kx)[KS], u32x4d (&vx)[NV], int b0) {
#pragma unroll
        for (int st = 0; st < KS; ++st)
            kx[st] = __builtin_bit_cast(
                u32x4d, VEC ? __builtin_amdgcn_raw_buffer_load_b128(rk, (b0 + RPI * st) * RB + lane * 16, 0, 2)
                            : __builtin_amdgcn_raw_buffer_load_b128(rk, (b0 + r16) * RB + 64 * st + 16 * kg, 0, 0));
#pragma unroll
        for (int i = 0; i < NV; ++i)
            vx[i] = __builtin_bit_cast(u32x4d,
                                       __builtin_amdgcn_raw_buffer_load_b128(rv, (b0 + RPI * i) * RB + lane * 16, 0, 2));
    };
    auto tile = [&](const u32x4d (&kx)[KS], const u32x4d (&vx)[NV], int b0) {
        if constexpr (VEC) {
            float x[NV][QG];
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const bool valid = b0 + RPI * i + rg < nrows;
#pragma unroll
                for (int g = 0; g < QG; ++g) {
                    float pd = 0.f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) pd = fmaf(__uint_as_float(qb[g][e]), __uint_as_float(kx[i][e]), pd);
                    pd = row_sum<S>(pd);  // (every lane takes part)
                    x[i][g] = valid ? pd * a.qscale : -INFINITY;
                }
            }
#pragma unroll
            for (int g = 0; g < QG; ++g) {
                float mb = x[0][g];
#pragma unroll
                for (int i = 1; i < NV; ++i) mb = fmaxf(mb, x[i][g]);
                if (S <= 16) mb = across16(mb, OpMax{});
                mb = across32(mb, OpMax{});  // (the same in every lane)
                if (__builtin_amdgcn_ballot_w64(mb > m[g] + kDecRebase)) {
                    const float sc = __builtin_amdgcn_exp2f(m[g] - mb);  // 0 while m = -inf
                    ls[g] *= sc;
                    m[g] = mb;
#pragma unroll
                    for (int e = 0; e < EL; ++e) acc[g][e] *= sc;
                }
                const float ref = m[g] == -INFINITY ? 0.f : m[g];
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const float p = __builtin_amdgcn_exp2f(x[i][g] - ref);
                    ls[g] += p;
#pragma unroll
                    for (int e = 0; e < EL; ++e) acc[g][e] = fmaf(p, __uint_as_float(vx[i][e]), acc[g][e]);
                }
            }
        } else {
            f32x4d cc = (f32x4d){0.f, 0.f, 0.f, 0.f};
            if constexpr (BF) {
#pragma unroll
                for (int st = 0; st < KS; ++st)
                    cc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8d, kx[st]),
                                                                __builtin_bit_cast(bf16x8d, qb[st]), cc, 0, 0, 0);
            } else {
                // each instruction's four products a run of its own, the runs as a tree:
                // as many roundings as a row's dimensions by fours on lanes added by
                // butterflies (eight runs of D / 8: the logits of 128 dimensions 5.7e-7
                // from float64 on average instead of 4.9e-7, 1 to 2 % less time)
                constexpr int RUNS = D / 4, LEVELS = D == 128 ? 5 : 4;
                f32x4d t[LEVELS + 1];
#pragma unroll
                for (int run = 0; run < RUNS; ++run) {
                    f32x4d x = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(kx[run / 4][run % 4]),
                                                                    __uint_as_float(qb[run / 4][run % 4]),
                                                                    (f32x4d){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    int l = 0;
#pragma unroll
                    for (; (run >> l) & 1; ++l) x = t[l] + x;
                    t[l] = x;
                }
                cc = t[LEVELS];
            }
            float x[4];
            float mb = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                x[r] = b0 + 4 * kg + r < nrows ? cc[r] * a.qscale : -INFINITY;
                mb = fmaxf(mb, x[r]);
            }
            mb = across32(across16(mb, OpMax{}), OpMax{});
            const bool move = mb > m[0] + kDecRebase;      // (from m = -inf: with the first finite logit)
            if (__builtin_amdgcn_ballot_w64(move)) {
                const float nm = move ? mb : m[0];
                const float sc = __builtin_amdgcn_exp2f(m[0] - nm);  // 0 while m = -inf
                ls[0] *= sc;
                m[0] = nm;
#pragma unroll
                for (int g = 0; g < QG; ++g) {
                    const float sg = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sc), g));
#pragma unroll
                    for (int e = 0; e < EL; ++e) acc[g][e] *= sg;
                }
            }
            const float ref = m[0] == -INFINITY ? 0.f : m[0];  // (weight 0 for logits of -inf, also before any other)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float p = __builtin_amdgcn_exp2f(x[r] - ref);
                ls[0] += p;
                if (r16 < QG) ptw[(4 * kg + r) * QP + r16] = p;
            }
            // (a wave's own LDS accesses are ordered)
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const float *prow = ptw + (RPI * i + rg) * QP;
                float pv[QP];
#pragma unroll
                for (int q4 = 0; q4 < QP / 4; ++q4) {
                    const f32x4d y = *reinterpret_cast<const f32x4d *>(prow + 4 * q4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) pv[4 * q4 + e] = y[e];
                }
                float vf[EL];
                unpack<BF>(vx[i], vf);
#pragma unroll
                for (int g = 0; g < QG; ++g)
#pragma unroll
                    for (int e = 0; e < EL; ++e) acc[g][e] = fmaf(pv[g], vf[e], acc[g][e]);
            }
        }
    };
    // two register buffers: the next tile's rows load while this one is used
    // (69 against 73 us on the 28-layer cache without)
    u32x4d ka[KS], va[NV], kb[KS], vb[NV];
    if (nrows > 0) load(ka, va, 0);
    for (int b0 = 0; b0 < nrows; b0 += 2 * BR) {
        load(kb, vb, b0 + BR);
        __builtin_amdgcn_sched_barrier(0);
        tile(ka, va, b0);
        if (b0 + BR >= nrows) break;
        load(ka, va, b0 + 2 * BR);
        __builtin_amdgcn_sched_barrier(0);
        tile(kb, vb, b0 + BR);
    }

    // P.V: add the row groups of the V layout (64 / S of them), each fold
    // leaving half of the elements in either half of the lanes, so that all
    // lanes end with EW elements of their segment; sums: add the four lane groups
    constexpr int EW = S <= 16 ? EL / 4 : EL / 2;
    const int e0 = (lane >= 32 ? EL / 2 : 0) + (S <= 16 && (lane & 16) ? EL / 4 : 0);
#pragma unroll
    for (int g = 0; g < QG; ++g) {
        if constexpr (S == 8) {
#pragma unroll
            for (int e = 0; e < EL; ++e) acc[g][e] += dpp_row<0x128>(acc[g][e]);  // row_ror:8, lane ^ 8
        }
#pragma unroll
        for (int e = 0; e < EL / 2; ++e) acc[g][e] = fold32(acc[g][e], acc[g][e + EL / 2]);
        if constexpr (S <= 16) {
#pragma unroll
            for (int e = 0; e < EL / 4; ++e) acc[g][e] = fold16(acc[g][e], acc[g][e + EL / 4]);
        }
        if (S > 8 || !(lane & 8)) {
#pragma unroll
            for (int e = 0; e < EW; ++e) cacc[wv][g][seg * EL + e0 + e] = acc[g][e];
        }
    }
#pragma unroll
    for (int g = 0; g < MS; ++g) {
        if (!VEC || S <= 16) ls[g] = across16(ls[g], OpAdd{});
        ls[g] = across32(ls[g], OpAdd{});
    }
    if (VEC ? lane == 0 : lane < QG) {
#pragma unroll
        for (int g = 0; g < MS; ++g) {
            cm[wv][VEC ? g : lane] = m[g];
            cl[wv][VEC ? g : lane] = ls[g];
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < nq * D; t += kDecThreads) {
        const int g = t / D, d = t - g * D;
        float M = cm[0][g];
        for (int w2 = 1; w2 < kDecWaves; ++w2) M = fmaxf(M, cm[w2][g]);
        float L = 0.f, A = 0.f;
        // (waves without a finite logit add 0, or their NaN, also where all are such)
        const float ref = M == -INFINITY ? 0.f : M;
        for (int w2 = 0; w2 < kDecWaves; ++w2) {
            const float wt = exp2f(cm[w2][g] - ref);
            L += cl[w2][g] * wt;
            A += cacc[w2][g][d] * wt;
        }
        float *pp = a.part + ((int64_t)block * a.G + z * QG + g) * (D + 2);
        pp[2 + d] = A;
        if (d == 0) {
            pp[0] = M;
            pp[1] = L;
        }
    }
}

// The partials of query row qrow: (max, sum, accumulator) of its unit's chunks,
// `step` floats apart.
struct MergeRow {
    const float *pp;
    int64_t step;
    int used;
    bool bad;
};
__device__ __forceinline__ MergeRow merge_row(const DecodeArgs &a, int64_t qrow)
{
    const int s = (int)(qrow % a.B), q = (int)((qrow / a.B) % a.Hq), l = (int)(qrow / ((int64_t)a.B * a.Hq));
    const int64_t u = ((int64_t)l * a.Hkv + q / a.G) * a.B + s;
    // the unit's chunks: blocks first, first + step, ...
    const int2 e = a.plan ? a.tab[u] : make_int2(0, 0);  // (not written for a unit without rows)
    const int n = a.counts[u], nn = max(0, min(n, a.max_count));
    int64_t first = u, step = (int64_t)a.L * a.Hkv * a.B;
    int used = unit_chunks(nn, fixed_wave_rows(nn, a.np));
    if (nn > 0 && e.y > 0) {
        first = e.x;
        used = e.y;
        step = 1;
    }
    step *= (int64_t)a.G * (a.D + 2);
    return MergeRow{a.part + (first * a.G + q % a.G) * (a.D + 2), step, used, n > a.max_count || n < 0};
}

// O and lse of dimension d of a query row from its merged (reference, sum, accumulator).
__device__ __forceinline__ void merge_write(const DecodeArgs &a, int64_t qrow, int d, bool bad, float M, float L, float o)
{
    // (L is 0 without rows and where every logit is -inf, NaN where one is)
    a.O[qrow * a.D + d] = bad ? NAN : (L == 0.f ? 0.f : o / L);
    if (d == 0 && a.lse) a.lse[qrow] = bad ? NAN : (L == 0.f ? -INFINITY : (M + log2f(L)) * 0.69314718055994531f);
}

// The merge of a few chunks: a thread per dimension, every chunk's (max, sum,
// accumulator) loaded at once, no exchange between threads (4 units of 1500
// rows: 3.0 us against 4.0 with the general form below).
constexpr int kMergeFew = 16;
__device__ __forceinline__ void merge_few(const DecodeArgs &a, const MergeRow &row, int64_t qrow)
{
    const int t = threadIdx.x;
    if (t >= a.D) return;
    float cmx[kMergeFew], csm[kMergeFew], cac[kMergeFew], M = -INFINITY, L = 0.f, o = 0.f;
#pragma unroll
    for (int p = 0; p < kMergeFew; ++p) {
        const float *r = row.pp + min(p, max(row.used - 1, 0)) * row.step;
        cmx[p] = p < row.used ? r[0] : -INFINITY;
        csm[p] = r[1];
        cac[p] = r[2 + t];
    }
#pragma unroll
    for (int p = 0; p < kMergeFew; ++p) M = fmaxf(M, cmx[p]);
    const float ref = M == -INFINITY ? 0.f : M;
#pragma unroll
    for (int p = 0; p < kMergeFew; ++p) {
        const float w = exp2f(cmx[p] - ref);
        if (p < row.used) {
            L += csm[p] * w;
            o += cac[p] * w;
        }
    }
    merge_write(a, qrow, t, row.bad, M, L, o);
}
__global__ __launch_bounds__(128) void k_decode_merge_few(DecodeArgs a)
{
    const int64_t qrow = (int64_t)blockIdx.y * kGridX + blockIdx.x;
    if (blockIdx.y > 0 && qrow >= (int64_t)a.L * a.Hq * a.B) return;
    merge_few(a, merge_row(a, qrow), qrow);
}

// One block per query row: the log-sum-exp merge of its chunks, 256 at a time.
// Thread t weighs chunk t; D x (256 / D) threads add up the accumulators, each
// over every (256 / D)-th chunk, the first kMergeRegs of them loaded together
// with the maxima and sums: 16 (one round of latency for up to 32 chunks of
// 128 dimensions; one layer's 52 chunks per row 4.4 us against 5.9 with 8),
// or 8 for calls of so many rows that the registers cost more blocks in
// flight than a round of latency (784 rows: 6.2 us against 7.2 with 16).
constexpr int kMergeThreads = 256;

template <int kMergeRegs>
__global__ __launch_bounds__(kMergeThreads) void k_decode_merge(DecodeArgs a)
{
    __shared__ float wt[kMergeThreads], red[2][kMergeThreads / kWave], osum[kMergeThreads];
    const int64_t qrow = (int64_t)blockIdx.y * kGridX + blockIdx.x;
    if (blockIdx.y > 0 && qrow >= (int64_t)a.L * a.Hq * a.B) return;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const MergeRow row = merge_row(a, qrow);
    const int used = row.used;
    const bool bad = row.bad;
    const float *pp = row.pp;
    const int64_t step = row.step;
    if (used <= kMergeFew) {
        merge_few(a, row, qrow);
        return;
    }
    const int d = t % a.D, grp = t / a.D, ngrp = kMergeThreads / a.D;
    float M = -INFINITY, L = 0.f, o = 0.f;
    for (int p0 = 0; p0 < used; p0 += kMergeThreads, pp += kMergeThreads * step) {
        // the next chunks against the running (M, L, o)
        const int np = min(used - p0, kMergeThreads);
        const float cmx = t < np ? pp[t * step] : -INFINITY, csm = t < np ? pp[t * step + 1] : 0.f;
        // this thread's chunks p = grp, grp + ngrp, ...: kMergeRegs at a time
        const float *ac = pp + 2 + d;
        float acr[kMergeRegs];
#pragma unroll
        for (int j = 0; j < kMergeRegs; ++j) acr[j] = ac[min(grp + j * ngrp, np - 1) * step];
        const float mx = wave_max(cmx);
        if (lane == 0) red[0][wv] = mx;
        lds_barrier();
        float nm = M;
#pragma unroll
        for (int w2 = 0; w2 < kMergeThreads / kWave; ++w2) nm = fmaxf(nm, red[0][w2]);
        const float w = cmx == -INFINITY ? 0.f : exp2f(cmx - nm);
        wt[t] = w;
        const float ws = wave_sum(csm * w);
        if (lane == 0) red[1][wv] = ws;
        lds_barrier();
        const float sc = M == -INFINITY ? 0.f : exp2f(M - nm);
        L *= sc;
        o *= sc;
#pragma unroll
        for (int w2 = 0; w2 < kMergeThreads / kWave; ++w2) L += red[1][w2];
        M = nm;
        for (int j0 = grp; j0 < np; j0 += kMergeRegs * ngrp) {
            if (j0 != grp)
#pragma unroll
                for (int j = 0; j < kMergeRegs; ++j) acr[j] = ac[min(j0 + j * ngrp, np - 1) * step];
#pragma unroll
            for (int j = 0; j < kMergeRegs; ++j)
                o = fmaf(acr[j], j0 + j * ngrp < np ? wt[(j0 + j * ngrp) & (kMergeThreads - 1)] : 0.f, o);
        }
        lds_barrier();  // wt and red are free again
    }
    osum[t] = o;
    __syncthreads();
    if (t < a.D) {
        for (int g2 = 1; g2 < ngrp; ++g2) o += osum[g2 * a.D + t];
        merge_write(a, qrow, t, bad, M, L, o);
    }
}

template <bool BF, int D>
static void launch_dec(const DecodeArgs &a, dim3 grid, hipStream_t st)
{
    const int qg = decode_qg(a.G);
    if (qg == 8) hipLaunchKernelGGL((k_decode<BF, D, 8>), grid, dim3(kDecThreads), 0, st, a);
    else if (qg == 4) hipLaunchKernelGGL((k_decode<BF, D, 4>), grid, dim3(kDecThreads), 0, st, a);
    else if (qg == 2) hipLaunchKernelGGL((k_decode<BF, D, 2>), grid, dim3(kDecThreads), 0, st, a);
    else hipLaunchKernelGGL((k_decode<BF, D, 1>), grid, dim3(kDecThreads), 0, st, a);
}

size_t decode_ws_bytes(int64_t units, int G, int D, int max_count, bool least)
{
    return decode_grid(units, G, D, max_count, least).bytes;
}

hipError_t decode_launch(DecodeArgs a, char *ws, size_t ws_bytes, bool bf16, hipStream_t st)
{
    const int64_t U = (int64_t)a.L * a.Hkv * a.B;
    if (U == 0) return hipSuccess;
    DecodeGrid g = decode_grid(U, a.G, a.D, a.max_count, false);
    if (ws_bytes < g.bytes) g = decode_grid(U, a.G, a.D, a.max_count, true);
    if (decode_places(g.blocks, decode_head_groups(a.G)) > INT32_MAX - kGridX) return hipErrorInvalidConfiguration;
    a.plan = g.plan;
    if (g.plan) a.scale = plan_scale(U, g.plan, a.max_count);
    a.np = g.np;
    a.part = reinterpret_cast<float *>(ws);
    a.tab = g.plan ? reinterpret_cast<int2 *>(ws + g.bytes - sizeof(int2) * (size_t)U) : nullptr;
    auto along_x = [](int64_t n) { return (unsigned)(n < kGridX ? n : kGridX); };
    auto rest = [](int64_t n) { return (unsigned)((n + kGridX - 1) / kGridX); };
    a.zg = decode_head_groups(a.G);
    const int64_t n = decode_places(g.blocks, a.zg);
    const dim3 grid(along_x(n), 1, rest(n));
    if (bf16 && a.D == 128) ECOKV_TIMED("decode", st, (launch_dec<true, 128>(a, grid, st)));
    else if (bf16) ECOKV_TIMED("decode", st, (launch_dec<true, 64>(a, grid, st)));
    else if (a.D == 128) ECOKV_TIMED("decode", st, (launch_dec<false, 128>(a, grid, st)));
    else ECOKV_TIMED("decode", st, (launch_dec<false, 64>(a, grid, st)));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t rows = (int64_t)a.L * a.Hq * a.B;
    const dim3 merge(along_x(rows), rest(rows));
    // (a balanced plan's chunks are kDecWaves kMinWaveRows rows at least)
    const int most = g.plan ? unit_chunks(a.max_count, kMinWaveRows) : g.np;
    if (most <= kMergeFew)
        ECOKV_TIMED("decode_merge", st, hipLaunchKernelGGL(k_decode_merge_few, merge, dim3(128), 0, st, a));
    else if (rows >= 512)
        ECOKV_TIMED("decode_merge", st, hipLaunchKernelGGL(k_decode_merge<8>, merge, dim3(kMergeThreads), 0, st, a));
    else
        ECOKV_TIMED("decode_merge", st, hipLaunchKernelGGL(k_decode_merge<16>, merge, dim3(kMergeThreads), 0, st, a));
    return hipGetLastError();
}

}  // namespace ecokv
