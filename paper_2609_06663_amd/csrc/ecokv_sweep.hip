// The two sweeps of ecokv_score over K for every shape that the 32-row
// streaming kernels do not take (gfx950): fp32 keys, head_dim 64, and more
// window rows than one 32-row operand holds.
//
// Both stream K as they do: each of a block's four waves takes a quarter of
// the block's keys in batches of 8 KiB (16 fp32 or 32 bf16 keys of 128
// dimensions, 32 or 64 of 64), eight coalesced 16-byte buffer loads per batch
// and two batches in flight in registers, and no barrier in the key loop.  A
// batch goes through a wave-private LDS stage (swizzled 16-byte chunks) into
// the operand layout of the 16 x 16 matrix instructions: lane l holds key
// l % 16 of each 16-key tile, chunks 4 st + l / 16.  A contraction may take
// its dimensions in any order as long as both operands agree, so the same
// registers serve
//   * q.k on the matrix cores: v_mfma_f32_16x16x32_bf16 per chunk, or, for
//     fp32 keys, four v_mfma_f32_16x16x4_f32 (fp32 products and sums) per
//     chunk, MT tiles of 16 window rows;
//   * everything per key (|k|^2, |k - kbar|^2, k.mu) as fp32 sums over the
//     lane's quarter of the dimensions, added over the four lane groups;
//   * the column sums as one fp32 accumulator per dimension and lane.
// R = (H_q / H_kv) w is padded to 16, 32 or 64 rows.
#include "ecokv_fast.h"

namespace ecokv {
namespace rows {

typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef u32x4 __attribute__((aligned(2))) u32x4_a2;  // 16 bytes at any element's alignment (buffer loads take any)

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kBatchBytes = 8192;
constexpr float kRebase = 16.f;  // log2 headroom of the lazily moved softmax reference

template <bool BF, int D>
struct Geo {
    static constexpr int RB = D * (BF ? 2 : 4);    // row bytes
    static constexpr int CR = RB / 16;             // 16-byte chunks per row
    static constexpr int BK = kBatchBytes / RB;    // keys per batch
    static constexpr int NT = BK / 16;             // 16-key tiles per batch
    static constexpr int HT = BF ? 2 : 1;          // tiles in registers at once
    static constexpr int NCH = CR / 4;             // chunks of a key in one lane
    static constexpr int EL = BF ? 8 : 4;          // elements per chunk
    static constexpr int DL = D / 4;               // dimensions in one lane
    static constexpr int kMaxKeys = BF ? 2048 : 1024;  // keys per block at most (the output stage)
    // Position of chunk c of row r in the stage: 16 rows read at one chunk
    // column, and the chunks of a row written together, fall on different banks.
    static __device__ __forceinline__ int pos(int r, int c) { return r * CR + (c ^ (CR == 8 ? (r >> 1) & 7 : r & 15)); }
};

// Batch g of the wave's keys (key0 .. key0 + BK - 1): 1 KiB per instruction,
// nontemporal; keys past the descriptor's end read as zero.
__device__ __forceinline__ void batch_load(u32x4 (&b)[8], __amdgpu_buffer_rsrc_t rs, int byte0, int lane)
{
#pragma unroll
    for (int i = 0; i < 8; ++i)
        b[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, byte0 + i * 1024 + lane * 16, 0, 2);
}

template <bool BF>
__device__ __forceinline__ void unpack_chunk(u32x4 q, float (&v)[BF ? 8 : 4])
{
    if constexpr (BF) {
        fast::unpack8(q, v);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(q[e]);
    }
}

// c += A B over one chunk of 16 rows (A) and 16 columns (B).
__device__ __forceinline__ f32x4v mfma_chunk(u32x4 x, u32x4 y, f32x4v c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c, 0, 0,
                                                  0);
}

// |k|^2 over the lane's dimensions of a chunk.
template <bool BF>
__device__ __forceinline__ float sq_chunk(u32x4 q, float s)
{
    if constexpr (BF) return fast::dot2sq(q[0], fast::dot2sq(q[1], fast::dot2sq(q[2], fast::dot2sq(q[3], s))));
    float v[BF ? 8 : 4];
    unpack_chunk<BF>(q, v);
#pragma unroll
    for (int e = 0; e < (BF ? 8 : 4); ++e) s = fmaf(v[e], v[e], s);
    return s;
}

// The unit's window rows as matrix operands: entry (mt, st, lane) is chunk
// 4 st + lane / 16 of window row 16 mt + lane % 16 (zero past R).  Their loads
// go out ahead of the first batches (loads return in order: behind them the
// set-up would wait for the keys), put() writes them to LDS (one 8192-token
// layer with 56 window rows, the anchors likewise: score 34.1 -> 31.7 us).
template <bool BF, int D, int MT>
struct Queries {
    using G = Geo<BF, D>;
    static constexpr int kAll = MT * G::NCH * 64, kPer = (kAll + kThreads - 1) / kThreads;
    u32x4 q[kPer];
    __device__ __forceinline__ void load(const ScoreArgs &a, const Unit &un)
    {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = k * kThreads + (int)threadIdx.x;
            const int l = i & 63, st = (i >> 6) % G::NCH, mt = (i >> 6) / G::NCH, r = 16 * mt + (l & 15);
            q[k] = *reinterpret_cast<const u32x4_a2 *>(static_cast<const char *>(a.Q) +
                                                       window_row(a, un, r < a.R ? r : 0) * G::RB + (4 * st + (l >> 4)) * 16);
        }
    }
    __device__ __forceinline__ void put(const ScoreArgs &a, u32x4 *qs) const
    {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = k * kThreads + (int)threadIdx.x;
            if (i >= kAll) break;  // (one 16-row tile of 64-wide bf16 rows: half the threads)
            const int r = 16 * ((i >> 6) / G::NCH) + (i & 15);
            qs[i] = r < a.R ? q[k] : (u32x4){0u, 0u, 0u, 0u};
        }
    }
};

// acc[mt][nt] = tiles of q.k, with the keys as the rows (A) if KEYS_A, else
// as the columns (B).
template <bool BF, int D, int MT, bool KEYS_A>
__device__ __forceinline__ void logits(const u32x4 (&kx)[Geo<BF, D>::HT][Geo<BF, D>::NCH], const u32x4 *qs, int lane,
                                       f32x4v (&acc)[MT][Geo<BF, D>::HT])
{
    using G = Geo<BF, D>;
    if constexpr (BF) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < G::HT; ++nt) acc[mt][nt] = (f32x4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < G::NCH; ++st) {
            // a chunk at a time: the operands of all at once would spill
            if (MT > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const u32x4 q = qs[(mt * G::NCH + st) * 64 + lane];
#pragma unroll
                for (int nt = 0; nt < G::HT; ++nt) {
                    // (64 dimensions are two instructions: their sums are added, not chained)
                    const f32x4v c0 = G::NCH > 2 ? acc[mt][nt] : (f32x4v){0.f, 0.f, 0.f, 0.f};
                    const f32x4v c = KEYS_A ? mfma_chunk(kx[nt][st], q, c0) : mfma_chunk(q, kx[nt][st], c0);
                    acc[mt][nt] = G::NCH > 2 || st == 0 ? c : acc[mt][nt] + c;
                }
            }
        }
    } else {
        // fp32 products are summed in 16 runs of D / 16, the runs as a tree, which
        // rounds as often as 16 lanes' dot products added by butterflies (eight
        // runs of D / 8: the logits of 128 dimensions 5.7e-7 from float64 instead of
        // 5.1e-7, logits of 6; for 3 to 6 % of a score: 28 layers of 4 x 16384 x
        // 128 with 28 window rows 437 -> 452 us, of 64 dimensions 262 -> 278)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (MT > 1) __builtin_amdgcn_sched_barrier(0);
            f32x4v t[5][G::HT];  // sums of 1, 2, 4, 8, 16 runs
#pragma unroll
            for (int run = 0; run < 16; ++run) {
                constexpr int RE = D / 64;  // instructions per run (2 or 1 of the chunk's elements)
                const int st = run * RE / 4, e0 = run * RE % 4;
                const u32x4 q = qs[(mt * G::NCH + st) * 64 + lane];
#pragma unroll
                for (int nt = 0; nt < G::HT; ++nt) {
                    const u32x4 x = KEYS_A ? kx[nt][st] : q, y = KEYS_A ? q : kx[nt][st];
                    f32x4v c = (f32x4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int e = e0; e < e0 + RE; ++e)
                        c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x[e]), __uint_as_float(y[e]), c, 0, 0, 0);
                    int l = 0;
#pragma unroll
                    for (; (run >> l) & 1; ++l) c = t[l][nt] + c;
                    // (four runs in flight: all 16 at once would spill)
                    if (D == 128 && run % 4 == 3) asm volatile("" : "+v"(c));
                    t[l][nt] = c;
                }
            }
#pragma unroll
            for (int nt = 0; nt < G::HT; ++nt) acc[mt][nt] = t[4][nt];
        }
    }
}

// The wave's key range, its batches and their loads.  Waves start at a
// rotated batch, so that at any moment they read different offsets of equally
// sized, equally aligned ranges.
template <bool BF, int D>
struct Stream {
    using G = Geo<BF, D>;
    int wbase, wkeys, ng, rot;
    __amdgpu_buffer_rsrc_t rs;
    __device__ __forceinline__ Stream(const ScoreArgs &a, const Unit &un, int row_base, int rpb, int T, int wv)
    {
        const int per = rpb / kWaves;
        wbase = row_base + wv * per;
        wkeys = uniform_i32(max(0, min(per, T - wbase)));
        ng = (wkeys + G::BK - 1) / G::BK;
        rot = uniform_i32((int)__umulhi((unsigned)((blockIdx.y * gridDim.x + blockIdx.x) * kWaves + wv) * 2654435761u, (unsigned)ng));
        const char *p = uniform_ptr(static_cast<const char *>(a.K) + (unit_row0(a, un) + wbase) * G::RB);
        rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), (short)0, wkeys * G::RB, 0x00020000);
    }
    // first key of slot g within the wave's range (slots past ng: past the range, zeros)
    __device__ __forceinline__ int key(int g) const { return G::BK * (g < ng ? (g + rot < ng ? g + rot : g + rot - ng) : ng); }
    __device__ __forceinline__ void load(u32x4 (&b)[8], int g, int lane) const
    {
        batch_load(b, rs, key(g) * G::RB, lane);
    }
    // The first two batches, issued right behind the block's set-up loads
    // (window rows, anchors), which are used while they are in flight.
    __device__ __forceinline__ void prefetch(u32x4 (&b)[2][8], int lane) const
    {
        load(b[0], 0, lane);
        load(b[1], 1, lane);
        __builtin_amdgcn_sched_barrier(0);
    }
    // f(batch, first key within the sequence) over the wave's batches,
    // the first two in b: two batches stay in flight while one is used; every
    // load is unconditional, so each wait covers only the batch about to be used
    template <class F>
    __device__ __forceinline__ void run(u32x4 (&b)[2][8], int lane, F &&f) const
    {
        u32x4 b2[8];
#pragma unroll 1
        for (int g = 0; g < ng; g += 3) {
            load(b2, g + 2, lane);
            __builtin_amdgcn_sched_barrier(0);  // keep the prefetch ahead of the use
            f(b[0], wbase + key(g));
            load(b[0], g + 3, lane);
            __builtin_amdgcn_sched_barrier(0);
            if (g + 1 < ng) f(b[1], wbase + key(g + 1));
            load(b[1], g + 4, lane);
            __builtin_amdgcn_sched_barrier(0);
            if (g + 2 < ng) f(b2, wbase + key(g + 2));
        }
    }
};

// A batch from the load layout into the wave's stage (a wave's own LDS
// accesses are ordered).
template <bool BF, int D>
__device__ __forceinline__ void to_stage(const u32x4 (&ld)[8], u32x4 *wst, int lane)
{
    using G = Geo<BF, D>;
    asm volatile("" ::: "memory");  // the window operands are read from LDS in every batch, not held
#pragma unroll
    for (int i = 0; i < 8; ++i) wst[G::pos(i * (64 / G::CR) + lane / G::CR, lane % G::CR)] = ld[i];
}

// Tile nt of the staged batch in the operand layout.
template <bool BF, int D>
__device__ __forceinline__ void tile_operand(const u32x4 *wst, int nt, int lane, u32x4 (&kx)[Geo<BF, D>::NCH])
{
    using G = Geo<BF, D>;
#pragma unroll
    for (int st = 0; st < G::NCH; ++st) kx[st] = wst[G::pos(16 * nt + (lane & 15), 4 * st + (lane >> 4))];
}

// v_sqrt_f32 errs by up to 0.9 of a last place and by 0.16 downwards on
// average, v_rsq_f32 by 0.1: the same way for all keys of about the same
// length, so that sums over keys keep it.  A Newton step each leaves a rounding
// of either sign (4096 lengths: d_E within 0.5 of a last place; 1 / |k| off by
// 0.005 x 2^-24 on average instead of 0.10) for 1 % of a call of 64-wide keys
// (12 layers of 4 heads x 16384: 64.9 -> 65.5 us).  128-wide bf16 keys keep the
// plain instructions, as in the streaming kernels.
template <bool BF, int D>
constexpr bool kRefine = !(BF && D == 128);

// 1 / sqrt(x), 1e-37 <= x < infinity.
__device__ __forceinline__ float rsq_refined(float x)
{
    const float r = __builtin_amdgcn_rsqf(x);
    return fmaf(0.5f * r, fmaf(-(x * r), r, 1.f), r);
}
// sqrt(x) from r = 1 / sqrt(x).
__device__ __forceinline__ float sqrt_refined(float x, float r)
{
    const float s = x * r;
    return fmaf(0.5f * r, fmaf(-s, s, x), s);
}

// Sums over the four 16-lane groups of four values at once: group 0 gets the
// total of a over the lanes of its column, group 1 of b, group 2 of c and
// group 3 of d.  Each swap gives both halves of two values to one addition:
// three swaps and three additions instead of eight lane moves and eight.
__device__ __forceinline__ float groups_sum4(float a, float b, float c, float d)
{
    return fold16(fold32(a, c), fold32(b, d));
}

// 2^x down to the least subnormal; v_exp_f32 gives zero below kExpLeast.
constexpr float kExpLeast = -126.f;
__device__ __forceinline__ float exp2_subnormal(float x)
{
    const bool low = x < kExpLeast;  // (x + 64 is exact there)
    return fast::fast_exp2(low ? x + 64.f : x) * (low ? 0x1p-64f : 1.f);
}

__device__ __forceinline__ float groups_sum(float x)
{
    return across32(across16(x, OpAdd{}), OpAdd{});
}

// Sweep 1, per block of a.rpb1 keys: column sums of k and k / |k|, and per
// window row the softmax reference and sum over the block's keys.  The keys
// are the A operand, so a lane holds one window row of each 16-row tile
// against four keys per 16-key tile and keeps that row's running reference
// and sum on its own (the reference moves only when a batch exceeds it by
// more than 2^16).
template <bool BF, int D, int MT>
__global__ __launch_bounds__(kThreads, 2) void k_rows1(ScoreArgs a)
{
    using G = Geo<BF, D>;
    __shared__ u32x4 stage[kWaves][kBatchBytes / 16];
    __shared__ u32x4 qs[MT * G::NCH * 64];
    __shared__ __attribute__((aligned(16))) float wcs[kWaves][2][D];
    __shared__ float wm[kWaves][16 * MT], wsm[kWaves][16 * MT];

    const SweepBlock sb = sweep_block(a);
    const int u = sb.u;
    const Unit un = sb.un;
    const int T = un.T;
    const int P = T - a.w;
    const int row_base = sb.x * a.rpb1;
    const int lane = threadIdx.x & 63, wv = uniform_i32(threadIdx.x >> 6);
    const float sc = a.inv_sqrt_d * kLog2e;
    const Stream<BF, D> in(a, un, row_base, a.rpb1, T, wv);
    Queries<BF, D, MT> wq;
    wq.load(a, un);
    __builtin_amdgcn_sched_barrier(0);
    u32x4 pf[2][8];
    in.prefetch(pf, lane);
    wq.put(a, qs);
    int lim[MT];  // last key visible to window row 16 mt + lane % 16
    float ms[MT], ss[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        lim[mt] = a.causal ? P + (16 * mt + (lane & 15)) % a.w : T - 1;
        ms[mt] = -INFINITY;
        ss[mt] = 0.f;
    }
    float sk[G::DL], sh[G::DL];
#pragma unroll
    for (int d = 0; d < G::DL; ++d) sk[d] = sh[d] = 0.f;
    u32x4 *wst = stage[wv];
    lds_barrier();

    in.run(pf, lane, [&](const u32x4 (&ld)[8], int key0) {
        to_stage<BF, D>(ld, wst, lane);
        const bool inside = key0 + G::BK <= P;  // every key visible to every row
#pragma unroll
        for (int t0 = 0; t0 < G::NT; t0 += G::HT) {
            u32x4 kx[G::HT][G::NCH];
#pragma unroll
            for (int nt = 0; nt < G::HT; ++nt) tile_operand<BF, D>(wst, t0 + nt, lane, kx[nt]);
            f32x4v acc[MT][G::HT];
            logits<BF, D, MT, true>(kx, qs, lane, acc);
            if (!inside) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < G::HT; ++nt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int gk = key0 + 16 * (t0 + nt) + 4 * (lane >> 4) + r;
                            acc[mt][nt][r] = gk < T && gk <= lim[mt] ? acc[mt][nt][r] : -INFINITY;
                        }
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                float x[G::HT][4], mx = -INFINITY;
#pragma unroll
                for (int nt = 0; nt < G::HT; ++nt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        x[nt][r] = acc[mt][nt][r] * sc;
                        mx = fmaxf(mx, x[nt][r]);
                    }
                const bool move = mx > ms[mt] + kRebase || (ms[mt] == -INFINITY && mx != -INFINITY);
                const float nm = move ? mx : ms[mt];
                if (nm != -INFINITY) {
                    float add = 0.f;
#pragma unroll
                    for (int nt = 0; nt < G::HT; ++nt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) add += fast::fast_exp2(x[nt][r] - nm);
                    ss[mt] = (move ? ss[mt] * fast::fast_exp2(ms[mt] - nm) : ss[mt]) + add;
                    ms[mt] = nm;
                }
            }
        }
        // column sums (zero rows past the range add nothing), from the stage again:
        // held through the softmax the batch would cost 32 registers
        asm volatile("" ::: "memory");
#pragma unroll
        for (int nt = 0; nt < G::NT; ++nt) {
            u32x4 q[G::NCH];
            float n2 = 0.f;
            tile_operand<BF, D>(wst, nt, lane, q);
#pragma unroll
            for (int st = 0; st < G::NCH; ++st) n2 = sq_chunk<BF>(q[st], n2);
            const float len2 = groups_sum(n2);
            const float inv = kRefine<BF, D> ? rsq_refined(__builtin_amdgcn_fmed3f(len2, 1e-24f, 3e38f))
                                             : __builtin_amdgcn_rsqf(fmaxf(len2, 1e-24f));
#pragma unroll
            for (int st = 0; st < G::NCH; ++st) {
                float v[G::EL];
                unpack_chunk<BF>(q[st], v);
#pragma unroll
                for (int e = 0; e < G::EL; ++e) {
                    sk[st * G::EL + e] += v[e];
                    sh[st * G::EL + e] = fmaf(v[e], inv, sh[st * G::EL + e]);
                }
            }
            // tile by tile: without the pins the compiler sinks the sums past the
            // next batches and spills the chunks it keeps for them
#pragma unroll
            for (int d = 0; d < G::DL; ++d) asm volatile("" : "+v"(sk[d]), "+v"(sh[d]));
        }
    });

    // merge: the four lane groups of a row, then the four waves (fixed order)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int msk = 16; msk < kWave; msk <<= 1) {
            const float m2 = __shfl_xor(ms[mt], msk, kWave), s2 = __shfl_xor(ss[mt], msk, kWave);
            softmax_merge2(ms[mt], ss[mt], m2, s2);
        }
        if (lane < 16) {
            wm[wv][16 * mt + lane] = ms[mt];
            wsm[wv][16 * mt + lane] = ss[mt];
        }
    }
#pragma unroll
    for (int d = 0; d < G::DL; ++d) {
        sk[d] = seg16_sum(sk[d]);
        sh[d] = seg16_sum(sh[d]);
    }
    if ((lane & 15) == 0) {
#pragma unroll
        for (int st = 0; st < G::NCH; ++st)
#pragma unroll
            for (int e = 0; e < G::EL; ++e) {
                wcs[wv][0][(4 * st + (lane >> 4)) * G::EL + e] = sk[st * G::EL + e];
                wcs[wv][1][(4 * st + (lane >> 4)) * G::EL + e] = sh[st * G::EL + e];
            }
    }
    __syncthreads();
    const int tid = threadIdx.x;
    float *part = a.part1 + ((int64_t)u * a.nch1 + sb.x) * (2 * D + 2 * a.R);
    if (tid < 2 * D) {
        float s = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < kWaves; ++w2) s += wcs[w2][tid / D][tid % D];
        part[tid] = s;
    }
    if (tid < a.R) {
        float m = wm[0][tid], s = wsm[0][tid];
#pragma unroll
        for (int w2 = 1; w2 < kWaves; ++w2) softmax_merge2(m, s, wm[w2][tid], wsm[w2][tid]);
        part[2 * D + tid] = m;
        part[2 * D + a.R + tid] = s;
    }
}

// Sweep 2, per block of a.rpb2 keys: d_E = |k - kbar| (from the differences,
// in fp32), khat.mu and the window-mean attention of every key, and the
// block's sum, extrema and sum of squares of d_E.  The keys are the B operand
// here, so a lane holds four window rows of each 16-row tile against its own
// key: att += 2^(x - M_m) / S_m (folding log2(S_m) into the shift would round
// it to the shift's last place, about 1e-6 of a row's weights).  The per-key outputs are collected in LDS and written once at the
// end (stores between the key loads interleave with the read stream at a high
// price).
template <bool BF, int D, int MT>
__global__ __launch_bounds__(kThreads, 2) void k_rows2(ScoreArgs a)
{
    using G = Geo<BF, D>;
    __shared__ u32x4 stage[kWaves][kBatchBytes / 16];
    __shared__ u32x4 qs[MT * G::NCH * 64];
    __shared__ __attribute__((aligned(16))) float outs[3][G::kMaxKeys];
    __shared__ __attribute__((aligned(16))) float sanc[2 * D];  // kbar, mu
    __shared__ __attribute__((aligned(16))) float rows[2][16 * MT];
    __shared__ float wred[4][kWaves];

    const SweepBlock sb = sweep_block(a);
    const int u = sb.u;
    const Unit un = sb.un;
    const int T = un.T;
    const int P = T - a.w;
    const int row_base = sb.x * a.rpb2;
    const int tid = threadIdx.x, lane = tid & 63, g4 = lane >> 4, wv = uniform_i32(tid >> 6);
    const int64_t obase = unit_out_base(a, un);
    const float sc = a.inv_sqrt_d * kLog2e, inv_r = 1.f / (float)a.R;
    const Stream<BF, D> in(a, un, row_base, a.rpb2, T, wv);
    Queries<BF, D, MT> wq;
    wq.load(a, un);
    // thread c < D: components c of kbar and mu; thread D + m: window row m's reference and sum
    static_assert(D + 16 * MT <= kThreads, "a thread for every column pair");
    const int am = min(max(tid - D, 0), a.R - 1);
    const int ac0 = tid < D ? tid : 2 * D + am, ac1 = tid < D ? D + tid : 2 * D + a.R + am;
    const float ld0 = anchor_load(a, u, ac0), ld1 = anchor_load(a, u, ac1);
    __builtin_amdgcn_sched_barrier(0);
    u32x4 pf[2][8];
    in.prefetch(pf, lane);
    wq.put(a, qs);
    // reference and 1 / sum of each window row (zero past R), four rows per lane
    // group and tile; with four tiles read from LDS where they are used (in
    // registers they would spill)
    const float av0 = anchor_convert(a, un, T, ac0, ld0), av1 = anchor_convert(a, un, T, ac1, ld1);
    if (tid < D) {
        sanc[tid] = av0;
        sanc[D + tid] = av1;
    } else if (tid < D + 16 * MT) {
        rows[0][tid - D] = tid - D < a.R ? av0 : 0.f;
        rows[1][tid - D] = tid - D < a.R ? 1.f / av1 : 0.f;
    }
    float dsum = 0.f, dsq = 0.f, dmn = INFINITY, dmx = -INFINITY;
    u32x4 *wst = stage[wv];
    lds_barrier();

    // kbar and mu at the lane's dimensions
    float kb[G::DL], mu[G::DL];
#pragma unroll
    for (int st = 0; st < G::NCH; ++st)
#pragma unroll
        for (int e = 0; e < G::EL; ++e) {
            kb[st * G::EL + e] = sanc[(4 * st + g4) * G::EL + e];
            mu[st * G::EL + e] = sanc[D + (4 * st + g4) * G::EL + e];
        }
    f32x4v rm[MT], rs[MT];
    auto load_rows = [&] {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            rm[mt] = *reinterpret_cast<const f32x4v *>(&rows[0][16 * mt + 4 * g4]);
            rs[mt] = *reinterpret_cast<const f32x4v *>(&rows[1][16 * mt + 4 * g4]);
        }
    };
    if constexpr (MT < 4) load_rows();
    in.run(pf, lane, [&](const u32x4 (&ld)[8], int key0) {
        to_stage<BF, D>(ld, wst, lane);
        u32x4 kx[G::HT][G::NCH];
        f32x4v acc[MT][G::HT];
#pragma unroll
        for (int t = 0; t < G::NT; ++t) {
            const int nt = t % G::HT;
            if (nt == 0) {
#pragma unroll
                for (int n = 0; n < G::HT; ++n) tile_operand<BF, D>(wst, t + n, lane, kx[n]);
                logits<BF, D, MT, false>(kx, qs, lane, acc);
            }
            __builtin_amdgcn_sched_barrier(0);  // tile by tile (register pressure)
            // four partial sums of each, so that no chain is longer than DL / 4
            float n2p[4] = {0.f, 0.f, 0.f, 0.f}, kmp[4] = {0.f, 0.f, 0.f, 0.f}, d2p[4] = {0.f, 0.f, 0.f, 0.f}, att = 0.f;
#pragma unroll
            for (int st = 0; st < G::NCH; ++st) {
                float v[G::EL];
                unpack_chunk<BF>(kx[nt][st], v);
                if constexpr (BF) n2p[st % 4] = sq_chunk<BF>(kx[nt][st], n2p[st % 4]);
#pragma unroll
                for (int e = 0; e < G::EL; ++e) {
                    const int d = st * G::EL + e;
                    const float x = v[e] - kb[d];
                    d2p[e % 4] = fmaf(x, x, d2p[e % 4]);
                    kmp[e % 4] = fmaf(v[e], mu[d], kmp[e % 4]);
                    if constexpr (!BF) n2p[e % 4] = fmaf(v[e], v[e], n2p[e % 4]);
                }
            }
            if constexpr (MT == 4) load_rows();
            // Keys whose attention falls below the least normal float still rank by
            // it: rare enough that a wave does them over.  (Not with 128-wide bf16
            // keys: the streaming kernels of that shape have zero there, and with four
            // tiles it would spill 31 registers.)
            constexpr bool kSubnormal = !(BF && D == 128);
            float least = 0.f;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = fmaf(acc[mt][nt][r], sc, -rm[mt][r]);
                    least = fminf(least, x);
                    att = fmaf(fast::fast_exp2(x), rs[mt][r], att);
                }
            if (kSubnormal && __builtin_amdgcn_ballot_w64(least < kExpLeast)) {
                att = 0.f;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        att = fmaf(exp2_subnormal(fmaf(acc[mt][nt][r], sc, -rm[mt][r])), rs[mt][r], att);
            }
            // totals over the four lane groups, one per group: |k - kbar|^2, k.mu,
            // |k|^2 and the attention of key lane % 16
            const float t4 = groups_sum4((d2p[0] + d2p[1]) + (d2p[2] + d2p[3]), (kmp[0] + kmp[1]) + (kmp[2] + kmp[3]),
                                         (n2p[0] + n2p[1]) + (n2p[2] + n2p[3]), att);
            float root, len;  // group 0: d_E; group 2: 1 / |k| (bf16), |k|
            if constexpr (!BF) {
                root = sqrtf(t4);
                len = fmaxf(root, 1e-12f);
            } else if constexpr (kRefine<BF, D>) {
                const float r = rsq_refined(__builtin_amdgcn_fmed3f(t4, 1e-37f, 3e38f));
                root = sqrt_refined(t4, r);
                len = fminf(r, 1e12f);
            } else {
                root = __builtin_amdgcn_sqrtf(t4);
                len = __builtin_amdgcn_rsqf(fmaxf(t4, 1e-24f));
            }
            const float klen = __shfl(len, 32 + (lane & 15), kWave);
            const float val = g4 == 0 ? root : g4 == 1 ? (BF ? t4 * klen : t4 / klen) : t4 * inv_r;
            const int gi = key0 + 16 * t + (lane & 15);
            if (gi < T) {
                if (g4 != 2) outs[g4 < 2 ? g4 : 2][gi - row_base] = val;
                if (g4 == 0) {
                    dsum += val;
                    dsq += val * val;
                    if (gi < P) {
                        dmn = fminf(dmn, val);
                        dmx = fmaxf(dmx, val);
                    }
                }
            }
        }
    });

    dsum = wave_sum(dsum);
    dsq = wave_sum(dsq);
    dmn = wave_min(dmn);
    dmx = wave_max(dmx);
    if (lane == 0) {
        wred[0][wv] = dsum;
        wred[1][wv] = dmn;
        wred[2][wv] = dmx;
        wred[3][wv] = dsq;
    }
    __syncthreads();
    {
        // keys row_base .. of the unit's P non-window keys (the descriptors end at P); written through
        float *const dst[3] = {a.bufA + obase, a.bufB + obase, a.bufC + obase};
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(dst[t], (short)0, P * 4, 0x00020000);
            for (int i = 4 * tid; i < a.rpb2; i += 4 * kThreads) {
                const f32x4v v = *reinterpret_cast<const f32x4v *>(&outs[t][i]);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), ro, (row_base + i) * 4, 0, 16);
            }
        }
    }
    if (tid == 0) {
        float s = 0.f, s2 = 0.f, mn = INFINITY, mx = -INFINITY;
        for (int k = 0; k < kWaves; ++k) {
            s += wred[0][k];
            mn = fminf(mn, wred[1][k]);
            mx = fmaxf(mx, wred[2][k]);
            s2 += wred[3][k];
        }
        float *pp = a.part2 + ((int64_t)u * a.nch2 + sb.x) * 4;
        pp[0] = s;
        pp[1] = mn;
        pp[2] = mx;
        pp[3] = s2;
    }
    bump_call_tag(a);
}

template <bool BF, int D, int MT>
static void launch(int pass, const ScoreArgs &a, dim3 grid, hipStream_t st)
{
    if (pass == 1) hipLaunchKernelGGL((k_rows1<BF, D, MT>), grid, dim3(kThreads), 0, st, a);
    else hipLaunchKernelGGL((k_rows2<BF, D, MT>), grid, dim3(kThreads), 0, st, a);
}

template <bool BF, int D>
static void launch_mt(int pass, const ScoreArgs &a, dim3 grid, hipStream_t st)
{
    if (a.R <= 16) launch<BF, D, 1>(pass, a, grid, st);
    else if (a.R <= 32) launch<BF, D, 2>(pass, a, grid, st);
    else launch<BF, D, 4>(pass, a, grid, st);
}

}  // namespace rows

int sweep_rows_max_keys(bool bf16) { return bf16 ? rows::Geo<true, 64>::kMaxKeys : rows::Geo<false, 64>::kMaxKeys; }

void sweep_rows_launch(int pass, const ScoreArgs &a, dim3 grid, hipStream_t st)
{
    if (!a.kbf16) {
        if (a.D == 128) rows::launch_mt<false, 128>(pass, a, grid, st);
        else rows::launch_mt<false, 64>(pass, a, grid, st);
    } else if (a.D == 64) {
        rows::launch_mt<true, 64>(pass, a, grid, st);
    } else {
        rows::launch_mt<true, 128>(pass, a, grid, st);
    }
}

}  // namespace ecokv
