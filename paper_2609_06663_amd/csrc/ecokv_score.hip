// ecokv_score kernels (gfx950): importance, diversity, redundancy and the
// final score of every (layer, KV head, sequence) unit.
//
// Stages, in stream order:
//   sweep1   one pass over K per block of rows: column sums of k and of k/|k|
//            (centroid kbar, Eq. (1); mean normalised key mu, Appendix A.1)
//            and, for every window row, the block's softmax maximum and sum of
//            exponentials of q.k/sqrt(d_k) (Sec. 3 attention, causal window).
//   reduce1  per unit: combine the block partials into kbar, mu and the
//            per-row softmax maximum and normaliser.
//   sweep2   second pass over K: per key d_E = |k - kbar| (Eq. (1)), khat.mu
//            and the window-mean attention a_i (Sec. 5.2: average attention
//            score over the window); block partials of sum/min/max d_E.
//   epilogue per unit: D_E (Eq. (4)), r_E (Eq. (5)), r_C (Appendix A.1),
//            lambda (Eq. (6)); pooled S_imp (Table 6), s_E (Eq. (2)), s_C,
//            S_div (Eq. (3)); the rescale of Sec. 5.2 and S (Eq. (7)).
//
// The sweeps of bf16 keys with head_dim 128 whose window rows fit one 32-row
// operand are here: each wave streams its own keys, v_mfma_f32_32x32x16_bf16
// with 32 window rows against 32 keys.  Those of every other shape are in
// ecokv_sweep.hip.
#include <stdlib.h>
#include <string.h>

#include "ecokv_fast.h"

namespace ecokv {

// ---------------------------------------------------------------------------
// bf16, head_dim 128, one 32-row window operand.
// ---------------------------------------------------------------------------
namespace fast {

// Window row lane & 31 as an MFMA operand (zero beyond R): for k-step s the
// lane holds elements 8*(2s + lane/32) .. +7.  The loads alone, and the rows
// beyond R cleared where they are first used, so that other loads go out
// between the two.
__device__ __forceinline__ void load_query_rows(const ScoreArgs &a, const Unit &un, int lane, u32x4 (&q)[8])
{
    const int r = lane & 31;
    const uint16_t *qp = static_cast<const uint16_t *>(a.Q) + window_row(a, un, r < a.R ? r : 0) * kD;
#pragma unroll
    for (int s = 0; s < 8; ++s) q[s] = *reinterpret_cast<const u32x4 *>(qp + 8 * (2 * s + (lane >> 5)));
}
__device__ __forceinline__ void query_operands(const ScoreArgs &a, int lane, const u32x4 (&q)[8], bf16x8 (&aq)[1][8])
{
    const bool ok = (lane & 31) < a.R;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        aq[0][s] = __builtin_bit_cast(bf16x8, ok ? q[s] : z);
    }
}

// Sweep 2, streaming form (window rows + 2 rows of mu in one 32-row operand,
// i.e. G*w <= 30): no LDS tile and no barrier in the key loop.  Each wave
// streams a quarter of the block's keys in groups of 32 from HBM into
// registers (three groups in flight, the first three right behind the loads of
// the window rows and anchors), re-lays them out through a
// wave-private LDS stage into MFMA B operands (lane l: key l % 32, 16-byte
// chunks 2s + l / 32).  The attention of row m is 2^(x - M'_m) with
// M'_m = M_m + log2(S_m), the normaliser folded into the shift.  Bound by the
// key stream and, within a few per cent of it, by the per-key arithmetic at
// two waves per SIMD.
constexpr int kS2Waves = 4;
constexpr int kS2KeysMin = 512;     // keys per block at least (one layer of 4 x 32768: 256 is no faster in either
                                    // sweep and doubles the partials, reduce1 4.8 -> 6.4 us)
constexpr int kS2KeysMax = 2048;    // and at most
constexpr int kS2KeysCache = 512;   // of the sweep that writes the cache

// Coalesced load of 32 key rows: instruction i covers rows 4i .. 4i+3, lane l
// chunk l % 16 of row 4i + l / 16 (four whole 256-byte rows per instruction).
// Nontemporal (cache policy nt): K streams through once per sweep, and keeping
// it out of the caches makes both sweeps 15-20 us faster.
__device__ __forceinline__ void group_load(u32x4 (&b)[8], __amdgpu_buffer_rsrc_t rs, int key0, int lane)
{
#pragma unroll
    for (int i = 0; i < 8; ++i)
        b[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (key0 + 4 * i + (lane >> 4)) * (kD * 2) + (lane & 15) * 16, 0, 2);
}

__global__ __launch_bounds__(256, 2) void k_fs2s(ScoreArgs a)
{
    const int wave_keys = a.rpb2 / kS2Waves;  // a multiple of 32
    __shared__ float wred[4][kS2Waves];
    __shared__ u32x4 stage[kS2Waves][32 * kChunks];  // per wave: 32 rows, swizzled 16-byte chunks
    __shared__ float wd2[kS2Waves][32];               // per wave: |k - kbar|^2 of its 32 rows
    // the block's per-key outputs (d_E, khat.mu, a), written out once at the end:
    // a few long stores instead of three 128-byte stores per 32 keys, which
    // interleave with the read stream at a high price
    __shared__ __attribute__((aligned(16))) float outs[3][kS2KeysMax];
    const SweepBlock sb = sweep_block(a);
    const int u = sb.u;
    const Unit un = sb.un;
    const int T = un.T;
    const int P = T - a.w;
    const int row_base = sb.x * a.rpb2;
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, kl = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint16_t *krow0 = static_cast<const uint16_t *>(a.K) + unit_row0(a, un) * kD;
    const int64_t obase = unit_out_base(a, un);
    // this wave's keys [wbase, wbase + wave_keys) only: loads past them read zero, no traffic
    const int wbase = row_base + wv * wave_keys;
    const int wkeys = __builtin_amdgcn_readfirstlane(max(0, min(wave_keys, T - wbase)));
    const __amdgpu_buffer_rsrc_t rs = key_rows_rsrc(krow0 + (int64_t)wbase * kD, wkeys);
    // Four register buffers in a ring: three groups (24 KiB per wave) stay in
    // flight while one is used.  Every load is unconditional (the descriptor
    // zero-fills past the wave's keys), so the outstanding-load count is the
    // same on every path and each wait covers only the group about to be used.
    const int ng = (wkeys + 31) >> 5;
    // Waves start at different groups of their range (rotation rot), so that
    // at any moment they read different offsets rather than the same offset
    // of equally sized, equally aligned ranges (which would crowd the same
    // memory channels).  Slot g >= ng reads past the range: zeros, skipped.
    const int rot = ng > 0 ? uniform_i32((int)(((unsigned)(sb.x * kS2Waves + wv) * 2654435761u + u * 40503u) % (unsigned)ng)) : 0;
    auto goff = [&](int g) { return g < ng ? 32 * (g + rot < ng ? g + rot : g + rot - ng) : 32 * ng; };
    // The set-up's loads go out first and the first three groups behind them:
    // loads return in order, so the set-up works while the groups are in flight
    // (the other way round, and each wave converting the anchors by itself, the
    // score of one 32768-token layer took 38.3 us instead of 34.5).
    u32x4 q[8];
    load_query_rows(a, un, lane, q);
    // thread c < D: components c of kbar and mu; thread D + m: window row m's reference and sum
    const int am = min(max(tid - kD, 0), a.R - 1);
    const int ac0 = tid < kD ? tid : 2 * kD + am, ac1 = tid < kD ? kD + tid : 2 * kD + a.R + am;
    const float ld0 = anchor_load(a, u, ac0), ld1 = anchor_load(a, u, ac1);
    __builtin_amdgcn_sched_barrier(0);
    u32x4 b0[8], b1[8], b2[8], b3[8];
    group_load(b0, rs, goff(0), lane);
    group_load(b1, rs, goff(1), lane);
    group_load(b2, rs, goff(2), lane);
    __builtin_amdgcn_sched_barrier(0);
    // The anchors through LDS, each converted once in the block: kbar, mu as two
    // bf16 rows (high part and remainder), and the row shifts M'_m.
    __shared__ __attribute__((aligned(16))) float kbs[kD];
    __shared__ __attribute__((aligned(16))) uint16_t mus[2][kD];
    __shared__ __attribute__((aligned(16))) float shs[32];
    const float av0 = anchor_convert(a, un, T, ac0, ld0), av1 = anchor_convert(a, un, T, ac1, ld1);
    if (tid < kD) {
        kbs[tid] = av0;
        const unsigned hi = bf16_rne(av1);
        mus[0][tid] = (uint16_t)hi;
        mus[1][tid] = (uint16_t)bf16_rne(av1 - __uint_as_float(hi << 16));
    } else if (tid < kD + 32) {
        shs[tid - kD] = tid - kD < a.R ? av0 + __log2f(av1) : INFINITY;
    }
    const float sc = a.inv_sqrt_d * kLog2e;
    constexpr int kAnc = 32 - 2;

    // A operand: window rows (zero beyond R), rows 30, 31 mu high / remainder
    bf16x8 aq[1][8];
    query_operands(a, lane, q, aq);
    lds_barrier();
    if (kl >= kAnc) {
#pragma unroll
        for (int s = 0; s < 8; ++s)
            aq[0][s] = *reinterpret_cast<const bf16x8 *>(&mus[kl - kAnc][8 * (2 * s + h)]);
    }
    // kbar at the 8 dimensions of chunk lane % 16, the chunk this lane loads
    float kbc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) kbc[e] = kbs[8 * (lane & 15) + e];
    // per-lane row shifts M'_m for the rows m = 8(r/4) + 4h + r%4 of accumulator r
    float rsh[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) rsh[r] = shs[8 * (r >> 2) + 4 * h + (r & 3)];

    float dsum = 0.f, dsq = 0.f, dmn = INFINITY, dmx = -INFINITY;
    const float inv_r = 1.f / (float)a.R;

    u32x4 *wst = stage[wv];
    float *wd = wd2[wv];
    auto group = [&](const u32x4 (&ld)[8], int key0) {
        // |k - kbar|^2 in the load layout (lane l: chunk l % 16 of rows 4i + l / 16):
        // the differences in fp32, summed over the lane's 8 dimensions, then
        // over the 16 lanes of a row by DPP; one lane per row parks the sum
        {
            float dp[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float s0 = 0.f, s1 = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float d0 = __uint_as_float(ld[i][e] << 16) - kbc[2 * e];
                    const float d1 = __uint_as_float(ld[i][e] & 0xffff0000u) - kbc[2 * e + 1];
                    s0 = fmaf(d0, d0, s0);
                    s1 = fmaf(d1, d1, s1);
                }
                dp[i] = row_sum<16>(s0 + s1);
            }
            if ((lane & 15) == 0) {
#pragma unroll
                for (int i = 0; i < 8; ++i) wd[4 * i + (lane >> 4)] = dp[i];
            }
        }
        // through this wave's LDS stage into the B-operand layout (lane l: key
        // l % 32, chunks 2s + l / 32); a wave's own LDS accesses are ordered
#pragma unroll
        for (int i = 0; i < 8; ++i) wst[sw(4 * i + (lane >> 4), lane & 15)] = ld[i];
        u32x4 b[8];
#pragma unroll
        for (int st = 0; st < 8; ++st) b[st] = wst[sw(kl, 2 * st + h)];
        f32x16 acc = (f32x16){};
        float n2 = 0.f;
#pragma unroll
        for (int st = 0; st < 8; ++st) {
            n2 = dot2sq(b[st][0], dot2sq(b[st][1], dot2sq(b[st][2], dot2sq(b[st][3], n2))));
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq[0][st], __builtin_bit_cast(bf16x8, b[st]), acc, 0, 0, 0);
        }
        float att = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) att += fast_exp2(fmaf(acc[r], sc, -rsh[r]));
        float kmu = h ? acc[14] + acc[15] : 0.f;
        n2 = across32(n2, OpAdd{});
        att = across32(att, OpAdd{});
        kmu = across32(kmu, OpAdd{});
        const float dE = __builtin_amdgcn_sqrtf(wd[kl]);
        const float cm = kmu * __builtin_amdgcn_rsqf(fmaxf(n2, 1e-24f));
        const int gi = key0 + kl;
        if (h == 0) {
            if (gi < T) {
                dsum += dE;
                dsq += dE * dE;
            }
            if (gi < P) {
                dmn = fminf(dmn, dE);
                dmx = fmaxf(dmx, dE);
            }
            outs[0][gi - row_base] = dE;
            outs[1][gi - row_base] = cm;
            outs[2][gi - row_base] = att * inv_r;
        }
    };

#pragma unroll 1
    for (int g = 0; g < ng; g += 4) {
        group_load(b3, rs, goff(g + 3), lane);
        __builtin_amdgcn_sched_barrier(0);  // keep the prefetch ahead of the use
        group(b0, wbase + goff(g));
        if (g + 1 >= ng) break;
        group_load(b0, rs, goff(g + 4), lane);
        __builtin_amdgcn_sched_barrier(0);
        group(b1, wbase + goff(g + 1));
        if (g + 2 >= ng) break;
        group_load(b1, rs, goff(g + 5), lane);
        __builtin_amdgcn_sched_barrier(0);
        group(b2, wbase + goff(g + 2));
        if (g + 3 >= ng) break;
        group_load(b2, rs, goff(g + 6), lane);
        __builtin_amdgcn_sched_barrier(0);
        group(b3, wbase + goff(g + 3));
    }

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
        // keys row_base .. of the unit's P non-window keys; the descriptors end at P
        float *const dst[3] = {a.bufA + obase, a.bufB + obase, a.bufC + obase};
        typedef float f32x4v __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const __amdgpu_buffer_rsrc_t ro =
                __builtin_amdgcn_make_buffer_rsrc(dst[t], (short)0, P * 4, 0x00020000);
            // cache policy sc1 (system scope): the outputs are written through
            // instead of lingering dirty in the caches while K streams in
            // (28-layer stack, sweep 2: default policy 173 us, nt 170, sc1 163;
            // sc0 175, nt + sc1 172)
            for (int i = 4 * tid; i < a.rpb2; i += 4 * 256) {
                const f32x4v v = *reinterpret_cast<const f32x4v *>(&outs[t][i]);
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), ro, (row_base + i) * 4, 0, 16);
            }
        }
    }
    if (tid == 0) {
        float s = 0.f, s2 = 0.f, mn = INFINITY, mx = -INFINITY;
        for (int k = 0; k < kS2Waves; ++k) {
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

// Sweep 1, streaming form (bf16, head_dim 128, G*w <= 32): like the streaming
// sweep 2, each wave streams its own keys in 32-key groups (coalesced
// loads, three register buffers in flight, a wave-private LDS stage) and no
// barrier is needed until the final merge of the four waves.
//  * window logits: v_mfma_f32_32x32x16_bf16 with the keys as the A operand and
//    the window rows as B, so each lane holds one window row against 16 keys
//    and keeps that row's running softmax maximum and sum on its own (the
//    reference moves only when a group exceeds it by more than 2^16);
//  * column sums of k and of k/|k|: v_mfma_f32_16x16x32_bf16 per 16-dimension
//    block with rows (1, 1/|k| high, remainder, 0...) over the wave's 32 keys
//    as A, and the keys transposed out of the stage with ds_read_b64_tr_b16
//    as B.
// With CACHE (the KV-cache write of ecokv_prefill_write), each key row is read
// from the token-major new rows a.Ksrc and the loaded registers are written to
// the head-major cache a.K on arrival, before the group is used: one read and
// one write of K, and the sweep rides on them.
constexpr float kRebase1 = 16.f;  // log2 headroom of the lazily moved row reference
template <bool CACHE>
__global__ __launch_bounds__(256, 2) void k_fs1s(ScoreArgs a)
{
    const int wave_keys = a.rpb1 / kS2Waves;  // a multiple of 32
    __shared__ u32x4 stage[kS2Waves][32 * kChunks];
    __shared__ __attribute__((aligned(16))) uint16_t wts[kS2Waves][4][32];  // 1, 1/|k| hi, remainder, 0
    __shared__ float wcs[kS2Waves][2][kD];                                 // per-wave column sums
    __shared__ float wm[kS2Waves][32], wsm[kS2Waves][32];                  // per-wave row max / sum

    const SweepBlock sb = sweep_block(a);
    const int u = sb.u;
    const Unit un = sb.un;
    const int T = un.T;
    const int P = T - a.w;
    const int row_base = sb.x * a.rpb1;
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, kl = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint16_t *krow0 = static_cast<const uint16_t *>(a.K) + unit_row0(a, un) * kD;
    const float sc = a.inv_sqrt_d * kLog2e;
    const int lim = a.causal ? P + kl % a.w : T - 1;  // last key visible to window row kl

    const int wbase = row_base + wv * wave_keys;
    const int wkeys = __builtin_amdgcn_readfirstlane(max(0, min(wave_keys, T - wbase)));
    // CACHE: key i of the unit at row (l Ttot + cu[s] + i) Hkv + h of the new rows
    const int src_row_bytes = CACHE ? a.Hkv * kD * 2 : kD * 2;
    const __amdgpu_buffer_rsrc_t rs =
        CACHE ? __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<uint16_t *>(uniform_ptr(static_cast<const uint16_t *>(a.Ksrc) +
                                                       (((int64_t)un.l * a.Ttot + un.c0 + wbase) * a.Hkv +
                                                        un.h) * kD)),
                    (short)0, wkeys * src_row_bytes, 0x00020000)
              : key_rows_rsrc(krow0 + (int64_t)wbase * kD, wkeys);
    const __amdgpu_buffer_rsrc_t rdst = key_rows_rsrc(krow0 + (int64_t)wbase * kD, CACHE ? wkeys : 0);
    u32x4 *wst = stage[wv];
    const int ng = (wkeys + 31) >> 5;
    const int rot = ng > 0 ? uniform_i32((int)(((unsigned)(sb.x * kS2Waves + wv) * 2654435761u + u * 40503u) % (unsigned)ng)) : 0;
    auto goff = [&](int g) { return g < ng ? 32 * (g + rot < ng ? g + rot : g + rot - ng) : 32 * ng; };
    u32x4 q[8];
    load_query_rows(a, un, lane, q);
    __builtin_amdgcn_sched_barrier(0);  // (ahead of the groups, as in sweep 2)
    u32x4 b0[8], b1[8], b2[8];
    group_load_rows(b0, rs, goff(0), lane, src_row_bytes);
    group_load_rows(b1, rs, goff(1), lane, src_row_bytes);

    __builtin_amdgcn_sched_barrier(0);
    bf16x8 aq[1][8];
    query_operands(a, lane, q, aq);
    if (lane < 32) {
        wts[wv][0][lane] = 0x3f80;
        wts[wv][3][lane] = 0;
    }

    float ms = -INFINITY, ss = 0.f;  // window row kl over this lane's keys
    typedef float f32x4v __attribute__((ext_vector_type(4)));
    f32x4v cs[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) cs[b] = (f32x4v){0.f, 0.f, 0.f, 0.f};
    // transposed-read addressing: lane 16G + 4a + b reads key row 8G + a (+4),
    // dimensions 16 blk + 4b .. +3; the read returns dimension 16 blk + lane % 16
    // of keys 8G + 0..3 (then 4..7)
    const int tr_row = 8 * (lane >> 4) + ((lane & 15) >> 2), tr_b = lane & 3;
    const int w_row = (lane & 15) < 3 ? (lane & 15) : 3;

    auto group = [&](const u32x4 (&ld)[8], int key0) {
        if constexpr (CACHE) group_store(ld, rdst, key0 - wbase, lane);  // (rows past the wave's end are dropped)
#pragma unroll
        for (int i = 0; i < 8; ++i) wst[sw(4 * i + (lane >> 4), lane & 15)] = ld[i];
        u32x4 b[8];
#pragma unroll
        for (int st = 0; st < 8; ++st) b[st] = wst[sw(kl, 2 * st + h)];
        f32x16 acc = (f32x16){};
        float n2 = 0.f;
#pragma unroll
        for (int st = 0; st < 8; ++st) {
            n2 = dot2sq(b[st][0], dot2sq(b[st][1], dot2sq(b[st][2], dot2sq(b[st][3], n2))));
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b[st]), aq[0][st], acc, 0, 0, 0);
        }
        n2 = across32(n2, OpAdd{});
        const float inv = __builtin_amdgcn_rsqf(fmaxf(n2, 1e-24f));
        if (h == 0) {
            const unsigned hi = bf16_rne(inv);
            wts[wv][1][kl] = (uint16_t)hi;
            wts[wv][2][kl] = (uint16_t)bf16_rne(inv - __uint_as_float(hi << 16));
        }
        // softmax statistics of row kl over keys key0 + 8(r/4) + 4h + r%4
        {
            float x[16];
            float mx = -INFINITY;
            if (key0 + 32 <= P) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    x[r] = acc[r] * sc;
                    mx = fmaxf(mx, x[r]);
                }
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int gk = key0 + 8 * (r >> 2) + 4 * h + (r & 3);
                    x[r] = (gk < T && gk <= lim) ? acc[r] * sc : -INFINITY;
                    mx = fmaxf(mx, x[r]);
                }
            }
            const bool move = mx > ms + kRebase1 || (ms == -INFINITY && mx != -INFINITY);
            const float nm = move ? mx : ms;
            if (nm != -INFINITY) {
                float add = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) add += fast_exp2(x[r] - nm);
                ss = (move ? ss * fast_exp2(ms - nm) : ss) + add;
                ms = nm;
            }
        }
        // column sums over the wave's 32 keys (zero rows past T add nothing)
        const bf16x8 wa = *reinterpret_cast<const bf16x8 *>(&wts[wv][w_row][8 * (lane >> 4)]);
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        const uint16_t *st16 = reinterpret_cast<const uint16_t *>(wst);
#pragma unroll
        for (int blk = 0; blk < 8; ++blk) {
            const int c = 2 * blk + (tr_b >> 1), off = (tr_b & 1) * 4;
            const uint16_t *p0 = st16 + tr_row * kD + ((c ^ (tr_row & 15)) << 3) + off;
            const uint16_t *p1 = st16 + (tr_row + 4) * kD + ((c ^ ((tr_row + 4) & 15)) << 3) + off;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) s16x4 *)(const_cast<uint16_t *>(p0)));
            const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) s16x4 *)(const_cast<uint16_t *>(p1)));
            const short __attribute__((ext_vector_type(8))) kb8 = {lo[0], lo[1], lo[2], lo[3],
                                                                    hi4[0], hi4[1], hi4[2], hi4[3]};
            cs[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa, __builtin_bit_cast(bf16x8, kb8), cs[blk], 0, 0, 0);
        }
    };

#pragma unroll 1
    for (int g = 0; g < ng; g += 3) {
        group_load_rows(b2, rs, goff(g + 2), lane, src_row_bytes);
        __builtin_amdgcn_sched_barrier(0);  // keep the prefetch ahead of the use
        group(b0, wbase + goff(g));
        if (g + 1 >= ng) break;
        group_load_rows(b0, rs, goff(g + 3), lane, src_row_bytes);
        __builtin_amdgcn_sched_barrier(0);
        group(b1, wbase + goff(g + 1));
        if (g + 2 >= ng) break;
        group_load_rows(b1, rs, goff(g + 4), lane, src_row_bytes);
        __builtin_amdgcn_sched_barrier(0);
        group(b2, wbase + goff(g + 2));
    }

    // merge: halves of a row, then the four waves (fixed order)
    {
        const float m2 = __shfl_xor(ms, 32, kWave), s2 = __shfl_xor(ss, 32, kWave);
        softmax_merge2(ms, ss, m2, s2);
    }
    if (lane < 32) {
        wm[wv][lane] = ms;
        wsm[wv][lane] = ss;
    }
    if (lane < 16) {
#pragma unroll
        for (int blk = 0; blk < 8; ++blk) {
            wcs[wv][0][16 * blk + lane] = cs[blk][0];
            wcs[wv][1][16 * blk + lane] = cs[blk][1] + cs[blk][2];
        }
    }
    __syncthreads();
    const int stride = 2 * kD + 2 * a.R;
    float *part = a.part1 + ((int64_t)u * a.nch1 + sb.x) * stride;
    for (int i = tid; i < 2 * kD; i += blockDim.x) {
        const int which = i / kD, d = i % kD;
        float s = 0.f;
        for (int w2 = 0; w2 < kS2Waves; ++w2) s += wcs[w2][which][d];
        part[i] = s;
    }
    if (tid < a.R) {
        float m = wm[0][tid], s = wsm[0][tid];
        for (int w2 = 1; w2 < kS2Waves; ++w2) softmax_merge2(m, s, wm[w2][tid], wsm[w2][tid]);
        part[2 * kD + tid] = m;
        part[2 * kD + a.R + tid] = s;
    }
}

}  // namespace fast

// ---------------------------------------------------------------------------
// Per-unit reduction of the sweep-1 partials.
// ---------------------------------------------------------------------------
// Columns of a unit's partial rows: sum k (D), sum k/|k| (D), the R window
// rows' (max, normaliser) pairs.  `lanes` lanes per column, each over every
// lanes-th block partial with its loads in flight together, then combined by
// butterflies of commutative steps, so every lane ends with the same value.
// Up to 16 partials per unit: 4 lanes, one block per unit looping over the
// columns; more (64 for a 32 Ki-token unit in 512-key blocks): 16 lanes, grid
// (unit, column group of 64), so that no lane waits on a chain of loads
// (one layer: 9 -> 7 us; the 28-layer stack in 2048-key blocks is 0.7 us
// faster with one block per unit).
constexpr int kReduceThreads = 1024;
inline int reduce1_lanes(int nch1) { return nch1 > 16 ? 16 : 4; }

// op over an aligned group of 4 or 16 lanes (a quad, a DPP row), every lane
// getting the result.
template <int LANES, class Op>
__device__ __forceinline__ float lane_group_reduce(float x, Op op)
{
    static_assert(LANES == 4 || LANES == 16, "a quad or a 16-lane row");
    if constexpr (LANES == 16) return row_reduce<16>(x, op);
    x = op(x, dpp_row<0xB1>(x));  // quad_perm [1, 0, 3, 2]
    return op(x, dpp_row<0x4E>(x));  // quad_perm [2, 3, 0, 1]
}

// Columns cg, cg + ncg, ... (in groups of blockDim.x / LANES) of unit u's
// partials, LANES lanes per column; the calling block's threads all take part.
// With PRE (ecokv_prefill_write) the unit's sums are written to a.pre_out in
// the layout ecokv_score_pre takes: plain sums, and the window rows'
// references in natural units (of q.k / sqrt(D)).
template <int LANES, bool PRE>
__device__ __forceinline__ void reduce1_columns(const ScoreArgs &a, int u, int cg, int ncg)
{
    const Unit un = score_unit(a, u);
    const int T = un.T;
    const int nb = (T + a.rpb1 - 1) / a.rpb1;
    const int stride = 2 * a.D + 2 * a.R;
    const float *p = a.part1 + (int64_t)u * a.nch1 * stride;
    float *anc = (PRE ? a.pre_out : a.anchors) + (int64_t)u * stride;
    constexpr int lanes = LANES;
    const int cpb = blockDim.x / lanes;  // columns per block per step
    const int q = threadIdx.x & (lanes - 1);
    // (every lane of a column takes the same path: the butterflies stay within it)
    for (int c = cg * cpb + threadIdx.x / lanes; c < 2 * a.D + a.R; c += ncg * cpb) {
        if (c < 2 * a.D) {
            float s = 0.f;
#pragma unroll 4
            for (int b = q; b < nb; b += lanes) s += p[(int64_t)b * stride + c];
            s = lane_group_reduce<lanes>(s, OpAdd{});
            if (q == 0) anc[c] = PRE ? s : c < a.D ? centroid_component(a, un, T, c, s) : s / (float)T;
        } else {
            const int r = c - 2 * a.D;
            float m = -INFINITY, s = 0.f;
#pragma unroll 4
            for (int b = q; b < nb; b += lanes)
                softmax_merge2(m, s, p[(int64_t)b * stride + 2 * a.D + r], p[(int64_t)b * stride + 2 * a.D + a.R + r]);
            // the group's largest reference, each lane's sum moved onto it, summed
            const float mg = lane_group_reduce<lanes>(m, OpMax{});
            s = lane_group_reduce<lanes>(m == -INFINITY ? 0.f : s * __builtin_amdgcn_exp2f(m - mg), OpAdd{});
            m = mg;
            if (q == 0) {
                anc[2 * a.D + r] = PRE ? m * (1.f / kLog2e) : m;
                anc[2 * a.D + a.R + r] = s;
            }
        }
    }
}

template <int LANES, bool PRE>
__global__ __launch_bounds__(kReduceThreads) void k_reduce1(ScoreArgs a)
{
    reduce1_columns<LANES, PRE>(a, blockIdx.x, blockIdx.y, gridDim.y);
}

// ---------------------------------------------------------------------------
// Epilogue, two launches over (key blocks, units):
//   epi1: pooled S_imp and S_div of each non-window key; block sums/extrema.
//   epi2: every block derives the unit constants from the partials (same
//         order in every block) and writes S; block 0 writes the statistics.
// Each thread takes 16 consecutive keys with 16-byte buffer loads; the
// descriptors span exactly the unit's P non-window keys, so the pooling halo
// reads zero outside [0, P) (the zero padding of the average pool).
// ---------------------------------------------------------------------------
constexpr int kEpiThreads = 256;
constexpr int kEpiPer = 16;                      // consecutive keys per thread
constexpr int kEpiKeys = kEpiThreads * kEpiPer;  // keys per block
constexpr int kPoolHalfMax = 4;                  // vector pooling for kernels up to 9

struct Red4 {
    float s0, s1, mn, mx;
};

__device__ Red4 block_red4(Red4 v, Red4 *lds)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    v.s0 = wave_sum(v.s0);
    v.s1 = wave_sum(v.s1);
    v.mn = wave_min(v.mn);
    v.mx = wave_max(v.mx);
    if (lane == 0) lds[wv] = v;
    __syncthreads();
    Red4 r = lds[0];
    for (int k = 1; k < nw; ++k) {
        r.s0 += lds[k].s0;
        r.s1 += lds[k].s1;
        r.mn = fminf(r.mn, lds[k].mn);
        r.mx = fmaxf(r.mx, lds[k].mx);
    }
    __syncthreads();
    return r;
}

__device__ __forceinline__ float pooled(const float *abuf, int i, int P, int half)
{
    float acc = 0.f;
    for (int t = -half; t <= half; ++t) {
        const int k = i + t;
        if (k >= 0 && k < P) acc += abuf[k];
    }
    return acc * (1.f / (float)(2 * half + 1));
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t float_rsrc(const float *p, int n)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), (short)0, n * 4, 0x00020000);
}

// d_E and khat.mu of keys i0 .. i0+PER-1 (zero past P).
template <int PER>
__device__ __forceinline__ void load_dc(const float *dbuf, const float *cbuf, int P, int i0, float (&d)[PER],
                                        float (&c)[PER])
{
    const __amdgpu_buffer_rsrc_t rd = float_rsrc(dbuf, P), rc = float_rsrc(cbuf, P);
#pragma unroll
    for (int q = 0; q < PER / 4; ++q) {
        const f32x4 x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rd, (i0 + 4 * q) * 4, 0, 0));
        const f32x4 y = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rc, (i0 + 4 * q) * 4, 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            d[4 * q + e] = x[e];
            c[4 * q + e] = y[e];
        }
    }
}

// Pooled window attention S_imp of keys i0 .. i0+PER-1 (zero past P).
template <int PER>
__device__ __forceinline__ void load_imp(const ScoreArgs &a, const float *abuf, int P, int i0, float (&imp)[PER])
{
    const __amdgpu_buffer_rsrc_t ra = float_rsrc(abuf, P);
    const int half = a.pool_half;
    const float inv_k = 1.f / (float)(2 * half + 1);
    if (half <= kPoolHalfMax) {
        // av[j] = a[i0 - 4 + j]; a negative offset wraps past the range and reads zero
        float av[PER + 2 * kPoolHalfMax];
#pragma unroll
        for (int q = 0; q < (PER + 2 * kPoolHalfMax) / 4; ++q) {
            const f32x4 x = __builtin_bit_cast(
                f32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, (unsigned)(i0 - kPoolHalfMax + 4 * q) * 4u, 0, 0));
#pragma unroll
            for (int e = 0; e < 4; ++e) av[4 * q + e] = x[e];
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            float acc = 0.f;
#pragma unroll
            for (int t = -kPoolHalfMax; t <= kPoolHalfMax; ++t)
                if (t >= -half && t <= half) acc += av[j + kPoolHalfMax + t];
            imp[j] = acc * inv_k;
        }
    } else {
#pragma unroll
        for (int j = 0; j < PER; ++j) imp[j] = i0 + j < P ? pooled(abuf, i0 + j, P, half) : 0.f;
    }
}

// d_E, khat.mu and pooled window attention of keys i0 .. i0+15 (zero past P).
__device__ __forceinline__ void epi_keys(const ScoreArgs &a, const float *dbuf, const float *cbuf, const float *abuf,
                                         int P, int i0, float (&d)[kEpiPer], float (&c)[kEpiPer],
                                         float (&imp)[kEpiPer])
{
    load_dc<kEpiPer>(dbuf, cbuf, P, i0, d, c);
    load_imp<kEpiPer>(a, abuf, P, i0, imp);
}

// s_E of a distance (the Eq. (2) step): min-max over the unit's non-window
// keys; or, after clipping to the q and 1 - q quantiles, min-max between
// them (winsorised); or a sigmoid of the deviation from the median in units
// of the median absolute deviation (MAD) (Sec. 6.3, Table 4).  The quantile
// pair of a unit comes from k_dquant.
struct DNorm {
    float lo, hi, g;
    int sig;
};

__device__ __forceinline__ DNorm d_norm(const ScoreArgs &a, int u, const Red4 &dst)
{
    DNorm n;
    n.sig = 0;
    if (a.norm_mode == ECOKV_NORM_MINMAX) {
        n.lo = dst.mn;
        n.hi = dst.mx;
        n.g = 1.f / (dst.mx - dst.mn + a.eps);
    } else if (a.norm_mode == ECOKV_NORM_WINSOR) {
        n.lo = a.dq[2 * (int64_t)u];
        n.hi = a.dq[2 * (int64_t)u + 1];
        n.g = 1.f / (n.hi - n.lo + a.eps);
    } else {
        n.lo = a.dq[2 * (int64_t)u];
        n.hi = INFINITY;
        n.g = 1.f / (a.mad_tau * a.dq[2 * (int64_t)u + 1] + a.eps);
        n.sig = 1;
    }
    return n;
}

__device__ __forceinline__ float s_euclid(float d, const DNorm &n)
{
    if (n.sig) return 1.f / (1.f + expf(-(d - n.lo) * n.g));
    return (fminf(fmaxf(d, n.lo), n.hi) - n.lo) * n.g;
}

// The per-unit constants of Eq. (3)-(7) from the unit's reductions: d_E
// (sum and sum of squares over T, min / max over P), S_div (sum, min, max over
// P) and S_imp (sum over P), and |mu|^2.
struct EpiConsts {
    float lam, rE, rC, DE, smin, sden, impmean, sbarmean, scale;
};

__device__ __forceinline__ EpiConsts epi_consts(const ScoreArgs &a, const Red4 &dst, const Red4 &sd, float mu2, int T,
                                                int P)
{
    EpiConsts k;
    k.DE = dst.s0 / (float)T;
    if (a.red_std)  // r_std = 1 - sigmoid(D_std / tau), D_std = sqrt(mean_T d_E^2) (Appendix D)
        k.rE = 1.f - 1.f / (1.f + expf(-sqrtf(dst.s1 / (float)T) / a.tau));
    else
        k.rE = 2.f - 2.f / (1.f + expf(-k.DE / a.tau));
    k.rC = ((float)T * mu2 - 1.f) / ((float)T - 1.f);
    k.lam = a.use_override ? a.lambda_override : a.beta * k.rE + (1.f - a.beta) * k.rC;
    if (sd.s0 != sd.s0) k.lam = NAN;  // the split epilogue's wait gave up (or NaN inputs)
    k.smin = sd.mn;
    k.sden = sd.mx - sd.mn + a.eps;
    k.impmean = sd.s1 / (float)P;
    k.sbarmean = (sd.s0 / (float)P - k.smin) / k.sden;
    k.scale = k.impmean / (k.sbarmean + a.eps);
    return k;
}

__device__ __forceinline__ void epi_write_stats(const ScoreArgs &a, int u, const EpiConsts &k, const Red4 &dst,
                                                const Red4 &sd, float mu2)
{
    float st[ECOKV_NSTATS];
    st[ECOKV_STAT_LAMBDA] = k.lam;
    st[ECOKV_STAT_RC] = k.rC;
    st[ECOKV_STAT_RE] = k.rE;
    st[ECOKV_STAT_DE] = k.DE;
    st[ECOKV_STAT_DMIN] = dst.mn;
    st[ECOKV_STAT_DMAX] = dst.mx;
    st[ECOKV_STAT_SDIV_MIN] = sd.mn;
    st[ECOKV_STAT_SDIV_MAX] = sd.mx;
    st[ECOKV_STAT_IMP_MEAN] = k.impmean;
    st[ECOKV_STAT_SBAR_MEAN] = k.sbarmean;
    st[ECOKV_STAT_MU_NORM2] = mu2;
    st[ECOKV_STAT_SCALE] = k.scale;
    if (a.stats)
        for (int q = 0; q < ECOKV_NSTATS; ++q) a.stats[(int64_t)u * ECOKV_NSTATS + q] = st[q];
    if (a.lambda) a.lambda[u] = k.lam;
}

// Sum, sum of squares, min and max of d_E over the unit, from the sweep-2 partials.
__device__ Red4 unit_distance_stats(const ScoreArgs &a, int u, int T, Red4 *lds)
{
    const int nb = (T + a.rpb2 - 1) / a.rpb2;
    Red4 v{0.f, 0.f, INFINITY, -INFINITY};
    for (int b = threadIdx.x; b < nb; b += blockDim.x) {
        const float *pp = a.part2 + ((int64_t)u * a.nch2 + b) * 4;
        v.s0 += pp[0];
        v.s1 += pp[3];
        v.mn = fminf(v.mn, pp[1]);
        v.mx = fmaxf(v.mx, pp[2]);
    }
    return block_red4(v, lds);
}

__global__ __launch_bounds__(kEpiThreads) void k_epi1(ScoreArgs a)
{
    __shared__ Red4 lds[kEpiThreads / kWave];
    const int u = blockIdx.y;
    const Unit un = score_unit(a, u);
    const int T = un.T;
    const int P = T - a.w;
    const int i0 = blockIdx.x * kEpiKeys;
    if (i0 >= P) return;
    const int i1 = min(i0 + kEpiKeys, P);
    const int64_t ob = unit_out_base(a, un);
    const float *dbuf = a.bufA + ob, *cbuf = a.bufB + ob, *abuf = a.bufC + ob;
    const Red4 dst = unit_distance_stats(a, u, T, lds);
    const DNorm dn = d_norm(a, u, dst);

    Red4 w{0.f, 0.f, INFINITY, -INFINITY};
    {
        const int k0 = i0 + kEpiPer * threadIdx.x;
        float d[kEpiPer], c[kEpiPer], imp[kEpiPer];
        epi_keys(a, dbuf, cbuf, abuf, P, k0, d, c, imp);
#pragma unroll
        for (int j = 0; j < kEpiPer; ++j)
            if (k0 + j < i1) {
                const float sE = s_euclid(d[j], dn);
                const float sC = (1.f - c[j]) * 0.5f;
                const float sdiv = a.alpha * sE + (1.f - a.alpha) * sC;
                w.s0 += sdiv;
                w.s1 += imp[j];
                w.mn = fminf(w.mn, sdiv);
                w.mx = fmaxf(w.mx, sdiv);
            }
    }
    const Red4 r = block_red4(w, lds);
    if (threadIdx.x == 0) {
        float *pp = a.part3 + ((int64_t)u * a.nch3 + blockIdx.x) * 4;
        pp[0] = r.s0;
        pp[1] = r.s1;
        pp[2] = r.mn;
        pp[3] = r.mx;
    }
}

__global__ __launch_bounds__(kEpiThreads) void k_epi2(ScoreArgs a)
{
    __shared__ Red4 lds[kEpiThreads / kWave];
    const int u = blockIdx.y;
    const Unit un = score_unit(a, u);
    const int T = un.T;
    const int P = T - a.w;
    const int i0 = blockIdx.x * kEpiKeys;
    if (i0 >= P) return;
    const int i1 = min(i0 + kEpiKeys, P);
    const int64_t ob = unit_out_base(a, un);
    const float *dbuf = a.bufA + ob, *cbuf = a.bufB + ob, *abuf = a.bufC + ob;


    const Red4 dst = unit_distance_stats(a, u, T, lds);
    Red4 v{0.f, 0.f, INFINITY, -INFINITY};
    const int nb3 = (P + kEpiKeys - 1) / kEpiKeys;
    for (int b = threadIdx.x; b < nb3; b += blockDim.x) {
        const float *pp = a.part3 + ((int64_t)u * a.nch3 + b) * 4;
        v.s0 += pp[0];
        v.s1 += pp[1];
        v.mn = fminf(v.mn, pp[2]);
        v.mx = fmaxf(v.mx, pp[3]);
    }
    const Red4 sd = block_red4(v, lds);
    Red4 m2{0.f, 0.f, 0.f, 0.f};
    for (int d = threadIdx.x; d < a.D; d += blockDim.x) {
        const float mv = anchor_value(a, un, u, T, a.D + d);
        m2.s0 += mv * mv;
    }
    const float mu2 = block_red4(m2, lds).s0;
    const EpiConsts k = epi_consts(a, dst, sd, mu2, T, P);
    const float lam = k.lam, smin = k.smin, sden = k.sden, scale = k.scale;
    const DNorm dn = d_norm(a, u, dst);

    float *out = a.scores + ob;
    {
        const int k0 = i0 + kEpiPer * threadIdx.x;
        float d[kEpiPer], c[kEpiPer], imp[kEpiPer], sv[kEpiPer];
        epi_keys(a, dbuf, cbuf, abuf, P, k0, d, c, imp);
#pragma unroll
        for (int j = 0; j < kEpiPer; ++j) {
            const float sE = s_euclid(d[j], dn);
            const float sC = (1.f - c[j]) * 0.5f;
            const float sdiv = a.alpha * sE + (1.f - a.alpha) * sC;
            sv[j] = lam * (((sdiv - smin) / sden) * scale) + (1.f - lam) * imp[j];
        }
        if (k0 + kEpiPer <= i1) {
            const __amdgpu_buffer_rsrc_t ro = float_rsrc(out, P);
#pragma unroll
            for (int q = 0; q < kEpiPer / 4; ++q) {
                const f32x4 x = {sv[4 * q], sv[4 * q + 1], sv[4 * q + 2], sv[4 * q + 3]};
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), ro, (k0 + 4 * q) * 4, 0, 0);
            }
        } else {
#pragma unroll
            for (int j = 0; j < kEpiPer; ++j)
                if (k0 + j < i1) out[k0 + j] = sv[j];
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) epi_write_stats(a, u, k, dst, sd, mu2);
}

// Epilogue in one launch: each unit's P non-window keys in SPLIT blocks
// (1, 2, 4 or 8) of 4096 KVEC keys (KVEC 1, 2, 4 or 8; at most 65536 keys per
// unit), the host choosing the most blocks per unit that fill at most half
// the device (else two per unit if it holds them; one block of 32768 keys
// when the caller allows no waits).  Every per-unit reduction is
// block-local, except that with SPLIT > 1 the parts of a unit exchange their
// S_div / S_imp sums and extrema once (tagged 64-bit relaxed atomics; the
// parts are combined in a fixed order, so all compute the same constants).
// The wait for the other parts is bounded: if it gives up, the unit's lambda
// and scores come out NaN and the workspace status word records the call's
// tag.  Each key's d_E, khat.mu and attention is read once.  Wave w holds
// KVEC chunks of 256 consecutive keys; lane l of chunk j holds keys
// 256 j + 4 l .. +3 of the wave's range, so each load instruction covers
// 1 KiB of consecutive keys.
// The pooling window (up to 4 keys on each side) comes from the neighbouring
// lanes' registers (or the neighbouring chunk's end lane); the wave's
// outermost neighbours come from the neighbouring waves through LDS, and at
// the ends of a block's range from memory.
constexpr int kUThreads = 1024;
constexpr int kUW = kUThreads / kWave;
constexpr int kUKeys = kUThreads * 32;  // 32768 keys: one block of the one-launch epilogue at most
constexpr int kEpiSplitMax = 8;         // blocks per unit at most
constexpr int kEpiUnitMax = 2 * kUKeys; // keys per unit at most (65536)

// Block sum / min / max whose barriers order LDS only, so that global loads
// issued before it stay in flight.
__device__ Red4 block_red4_lds(Red4 v, Red4 *lds)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    v.s0 = wave_sum(v.s0);
    v.s1 = wave_sum(v.s1);
    v.mn = wave_min(v.mn);
    v.mx = wave_max(v.mx);
    if (lane == 0) lds[wv] = v;
    lds_barrier();
    Red4 r = lds[0];
    for (int k = 1; k < nw; ++k) {
        r.s0 += lds[k].s0;
        r.s1 += lds[k].s1;
        r.mn = fminf(r.mn, lds[k].mn);
        r.mx = fmaxf(r.mx, lds[k].mx);
    }
    lds_barrier();
    return r;
}

// Whole-wave shifts by one lane (DPP wave_shr:1 / wave_shl:1): lane l gets
// lane l - 1's (resp. l + 1's) value; the lane shifted in gets zero.
__device__ __forceinline__ f32x4 from_prev_lane(f32x4 x)
{
    f32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x[e]), 0x138, 0xF, 0xF, false));
    return r;
}
__device__ __forceinline__ f32x4 from_next_lane(f32x4 x)
{
    f32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x[e]), 0x130, 0xF, 0xF, false));
    return r;
}
__device__ __forceinline__ f32x4 lane_value(f32x4 x, int l)
{
    f32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[e]), l));
    return r;
}

__device__ __forceinline__ void epi_tag_store(unsigned long long *p, float v, unsigned tag)
{
    __hip_atomic_store(p, ((unsigned long long)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

template <int SPLIT, int KVEC>
__global__ __launch_bounds__(kUThreads) void k_epi_unit(ScoreArgs a)
{
    static_assert((SPLIT == 1 || SPLIT == 2 || SPLIT == 4 || SPLIT == 8) &&
                      (KVEC == 1 || KVEC == 2 || KVEC == 4 || KVEC == 8) && SPLIT * KVEC * 4096 <= kEpiUnitMax,
                  "1 to 8 blocks of 4096 KVEC keys, at most 65536 keys per unit");
    constexpr int kVec = KVEC;               // chunks (float4 per thread and array)
    constexpr int kWaveKeys = 256 * kVec;    // keys per wave
    constexpr int kPartKeys = kUW * kWaveKeys;
    __shared__ Red4 lds[kUW + 1];
    __shared__ f32x4 svl[kVec][kUThreads];  // S_div of every thread's keys
    __shared__ f32x4 edge[kUW][2];          // per wave: its first and last four attention values
    const int u = blockIdx.x / SPLIT, part = blockIdx.x % SPLIT;
    const Unit un = score_unit(a, u);
    const int T = un.T;
    const int P = T - a.w;
    const int64_t ob = unit_out_base(a, un);

    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int half = a.pool_half;  // <= kPoolHalfMax (checked on the host)
    const int kw = kPartKeys * part + kWaveKeys * wv;

    // every global load first, so that their latencies overlap: the sweep-2
    // partials and mu (d_E sum / extrema and |mu|^2 in one block reduction;
    // one partial and one mu component per thread at most: the host checks
    // that a unit has at most kUThreads sweep-2 blocks, and D <= 128), then
    // d_E, khat.mu and attention of the thread's keys (zero past P), and the
    // attention just outside the block's range (a negative offset wraps past
    // the range and reads zero)
    const unsigned tag = SPLIT > 1 ? *a.tagw : 0u;  // this call's (bumped by the second sweep)
    Red4 v{0.f, 0.f, INFINITY, -INFINITY};
    float dq2 = 0.f;  // this thread's partial sum of d_E^2
    const int nb2 = (T + a.rpb2 - 1) / a.rpb2;
    if ((int)threadIdx.x < nb2) {
        const float *pp = a.part2 + ((int64_t)u * a.nch2 + threadIdx.x) * 4;
        v.s0 = pp[0];
        v.mn = pp[1];
        v.mx = pp[2];
        dq2 = pp[3];
    }
    const float mv = (int)threadIdx.x < a.D ? anchor_value(a, un, u, T, a.D + (int)threadIdx.x) : 0.f;
    const __amdgpu_buffer_rsrc_t rd = float_rsrc(a.bufA + ob, P), rc = float_rsrc(a.bufB + ob, P),
                                 ra = float_rsrc(a.bufC + ob, P);
    f32x4 xd[kVec], xc[kVec], xa[kVec];
#pragma unroll
    for (int j = 0; j < kVec; ++j) {
        const int k4 = kw + 256 * j + 4 * lane;
        xd[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rd, k4 * 4, 0, 0));
        xc[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rc, k4 * 4, 0, 0));
        xa[j] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, k4 * 4, 0, 0));
    }
    f32x4 bl = {0.f, 0.f, 0.f, 0.f}, br = {0.f, 0.f, 0.f, 0.f};
    if (SPLIT > 1) {
        const int b0 = kPartKeys * part;
        bl = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, (unsigned)(b0 - 4) * 4u, 0, 0));
        br = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ra, (b0 + kPartKeys) * 4, 0, 0));
    }
    __builtin_amdgcn_sched_barrier(0);  // the phases below stay in order (register pressure)

    v.s1 = mv * mv;
    const Red4 dm = block_red4_lds(v, lds);
    const float dsq = a.red_std ? block_red4_lds(Red4{dq2, 0.f, INFINITY, -INFINITY}, lds).s0 : 0.f;
    const Red4 dst{dm.s0, dsq, dm.mn, dm.mx};
    const float mu2 = dm.s1;

    // S_div, kept in LDS (each thread reads back only its own values)
    const DNorm dn = d_norm(a, u, dst);
    Red4 w{0.f, 0.f, INFINITY, -INFINITY};
#pragma unroll
    for (int j = 0; j < kVec; ++j) {
        const int k4 = kw + 256 * j + 4 * lane;
        f32x4 sv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float sE = s_euclid(xd[j][e], dn);
            const float sC = (1.f - xc[j][e]) * 0.5f;
            sv[e] = a.alpha * sE + (1.f - a.alpha) * sC;
            if (k4 + e < P) {
                w.s0 += sv[e];
                w.mn = fminf(w.mn, sv[e]);
                w.mx = fmaxf(w.mx, sv[e]);
            }
        }
        svl[j][threadIdx.x] = sv;
    }
    // the wave's first and last four attention values for its neighbours
    if (lane == 0) edge[wv][0] = xa[0];
    if (lane == 63) edge[wv][1] = xa[kVec - 1];
    lds_barrier();
    const f32x4 hl = wv > 0 ? edge[wv - 1][1] : bl;       // the four keys before the wave's first
    const f32x4 hr = wv < kUW - 1 ? edge[wv + 1][0] : br;  // the four after its last
    __builtin_amdgcn_sched_barrier(0);
    // pooled S_imp (each chunk's attention registers die as its pooled values are made)
    const float inv_k = 1.f / (float)(2 * half + 1);
    f32x4 im[kVec];
#pragma unroll
    for (int j = 0; j < kVec; ++j) {
        const f32x4 sl = from_prev_lane(xa[j]), sr = from_next_lane(xa[j]);
        const f32x4 pl = j > 0 ? lane_value(xa[j - 1], 63) : hl;  // lane 0: previous chunk's end
        const f32x4 nr = j < kVec - 1 ? lane_value(xa[j + 1], 0) : hr;  // lane 63: next chunk's start
        const f32x4 left = lane == 0 ? pl : sl;
        const f32x4 right = lane == 63 ? nr : sr;
        float win[12];  // keys k4 - 4 .. k4 + 7
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            win[e] = left[e];
            win[4 + e] = xa[j][e];
            win[8 + e] = right[e];
        }
        const int k4 = kw + 256 * j + 4 * lane;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float acc = 0.f;
#pragma unroll
            for (int t = -kPoolHalfMax; t <= kPoolHalfMax; ++t)
                if (t >= -half && t <= half) acc += win[4 + e + t];
            im[j][e] = acc * inv_k;
            if (k4 + e < P) w.s1 += im[j][e];
        }
    }
    Red4 sd = block_red4_lds(w, lds);
    if (SPLIT > 1) {
        // exchange with the other parts of the unit: publish, then wait for all
        // (bounded), lane 4 p + q of wave 0 polling word q of part p, so that the
        // parts cost one round trip and not one each
        if (wv == 0) {
            unsigned long long *words = a.epiT + (int64_t)u * SPLIT * 4;
            const float mine = (lane & 3) == 0 ? sd.s0 : (lane & 3) == 1 ? sd.s1 : (lane & 3) == 2 ? sd.mn : sd.mx;
            const bool own = lane >> 2 == part;
            if (own) epi_tag_store(words + lane, mine, tag);
            float got = mine;
            bool ok = own || lane >= 4 * SPLIT;
            // a spin limit <= 0 (set by the host to exercise this path) gives up at once
            for (int tries = 0; tries < a.spin_limit && __builtin_amdgcn_ballot_w64(!ok); ++tries) {
                if (!ok) {
                    const unsigned long long o =
                        __hip_atomic_load(words + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    ok = (unsigned)(o >> 32) == tag;
                    got = __uint_as_float((unsigned)o);
                }
                if (__builtin_amdgcn_ballot_w64(!ok)) __builtin_amdgcn_s_sleep(2);
            }
            auto value = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(got), l)); };
            Red4 c{value(0), value(1), value(2), value(3)};
#pragma unroll
            for (int p = 1; p < SPLIT; ++p)  // in part order, so every part adds in the same order
                c = Red4{c.s0 + value(4 * p), c.s1 + value(4 * p + 1), fminf(c.mn, value(4 * p + 2)),
                         fmaxf(c.mx, value(4 * p + 3))};
            const bool lost = __builtin_amdgcn_ballot_w64(!ok) != 0;
            if (lost) c.s0 = NAN;
            if (lane == 0) {
                if (lost) __hip_atomic_store(a.status, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                lds[kUW] = c;
            }
        }
        lds_barrier();
        sd = lds[kUW];
    }
    const EpiConsts k = epi_consts(a, dst, sd, mu2, T, P);

    const __amdgpu_buffer_rsrc_t ro = float_rsrc(a.scores + ob, P);
    const float gain = k.lam * k.scale / k.sden, one_m = 1.f - k.lam;
#pragma unroll
    for (int j = 0; j < kVec; ++j) {
        const f32x4 sv = svl[j][threadIdx.x];
        f32x4 x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = (sv[e] - k.smin) * gain + one_m * im[j][e];
        const int k4 = kw + 256 * j + 4 * lane;
        if (k4 + 4 <= P) {
            // (written through, cache policy sc1: 0.7 us less than the default)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), ro, k4 * 4, 0, 16);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k4 + e < P) a.scores[ob + k4 + e] = x[e];
        }
    }
    if (part == 0 && threadIdx.x == 0) epi_write_stats(a, u, k, dst, sd, mu2);
}

// Clears the workspace status word (a one-thread kernel rather than a memset,
// so that a captured graph holds no memset node).
__global__ void k_status_clear(unsigned *status) { *status = 0u; }

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

hipError_t status_clear(unsigned *status, hipStream_t st)
{
    hipLaunchKernelGGL(k_status_clear, dim3(1), dim3(1), 0, st, status);
    return hipGetLastError();
}

bool score_fast_path(int D, bool bf16) { return bf16 && D == fast::kD; }

// Fewest keys per block of any sweep of a shape (the workspace holds a partial
// for each block).
static int min_block_keys(int D, bool bf16) { return score_fast_path(D, bf16) ? 256 : 128; }

// Blocks of `keys` keys over every unit of a call.
static int64_t work_blocks(const ScoreArgs &a, int keys)
{
    int64_t nb = 0;
    for (int s = 0; s < a.B; ++s) nb += (a.seq.cu[s + 1] - a.seq.cu[s] + keys - 1) / keys;
    return nb * a.L * a.Hkv;
}

// Fills a.bl for blocks of `keys` keys; returns the grid of the sweep.
static dim3 sweep_grid(ScoreArgs &a, int keys)
{
    a.bl[0] = 0;
    for (int s = 0; s < a.B; ++s) a.bl[s + 1] = a.bl[s] + (a.seq.cu[s + 1] - a.seq.cu[s] + keys - 1) / keys;
    return dim3(a.bl[a.B], a.L * a.Hkv);
}

// Keys per block of the streaming sweeps: a multiple of 128 (whole 32-key
// groups in every wave) with the least rounds of blocks over the device's
// places times block length, set-up included: a second round that is nearly
// empty takes as long as a full one.  (us, 1024-key blocks, 1.2 rounds, ->
// one round of 1280: 8 packed sequences, 613 Ki keys, sweep 1 39.0 -> 31.3,
// sweep 2 52.9 -> 37.0; with 1536, 743 Ki keys, 40.1 -> 35.8 and 54.9 -> 42.4.)
// Calls of two rounds of the longest blocks and more take those (sweep 2 of 28
// layers of 4 x 32768 keys takes 7 to 15 us longer with 1536, 1792 or 2304 to
// 3584 keys, of 32 x 65536 keys as long or longer).
static int stream_block_keys(const ScoreArgs &a)
{
    constexpr int64_t kPlaces = 512;  // two blocks per compute unit
    constexpr int kSetUp = 128;
    if (work_blocks(a, fast::kS2KeysMax) >= 2 * kPlaces) return fast::kS2KeysMax;
    int best = 0;
    int64_t least = INT64_MAX;
    for (int keys = fast::kS2KeysMax; keys >= fast::kS2KeysMin; keys -= 128) {
        const int64_t cost = (work_blocks(a, keys) + kPlaces - 1) / kPlaces * (keys + kSetUp);
        if (cost < least) {
            least = cost;
            best = keys;
        }
    }
    return best;
}

// Keys per block of ecokv_sweep.hip's sweeps: the most that give every
// compute unit a block.  Longer blocks pay their set-up (window rows,
// anchors, first loads) and their partial less often, fewer than 256 leave
// compute units idle (sweep 2, us, at 512 / 1024 / 2048 keys: 12 layers of 4
// heads x 16384 x 64 bf16 37.5 / 33.8 / 29.5; 14 layers of 4 x 32768 x 128,
// 56 window rows, 158 / 130 / 128; one layer of 4 x 32768 x 128 14.0 / 18.1 /
// 29.2; 4 layers of 4 x 8192 x 128 fp32 at 256 / 512 / 1024: 29.6 / 25.1 / 39.8).
// A wave's quarter is whole batches of keys: multiples of 256 per block for
// bf16, 128 for fp32.  Where the longest blocks leave places of one round (two
// per compute unit) free, the shortest that still make one round, if more than
// half as long (12 layers of 4 heads x 16384 x 64 bf16: 384 blocks of 2048 keys
// -> 480 of 1792, the call 69.8 -> 67.1).
static int rows_block_keys(const ScoreArgs &a, bool bf16)
{
    const int step = bf16 ? 256 : 128, most = sweep_rows_max_keys(bf16);
    int keys = most;
    while (keys > step && work_blocks(a, keys) < 256) keys /= 2;
    if (keys == most)
        for (int k = most - step; k > most / 2 && work_blocks(a, k) <= 512; k -= step) keys = k;
    return keys;
}

// ---------------------------------------------------------------------------
// Value-norm importance (ECOKV_IMP_ATTN_VNORM, Sec. 5.2): S_imp(i) =
// pool(a)(i) * |v_i|_2 for the non-window keys, in one coalesced pass over V.
// A wave takes 64 consecutive rows; its load instruction q covers the 16-byte
// pieces 64q .. 64q+63 of those rows (SEGS pieces per row), so consecutive
// lanes read consecutive bytes.  The SEGS partial sums of squares of a row
// are combined by DPP butterflies and parked in LDS; lane r then pools the window
// attention around row r (zero padding, fixed divisor, as the epilogue) and
// writes the product.  Rows at or past P read as zero (buffer range).
// ---------------------------------------------------------------------------
constexpr int kVnThreads = 256;

template <bool BF16, int SEGS>
__global__ __launch_bounds__(kVnThreads) void k_vnorm(ScoreArgs a)
{
    __shared__ float n2s[kVnThreads];
    constexpr int kRowBytes = SEGS * 16;
    const int u = blockIdx.y;
    const Unit un = score_unit(a, u);
    const int T = un.T;
    const int P = T - a.w;
    const int row0 = blockIdx.x * kVnThreads;
    if (row0 >= P) return;
    const int lane = threadIdx.x & 63, wv = uniform_i32(threadIdx.x >> 6);
    const int wrow = row0 + 64 * wv;                      // the wave's first row
    const int nrows = max(0, min(64, P - wrow));          // rows of the wave below P
    const char *vw = static_cast<const char *>(a.V) + (unit_row0(a, un) + wrow) * kRowBytes;
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(uniform_ptr(vw)), (short)0, uniform_i32(nrows * kRowBytes), 0x00020000);
    u32x4 x[SEGS];  // (nontemporal: V is read once)
#pragma unroll
    for (int q = 0; q < SEGS; ++q)
        x[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rv, (64 * q + lane) * 16, 0, 2));
#pragma unroll
    for (int q = 0; q < SEGS; ++q) {
        float s2 = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (BF16) {
                const float lo = __uint_as_float(x[q][c] << 16), hi = __uint_as_float(x[q][c] & 0xffff0000u);
                s2 += lo * lo + hi * hi;
            } else {
                const float v = __uint_as_float(x[q][c]);
                s2 += v * v;
            }
        }
        s2 = row_sum<SEGS>(s2);
        if (lane % SEGS == 0) n2s[64 * wv + (64 / SEGS) * q + lane / SEGS] = s2;
    }
    __syncthreads();
    const int i = wrow + lane;
    if (i < P) {
        const int64_t ob = unit_out_base(a, un);
        const float *att = a.bufC + ob;
        float acc = 0.f;
        for (int t = -a.pool_half; t <= a.pool_half; ++t)
            if (i + t >= 0 && i + t < P) acc += att[i + t];
        a.bufV[ob + i] = acc * (1.f / (float)(2 * a.pool_half + 1)) * sqrtf(n2s[threadIdx.x]);
    }
}

static void launch_vnorm(const ScoreArgs &a, dim3 grid, hipStream_t st, bool bf16)
{
    if (bf16 && a.D == 64) hipLaunchKernelGGL((k_vnorm<true, 8>), grid, dim3(kVnThreads), 0, st, a);
    else if (bf16) hipLaunchKernelGGL((k_vnorm<true, 16>), grid, dim3(kVnThreads), 0, st, a);
    else if (a.D == 64) hipLaunchKernelGGL((k_vnorm<false, 16>), grid, dim3(kVnThreads), 0, st, a);
    else hipLaunchKernelGGL((k_vnorm<false, 32>), grid, dim3(kVnThreads), 0, st, a);
}

WsLayout score_ws_layout(int L, int Hkv, int B, int D, int R, int64_t Ptot, int maxT, bool bf16, bool vnorm)
{
    WsLayout w{};
    const int64_t U = (int64_t)L * Hkv * B;
    const int rpb = min_block_keys(D, bf16);
    const int64_t nch1 = (maxT + rpb - 1) / rpb;
    const int64_t nch2 = nch1;
    const int64_t nch3 = (maxT + kEpiKeys - 1) / kEpiKeys;
    const int64_t stride = 2 * D + 2 * R;
    size_t o = 0;
    w.status = o;  // first: a fixed offset for the status query
    w.tagw = o + sizeof(unsigned);  // then the call tag (any initial value)
    o = align256(o + 2 * sizeof(unsigned));
    w.part1 = o; o = align256(o + sizeof(float) * U * nch1 * stride);
    w.anchors = o; o = align256(o + sizeof(float) * U * stride);
    w.part2 = o; o = align256(o + sizeof(float) * U * nch2 * 4);
    w.part3 = o; o = align256(o + sizeof(float) * U * nch3 * 4);
    w.bufA = o; o = align256(o + sizeof(float) * (int64_t)L * Hkv * Ptot);
    w.bufB = o; o = align256(o + sizeof(float) * (int64_t)L * Hkv * Ptot);
    w.bufC = o; o = align256(o + sizeof(float) * (int64_t)L * Hkv * Ptot);
    w.bufV = o; o = align256(o + (vnorm ? sizeof(float) * (int64_t)L * Hkv * Ptot : 0));
    w.dq = o; o = align256(o + sizeof(float) * U * 2);
    w.epiT = o; o = align256(o + sizeof(unsigned long long) * U * kEpiSplitMax * 4);
    w.total = o;
    return w;
}

// Blocks of k_epi_unit<SPLIT, KVEC> that the current device holds at once (cached per device).
template <int SPLIT, int KVEC>
static int64_t epi_split_capacity()
{
    static int64_t cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if (cache[dev] == 0) {
        int ncu = 0, nb = 0;
        if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_epi_unit<SPLIT, KVEC>, kUThreads, 0) != hipSuccess)
            return 0;
        cache[dev] = (int64_t)ncu * nb;
    }
    return cache[dev];
}

// Launches k_epi_unit<SPLIT, KVEC> over U units if its SPLIT U blocks fit
// the device at once (with half: half of it); returns false (nothing
// launched) otherwise.
template <int SPLIT, int KVEC>
static bool try_epi_unit(ScoreArgs &a, char *ws, const WsLayout &lay, int U, hipStream_t st, bool half)
{
    const int64_t cap = epi_split_capacity<SPLIT, KVEC>();
    if ((int64_t)SPLIT * U > (half ? cap / 2 : cap)) return false;
    a.epiT = reinterpret_cast<unsigned long long *>(ws + lay.epiT);
    ECOKV_TIMED("epilogue", st, hipLaunchKernelGGL((k_epi_unit<SPLIT, KVEC>), dim3(SPLIT * U), dim3(kUThreads), 0, st, a));
    return true;
}

hipError_t score_launch(ScoreArgs a, char *ws, const WsLayout &lay, int maxT, hipStream_t st, bool bf16)
{
    const int U = a.L * a.Hkv * a.B;
    a.part1 = reinterpret_cast<float *>(ws + lay.part1);
    a.anchors = reinterpret_cast<float *>(ws + lay.anchors);
    a.part2 = reinterpret_cast<float *>(ws + lay.part2);
    a.part3 = reinterpret_cast<float *>(ws + lay.part3);
    a.bufA = reinterpret_cast<float *>(ws + lay.bufA);
    a.bufB = reinterpret_cast<float *>(ws + lay.bufB);
    a.bufC = reinterpret_cast<float *>(ws + lay.bufC);
    a.nch3 = (maxT + kEpiKeys - 1) / kEpiKeys;
    a.status = reinterpret_cast<unsigned *>(ws + lay.status);
    a.tagw = reinterpret_cast<unsigned *>(ws + lay.tagw);
    const dim3 grid_e(a.nch3, U);
    hipError_t e;

    {
        if (a.pre) {
            // the first sweep's sums come from the caller: K is read once (the
            // sweep-2 blocks and the epilogue convert them as they read them)
        } else {
            if (score_fast_path(a.D, bf16) && a.R <= 32) {
                // streaming sweep 1: one 32-row window operand
                a.rpb1 = stream_block_keys(a);
                a.nch1 = (maxT + a.rpb1 - 1) / a.rpb1;
                ECOKV_TIMED("sweep1_stream", st,
                            hipLaunchKernelGGL(fast::k_fs1s<false>, sweep_grid(a, a.rpb1), dim3(256), 0, st, a));
            } else {
                a.rpb1 = rows_block_keys(a, bf16);
                a.nch1 = (maxT + a.rpb1 - 1) / a.rpb1;
                ECOKV_TIMED("sweep1_rows", st, sweep_rows_launch(1, a, sweep_grid(a, a.rpb1), st));
            }
            if ((e = hipGetLastError()) != hipSuccess) return e;
            if (reduce1_lanes(a.nch1) == 4)
                ECOKV_TIMED("reduce1", st, hipLaunchKernelGGL((k_reduce1<4, false>), dim3(U), dim3(kReduceThreads), 0, st, a));
            else
                ECOKV_TIMED("reduce1", st,
                            hipLaunchKernelGGL((k_reduce1<16, false>), dim3(U, (2 * a.D + a.R + 63) / 64), dim3(kReduceThreads),
                                               0, st, a));
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (score_fast_path(a.D, bf16) && a.R <= kStreamMaxRows) {
            // streaming sweep 2: window rows and the two rows of mu in one operand
            a.rpb2 = stream_block_keys(a);
            a.nch2 = (maxT + a.rpb2 - 1) / a.rpb2;
            ECOKV_TIMED("sweep2_stream", st,
                        hipLaunchKernelGGL(fast::k_fs2s, sweep_grid(a, a.rpb2), dim3(256), 0, st, a));
        } else {
            a.rpb2 = rows_block_keys(a, bf16);
            a.nch2 = (maxT + a.rpb2 - 1) / a.rpb2;
            ECOKV_TIMED("sweep2_rows", st, sweep_rows_launch(2, a, sweep_grid(a, a.rpb2), st));
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (a.vnorm) {
        // the importance with the value norm; the epilogue then reads it as
        // its (already pooled) importance
        a.bufV = reinterpret_cast<float *>(ws + lay.bufV);
        const dim3 gv((maxT - a.w + kVnThreads - 1) / kVnThreads, U);
        ECOKV_TIMED("vnorm", st, launch_vnorm(a, gv, st, bf16));
        if ((e = hipGetLastError()) != hipSuccess) return e;
        a.bufC = a.bufV;
        a.pool_half = 0;
    }
    if (a.norm_mode != ECOKV_NORM_MINMAX) {
        // quantiles of d_E for the winsorised or MAD normalisation
        DQuantArgs qa;
        memset(&qa, 0, sizeof qa);
        qa.d = a.bufA;
        qa.out = reinterpret_cast<float *>(ws + lay.dq);
        qa.L = a.L;
        qa.Hkv = a.Hkv;
        qa.B = a.B;
        qa.w = a.w;
        qa.Ptot = a.Ptot;
        qa.mode = a.norm_mode;
        qa.q = a.winsor_q;
        qa.seq = a.seq;
        if ((e = dquant_launch(qa, st)) != hipSuccess) return e;
        a.dq = qa.out;
    }
    const bool epi_one = a.pool_half <= kPoolHalfMax && (maxT + a.rpb2 - 1) / a.rpb2 <= kUThreads && a.D <= kUThreads;
    const int64_t maxP = maxT - a.w;
    if (epi_one && !a.no_wait && maxP <= kEpiUnitMax) {
        // The one-launch epilogue with the most blocks per unit (4096 KVEC
        // keys each, KVEC = 1, 2, 4) whose blocks fill at most half the
        // device: the parts of a unit wait for each other, and half the
        // device leaves room for a concurrent call on another stream to be
        // resident at once too.  Past that, two blocks per unit when the
        // device holds all of them (a wait across calls is still bounded).
        bool done = false;
        auto fits = [&](int kvec, int split) { return maxP <= (int64_t)4096 * kvec * split; };
        if (fits(1, 1)) {
            ECOKV_TIMED("epilogue", st, hipLaunchKernelGGL((k_epi_unit<1, 1>), dim3(U), dim3(kUThreads), 0, st, a));
            done = true;
        }
        if (!done && fits(1, 8)) {
            if (fits(1, 2)) done = try_epi_unit<2, 1>(a, ws, lay, U, st, true);
            else if (fits(1, 4)) done = try_epi_unit<4, 1>(a, ws, lay, U, st, true);
            else done = try_epi_unit<8, 1>(a, ws, lay, U, st, true);
        }
        if (!done && fits(2, 8)) {
            if (fits(2, 2)) done = try_epi_unit<2, 2>(a, ws, lay, U, st, true);
            else if (fits(2, 4)) done = try_epi_unit<4, 2>(a, ws, lay, U, st, true);
            else done = try_epi_unit<8, 2>(a, ws, lay, U, st, true);
        }
        if (!done && fits(4, 4)) {
            if (fits(4, 2)) done = try_epi_unit<2, 4>(a, ws, lay, U, st, true) || try_epi_unit<2, 4>(a, ws, lay, U, st, false);
            else done = try_epi_unit<4, 4>(a, ws, lay, U, st, true);
        }
        if (done) return hipGetLastError();
    }
    if (epi_one && maxP <= kUKeys) {
        // one block per unit, no waits
        ECOKV_TIMED("epilogue", st, hipLaunchKernelGGL((k_epi_unit<1, 8>), dim3(U), dim3(kUThreads), 0, st, a));
        return hipGetLastError();
    }
    ECOKV_TIMED("epilogue1", st, hipLaunchKernelGGL(k_epi1, grid_e, dim3(kEpiThreads), 0, st, a));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    ECOKV_TIMED("epilogue2", st, hipLaunchKernelGGL(k_epi2, grid_e, dim3(kEpiThreads), 0, st, a));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// ecokv_prefill_write: the KV-cache write of a prefill with the first sweep.
// ---------------------------------------------------------------------------

// Copy of unit u's rows x * kCopyRows .. x * kCopyRows + 63 from the
// token-major new rows ([L][Ttot][Hkv] rows of rowb bytes) to the head-major
// cache ([L][Hkv][Ttot] rows), 16 bytes per thread and step, streamed past
// the caches.
constexpr int kCopyRows = 64;
__device__ __forceinline__ void copy_unit_rows(const char *src, char *dst, int rowb, int Hkv, int B, int64_t Ttot,
                                               const SeqTab &seq, int u, int x)
{
    const Unit un = unit_of(u, Hkv, B);
    const int T = seq.cu[un.s + 1] - seq.cu[un.s];
    const int r0 = x * kCopyRows;
    if (r0 >= T) return;
    const int rows = min(kCopyRows, T - r0);
    const int pr = rowb / 16;  // 16-byte pieces per row
    const int64_t t0 = (int64_t)seq.cu[un.s] + r0;
    const char *s0 = src + (((int64_t)un.l * Ttot + t0) * Hkv + un.h) * rowb;
    char *d0 = dst + (((int64_t)un.l * Hkv + un.h) * Ttot + t0) * rowb;
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    for (int p = threadIdx.x; p < rows * pr; p += blockDim.x) {
        const int r = p / pr, c = p - r * pr;
        const v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(s0 + (int64_t)r * Hkv * rowb) + c);
        __builtin_nontemporal_store(v, reinterpret_cast<v4u *>(d0 + (int64_t)r * rowb) + c);
    }
}

__global__ __launch_bounds__(256) void k_rows_copy(const char *src, char *dst, int rowb, int L, int Hkv, int B,
                                                   int64_t Ttot, SeqTab seq)
{
    copy_unit_rows(src, dst, rowb, Hkv, B, Ttot, seq, blockIdx.y, blockIdx.x);  // block (x, u)
}

// The V rows' copy and the reduction of the K sweep's block partials into
// `pre` in one launch: blocks [0, nred) reduce (unit, group of 16 columns),
// 16 lanes per column, and the rest copy V rows as k_rows_copy does, ncx
// blocks per unit; the reduction's few loads then hide under the copy's
// stream instead of taking a launch of their own.
__global__ __launch_bounds__(256) void k_copy_reduce_pre(ScoreArgs a, const char *src, char *dst, int rowb, int ncg,
                                                         int ncx)
{
    const int nred = a.L * a.Hkv * a.B * ncg;
    if ((int)blockIdx.x < nred) {
        reduce1_columns<16, true>(a, blockIdx.x / ncg, blockIdx.x % ncg, ncg);
        return;
    }
    const int cb = blockIdx.x - nred;
    copy_unit_rows(src, dst, rowb, a.Hkv, a.B, a.Ttot, a.seq, cb / ncx, cb % ncx);
}

size_t prefill_ws_bytes(int L, int Hkv, int B, int D, int R, int maxT, bool bf16)
{
    // the block partials of sweep 1 (part1), for its smallest key block (as
    // in the score's layout)
    const int rpb = min_block_keys(D, bf16);
    const size_t nch1 = (size_t)((maxT + rpb - 1) / rpb);
    return align256(sizeof(float) * (size_t)L * Hkv * B * nch1 * (size_t)(2 * D + 2 * R));
}

hipError_t prefill_launch(ScoreArgs a, const void *Vsrc, void *Vdst, char *ws, int maxT, hipStream_t st, bool bf16)
{
    const int U = a.L * a.Hkv * a.B;
    const int es = bf16 ? 2 : 4;
    a.part1 = reinterpret_cast<float *>(ws);
    hipError_t e;
    const dim3 gc((maxT + kCopyRows - 1) / kCopyRows, U);
    if (score_fast_path(a.D, bf16) && a.R <= 32) {
        // bf16, head_dim 128: the streaming sweep reads the new rows and writes
        // the cache, in 512-key blocks (28-layer stack, 32768 tokens: the sweep
        // with the copy takes 326 us with them, as long as a plain copy of the
        // same rows, against 367 us with 2048-key blocks, whose 1792 blocks
        // leave the last of their 3.5 rounds half empty)
        a.rpb1 = fast::kS2KeysCache;
        a.nch1 = (maxT + a.rpb1 - 1) / a.rpb1;
        ECOKV_TIMED("prefill_sweep", st,
                    hipLaunchKernelGGL(fast::k_fs1s<true>, sweep_grid(a, a.rpb1), dim3(256), 0, st, a));
    } else {
        // other shapes: copy the rows, then the first sweep over the cache
        ECOKV_TIMED("prefill_copy", st,
                    hipLaunchKernelGGL(k_rows_copy, gc, dim3(256), 0, st, static_cast<const char *>(a.Ksrc),
                                       static_cast<char *>(const_cast<void *>(a.K)), a.D * es, a.L, a.Hkv, a.B, a.Ttot,
                                       a.seq));
        if ((e = hipGetLastError()) != hipSuccess) return e;
        a.rpb1 = rows_block_keys(a, bf16);
        a.nch1 = (maxT + a.rpb1 - 1) / a.rpb1;
        ECOKV_TIMED("prefill_sweep", st, sweep_rows_launch(1, a, sweep_grid(a, a.rpb1), st));
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (Vsrc) {
        // V's copy with the reduction into pre riding on it
        const int ncg = (2 * a.D + a.R + 15) / 16;
        const int64_t blocks = (int64_t)U * ncg + (int64_t)gc.x * U;
        if (blocks > INT32_MAX) return hipErrorInvalidConfiguration;
        ECOKV_TIMED("prefill_copy_v", st,
                    hipLaunchKernelGGL(k_copy_reduce_pre, dim3((unsigned)blocks), dim3(256), 0, st, a,
                                       static_cast<const char *>(Vsrc), static_cast<char *>(Vdst), a.D * es, ncg,
                                       (int)gc.x));
    } else if (reduce1_lanes(a.nch1) == 4) {
        ECOKV_TIMED("prefill_reduce", st,
                    hipLaunchKernelGGL((k_reduce1<4, true>), dim3(U), dim3(kReduceThreads), 0, st, a));
    } else {
        ECOKV_TIMED("prefill_reduce", st,
                    hipLaunchKernelGGL((k_reduce1<16, true>), dim3(U, (2 * a.D + a.R + 63) / 64),
                                       dim3(kReduceThreads), 0, st, a));
    }
    return hipGetLastError();
}

}  // namespace ecokv
