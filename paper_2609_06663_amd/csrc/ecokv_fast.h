// Device helpers shared by the score kernels (gfx950): vector types, unit
// addressing, log2-domain softmax merging, the anchors of the second sweep and
// the LDS stage geometry of the bf16 / head_dim 128 path.  Not part of the ABI.
#pragma once

#include "ecokv_internal.h"

namespace ecokv {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Unit u with its sequence's place.
__device__ __forceinline__ Unit score_unit(const ScoreArgs &a, int u)
{
    Unit un = unit_of(u, a.Hkv, a.B);
    const SeqSpan q = seq_span(a.seq, a.B, un.s);
    un.c0 = q.c0;
    un.T = q.T;
    return un;
}

__device__ __forceinline__ int64_t unit_out_base(const ScoreArgs &a, const Unit &un)
{
    return (int64_t)un.lh * a.Ptot + (un.c0 - un.s * a.w);
}

__device__ __forceinline__ int64_t unit_row0(const ScoreArgs &a, const Unit &un)
{
    return (int64_t)un.lh * a.Ttot + un.c0;
}

// Global row index of window row r = (g, j) of unit `un` in Q_win.
__device__ __forceinline__ int64_t window_row(const ScoreArgs &a, const Unit &un, int r)
{
    const int g = r / a.w, j = r % a.w;
    return (((int64_t)un.lh * a.G + g) * a.B + un.s) * a.w + j;
}

// The unit u and the block x of its keys that this block of a sweep takes.
// The grid holds exactly the blocks that have keys (a.bl): with a place for
// every block of the longest sequence in every unit, ragged calls end up
// with unequal numbers of working blocks on the eight XCDs, to which
// consecutive blocks are dealt in turn.
struct SweepBlock {
    Unit un;
    int u, x;
};
__device__ __forceinline__ SweepBlock sweep_block(const ScoreArgs &a)
{
    // grid (blocks of a pair, pairs)
    SweepBlock b;
    const int lh = blockIdx.y, r = blockIdx.x;
    int s = 0;
    if (a.B > 1)
        for (int n = a.B; n > 1;) {  // the last s with bl[s] <= r
            const int half = n >> 1;
            if (a.bl[s + half] <= r) s += half;
            n -= half;
        }
    b.x = a.B > 1 ? r - a.bl[s] : r;
    const SeqSpan q = seq_span(a.seq, a.B, s);
    const int l = lh / a.Hkv;
    b.un = Unit{l, lh - l * a.Hkv, q.s, lh, q.c0, q.T};
    b.u = lh * a.B + q.s;
    return b;
}

constexpr float kLog2e = 1.4426950408889634f;

// Combine two softmax partials (max, sum of 2^(x - max)), x in log2 units.
__device__ __forceinline__ void softmax_merge2(float &m, float &s, float m2, float s2)
{
    const float nm = fmaxf(m, m2);
    const float a = (m == -INFINITY) ? 0.f : s * __builtin_amdgcn_exp2f(m - nm);
    const float b = (m2 == -INFINITY) ? 0.f : s2 * __builtin_amdgcn_exp2f(m2 - nm);
    m = nm;
    s = a + b;
}

// Component c of kbar from the sum of the unit's T keys: divided by T, or,
// with the centroid over the non-window keys, the w window rows taken out
// and divided by P.
__device__ __forceinline__ float centroid_component(const ScoreArgs &a, const Unit &un, int T, int c, float s)
{
    if (!a.centroid_prefix) return s / (float)T;
    const int64_t r0 = unit_row0(a, un) + (T - a.w);
    float ws = 0.f;
    for (int j = 0; j < a.w; ++j) {
        const int64_t off = (r0 + j) * a.D + c;
        ws += a.kbf16 ? __uint_as_float((uint32_t)static_cast<const uint16_t *>(a.K)[off] << 16)
                      : static_cast<const float *>(a.K)[off];
    }
    return (s - ws) / (float)(T - a.w);
}

// Anchor column c of unit u (the layout of a.anchors: kbar, mu, the window
// rows' base-2 references and sums): from the workspace after the first sweep,
// or converted from the sums a prefill handed over (ecokv_score_pre: plain
// sums over the T keys, references in natural units).
__device__ __forceinline__ float anchor_load(const ScoreArgs &a, int u, int c)
{
    return (a.pre ? a.pre : a.anchors)[(int64_t)u * (2 * a.D + 2 * a.R) + c];
}
__device__ __forceinline__ float anchor_convert(const ScoreArgs &a, const Unit &un, int T, int c, float v)
{
    if (!a.pre) return v;
    if (c < a.D) return centroid_component(a, un, T, c, v);
    if (c < 2 * a.D) return v / (float)T;
    if (c < 2 * a.D + a.R) return v * kLog2e;
    return v;
}
__device__ __forceinline__ float anchor_value(const ScoreArgs &a, const Unit &un, int u, int T, int c)
{
    return anchor_convert(a, un, T, c, anchor_load(a, u, c));
}

// The workspace's exchange tag, bumped once per score call by the second
// sweep's first block, when it is done, and read by the split epilogue after it, so that every
// call (every replay of a captured call included) tags its exchanges afresh
// and never reads an older call's words (0 is skipped: the status word
// records the tag of a call whose wait gave up).
__device__ __forceinline__ void bump_call_tag(const ScoreArgs &a)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        const unsigned t = *a.tagw + 1u;
        *a.tagw = t ? t : 1u;
    }
}

namespace fast {

// Hot-loop transcendentals as single instructions (v_exp_f32, v_rsq_f32,
// v_sqrt_f32, about 1 ulp).  Every exponent argument here is <= 0, so results
// below 2^-126 (flushed to zero) are negligible next to the softmax terms of
// size 1 they are added to.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

constexpr int kD = 128;
constexpr int kChunks = 16;           // 16-byte chunks per key row

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void unpack8(u32x4 q, float *v)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[2 * e] = __uint_as_float(q[e] << 16);
        v[2 * e + 1] = __uint_as_float(q[e] & 0xffff0000u);
    }
}

// acc + lo*lo + hi*hi of the two bf16 halves of w (v_dot2c_f32_bf16).
__device__ __forceinline__ float dot2sq(unsigned w, float acc)
{
    const bf16x2 v = __builtin_bit_cast(bf16x2, w);
    return __builtin_amdgcn_fdot2_f32_bf16(v, v, acc, false);
}

// Round-to-nearest-even bf16 of a finite float (bit pattern in the low half).
__device__ __forceinline__ unsigned bf16_rne(float f)
{
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// Swizzled position of 16-byte chunk c of tile row r.
__device__ __forceinline__ int sw(int r, int c) { return r * kChunks + (c ^ (r & 15)); }

// Buffer descriptor over the key rows [0, rows) of a unit (raw buffer, no
// stride): loads at or past the end return zero without touching memory.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t key_rows_rsrc(const uint16_t *krow0, int rows)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(krow0), (short)0, rows * (kD * 2), 0x00020000);
}

// group_load over rows `row_bytes` apart (key rows interleaved with other
// heads' rows, as a projection writes them): the same lane layout.
__device__ __forceinline__ void group_load_rows(u32x4 (&b)[8], __amdgpu_buffer_rsrc_t rs, int key0, int lane,
                                                int row_bytes)
{
#pragma unroll
    for (int i = 0; i < 8; ++i)
        b[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (key0 + 4 * i + (lane >> 4)) * row_bytes + (lane & 15) * 16, 0,
                                                     2);
}

// Store of 32 key rows held in the load layout of group_load to consecutive
// 256-byte rows (stores at or past the descriptor's end are dropped).
__device__ __forceinline__ void group_store(const u32x4 (&b)[8], __amdgpu_buffer_rsrc_t rs, int key0, int lane)
{
#pragma unroll
    for (int i = 0; i < 8; ++i)
        __builtin_amdgcn_raw_buffer_store_b128(b[i], rs, (key0 + 4 * i + (lane >> 4)) * (kD * 2) + (lane & 15) * 16, 0,
                                               2);
}

}  // namespace fast
}  // namespace ecokv
