// How ecokv_decode splits the rows of a call over blocks: the arithmetic that
// the workspace size, the grid and the kernels share.  Values only, no device
// state, so that it can be evaluated on the host for any shape.
#pragma once

#include <math.h>
#include <stddef.h>
#include <stdint.h>

namespace ecokv {

constexpr int kDecWaves = 4;      // waves per block
constexpr int kWaveRows = 192;    // rows per wave at most (256 measured no faster)
constexpr int kMinWaveRows = 32;  // and at least: a wave's second tile loads while its first is used
constexpr int kDecChunk = kDecWaves * kWaveRows;
constexpr int kDecQG = 8;         // query heads per block at most
constexpr int kOneRound = 256;    // blocks that give every compute unit one
constexpr int kOneRows = 128;     // rows per wave up to which one round is enough
constexpr int kGridX = 1 << 20;   // blocks along x at most: a dimension's threads past 2^32 would wrap round
constexpr int kPlanPer = 4;       // units per lane of a balanced plan
constexpr int kPlanUnits = kPlanPer * 64;  // and at most

// Query heads per block: all of G up to 8 (so that Kc / Vc are read once),
// rounded up to 1, 2, 4 or 8; larger G takes several blocks of 8 per chunk.
__host__ __device__ inline int decode_qg(int G) { return G > 4 ? kDecQG : G > 2 ? 4 : G; }
__host__ __device__ inline int decode_head_groups(int G) { return (G + decode_qg(G) - 1) / decode_qg(G); }

__host__ __device__ inline int clamp_wave_rows(int rows)
{
    const int r = (rows + 15) & ~15;  // whole 16-row tiles
    return r < kMinWaveRows ? kMinWaveRows : r > kWaveRows ? kWaveRows : r;
}

// Rows per wave of a unit of n rows in np fixed chunks.
__host__ __device__ inline int fixed_wave_rows(int n, int np)
{
    return clamp_wave_rows((n + kDecWaves * np - 1) / (kDecWaves * np));
}

// Rows per wave of a balanced plan over `units` units of `rows` rows in all,
// each chunk read by zg blocks (one per group of query heads), so that a round
// of blocks holds 1 / zg as many chunks; 0 where the call takes fixed chunks.
// The chunks of a plan, sum of ceil(n / chunk) <= units + rows / chunk, always
// fit decode_grid's blocks: with `one` or `two` rows per wave
// rows / chunk <= (2 kOneRound - units / 2) / zg, and the half unit left over
// is more than the rounding of `rows`; at kWaveRows the chunk is kDecChunk.
// Where even two rounds would take more than kWaveRows rows, units that are
// nearly all of max_count rows take fixed chunks too: those launch chunk by
// chunk of every unit, so that the units' shorter last chunks end the call (256
// units of 1600 fp32 rows of 128 dimensions 78 -> 65 us).
struct PlanScale {
    float one, two;  // rows per wave in one and in two rounds, per row of the call
    float full;      // rows from which on units are nearly full
};
inline PlanScale plan_scale(int64_t units, int zg, int max_count)
{
    const float lost = 0.5f * (float)units;  // a unit's last chunk is half empty on average
    const float per = (float)zg / (float)kDecWaves;
    return PlanScale{per / (kOneRound - lost), per / (2 * kOneRound - lost), 0.75f * (float)units * (float)max_count};
}
__host__ __device__ inline int plan_wave_rows(float rows, PlanScale p)
{
    const float one = rows * p.one, two = rows * p.two;
    if (two > 2.f * (float)kWaveRows || (two > (float)kWaveRows && rows > p.full)) return 0;
    return clamp_wave_rows((int)ceilf(one <= (float)kOneRows ? one : two));
}

// Chunks of a unit of n rows.
__host__ __device__ inline int unit_chunks(int n, int wave_rows)
{
    return (n + kDecWaves * wave_rows - 1) / (kDecWaves * wave_rows);
}

// Chunks, blocks (per group of query heads) and workspace of a call.
//  * `least`, what any call can do with: one chunk for every kDecChunk rows of
//    max_count.  Calls of at most two such chunks (max_count up to 1536) ask
//    for no more: the size returned for them is part of the interface (the ABI
//    tests hold it), so they are split no finer, however idle the device: 4
//    units of 1536 rows are 8 blocks, 4 of 1537 rows 52.
//  * chunks of kMinWaveRows rows per wave where max_count rows in every unit
//    make at most one round of them;
//  * else a balanced plan: at most one chunk per unit more than its rows
//    divided by the chunk, and room in its grid for fixed chunks.
struct DecodeGrid {
    int plan;  // groups of query heads of a balanced plan, 0: fixed chunks
    int np;    // fixed chunks per unit at most
    int64_t blocks;
    size_t bytes;
};

inline DecodeGrid decode_grid(int64_t units, int G, int D, int max_count, bool least)
{
    DecodeGrid g{};
    const size_t part = sizeof(float) * (size_t)G * (size_t)(D + 2);
    const int zg = decode_head_groups(G);
    constexpr int kSmall = kDecWaves * kMinWaveRows;
    const int coarse = (max_count + kDecChunk - 1) / kDecChunk, fine = (max_count + kSmall - 1) / kSmall;
    const bool few = units * fine * zg <= kOneRound;
    least = least || coarse <= 2;
    g.np = !least && few ? fine : coarse;
    g.blocks = units * g.np;
    g.bytes = part * (size_t)g.blocks;
    if (least || few || units > kPlanUnits) return g;
    // (blocks past the last chunk read the counts and end: with eight groups of
    // query heads, 4352 blocks for the 768 that 32 units of 2048 rows need took
    // 47 us where 944 take 40)
    const int64_t fixed = (units * max_count + kDecChunk - 1) / kDecChunk, rounds = (2 * kOneRound + zg - 1) / zg;
    g.plan = zg;
    g.blocks = units + (fixed > rounds ? fixed : rounds);
    g.bytes = part * (size_t)g.blocks + 2 * sizeof(int) * (size_t)units;  // and the units' (first block, blocks)
    return g;
}

// The launch of a grid of `blocks` chunks with zg groups of query heads each.
// Consecutive blocks of a launch go to the eight XCDs in turn: the groups of a
// chunk are eight apart, so that the L2 of one XCD reads its rows (us, the
// groups in a grid dimension of their own -> so, 128-wide bf16 rows: 16 units
// of 20000 rows, 16 query heads 54 -> 44; 32 of 2048, 64 query heads 40 -> 33).
struct DecodePlace {
    int block, z;
};
inline int64_t decode_places(int64_t blocks, int zg) { return zg > 1 ? (blocks + 7) / 8 * 8 * zg : blocks; }
__host__ __device__ inline DecodePlace decode_place(int index, int zg)
{
    const int e = index / (8 * zg), r = index - e * 8 * zg;
    return DecodePlace{8 * e + (r & 7), r >> 3};  // (blocks past the last chunk among them)
}

}  // namespace ecokv
