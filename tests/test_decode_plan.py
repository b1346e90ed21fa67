"""The arithmetic that splits ecokv_decode's rows over blocks (CPU): workspace,
grid and kernels evaluate the functions of ecokv_decode_plan.h, compiled here
for the host.  For every number of query heads per KV head, units from one to
past a balanced plan's limit, and uniform, ragged, skewed and empty counts:
every chunk that the counts make has a block in the grid and a place in the
workspace, and the chunks cover each unit's rows once."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from test_gpu_decode import PLAN_CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_06663_amd", "csrc")

SHIM = r"""
#define __host__
#define __device__
#include <vector>
#include "ecokv_decode_plan.h"
using namespace ecokv;
static int chunk_rows(int n, int c, int rows) {  // the rows of chunk c, as the kernel's waves take them
    int got = 0;
    for (int wv = 0; wv < kDecWaves; ++wv) {
        const int row0 = (c * kDecWaves + wv) * rows, left = n - row0;
        got += left < 0 ? 0 : left < rows ? left : rows;
    }
    return got;
}
// out: plan (0 fixed, else 1), rows per wave of a balanced plan, chunks, blocks.  Returns 0, or what is wrong.
extern "C" int plan(long long units, int G, int D, int max_count, const int *counts, int least, float rounding, long long *out) {
    const DecodeGrid g = decode_grid(units, G, D, max_count, least != 0);
    const size_t part = sizeof(float) * G * (D + 2);
    if (g.bytes < part * g.blocks + (g.plan ? 2 * sizeof(int) * units : 0)) return 1;
    float rows = 0.f;
    for (long long u = 0; u < units; ++u) rows += (float)counts[u];
    const int wr = g.plan ? plan_wave_rows(rows * rounding, plan_scale(units, g.plan, max_count)) : 0;
    out[0] = wr > 0;
    out[1] = wr;
    out[2] = 0;
    out[3] = g.blocks;
    for (long long u = 0; u < units; ++u) {
        const int n = counts[u], r = wr > 0 ? wr : fixed_wave_rows(n, g.np), chunks = unit_chunks(n, r);
        if (r < kMinWaveRows || r > kWaveRows || r % 16) return 2;
        long long got = 0;
        for (int c = 0; c < chunks; ++c) got += chunk_rows(n, c, r);
        if (got != n || chunk_rows(n, chunks, r) != 0) return 3;         // every row in one chunk
        if (wr == 0 && chunks > 0 && u + units * (chunks - 1) >= g.blocks) return 4;  // block c * units + u
        out[2] += chunks;
    }
    if (wr > 0 && out[2] > g.blocks) return 5;                           // blocks 0 .. chunks - 1
    // blocks that find no chunk cost a read of the counts each: with every group
    // of query heads no more than two rounds past what the units and fixed chunks need
    const long long zg = decode_head_groups(G), fixed = (units * max_count + kDecChunk - 1) / kDecChunk;
    if (g.plan && g.blocks * zg > (units + fixed) * zg + 2 * kOneRound + zg) return 6;
    if (zg > 1) {  // every (chunk, group of query heads) has one place of the launch
        const long long places = decode_places(g.blocks, (int)zg);
        if (places < g.blocks * zg || places >= (g.blocks + 8) * zg) return 7;
        std::vector<char> seen((g.blocks + 8) * zg, 0);
        for (int i = 0; i < places; ++i) {
            const DecodePlace p = decode_place(i, (int)zg);
            if (p.block < 0 || p.block >= g.blocks + 8 || p.z < 0 || p.z >= zg || seen[p.block * zg + p.z]++) return 8;
        }
        for (long long i = 0; i < g.blocks * zg; ++i)
            if (!seen[i]) return 9;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(SHIM)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "plan.so"),
                           str(d / "plan.cpp")])
    f = ctypes.CDLL(str(d / "plan.so")).plan
    f.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_int,
                  ctypes.c_float, ctypes.c_void_p]

    def call(G, D, max_count, counts, least=False, rounding=1.0):
        c = np.ascontiguousarray(counts, np.int32)
        out = np.zeros(4, np.int64)
        rc = f(len(c), G, D, max_count, c.ctypes.data, int(least), rounding, out.ctypes.data)
        return rc, out

    return call


def patterns(rng, units, mc):
    yield np.full(units, mc)
    yield np.ones(units)
    yield rng.integers(0, mc + 1, units)
    yield np.where(np.arange(units) == rng.integers(units), mc, rng.integers(0, 3, units))  # one long unit
    yield np.where(rng.random(units) < 0.5, 0, mc)
    yield np.minimum(mc, (128 * 2.0 ** rng.integers(0, 9, units) + rng.integers(-1, 2, units)))
    yield np.zeros(units)


@pytest.mark.parametrize("G", range(1, 65))
def test_every_chunk_has_a_block(plan, G):
    rng = np.random.default_rng(G)
    for units in (1, 2, 3, 4, 8, 16, 31, 48, 64, 112, 200, 255, 256, 257):
        for mc in (1, 128, 768, 1536, 1537, 2304, 3276, 6553, 9001, 19660, 32768, 65536):
            for k, counts in enumerate(patterns(rng, units, mc)):
                for least in (False, True):
                    # (the sum of the rows is a float: a few roundings either way)
                    for rounding in (1.0, 1.0 + 2.0 ** -16, 1.0 - 2.0 ** -16):
                        rc, out = plan(G, 128, mc, counts, least, rounding)
                        assert rc == 0, (rc, G, units, mc, k, least, rounding, out.tolist())


@pytest.mark.parametrize("case", PLAN_CASES, ids=lambda c: f"{c[0]}-D{c[1]}-Hq{c[2]}-Hkv{c[3]}-B{c[4]}-{c[6]}")
def test_the_gpu_cases_take_the_split_they_name(plan, case):
    dtype, D, Hq, Hkv, B, counts, max_count, split = case
    assert len(counts) == Hkv * B and max(counts) <= max_count
    rc, out = plan(Hq // Hkv, D, max_count, counts)
    assert rc == 0
    assert (f"balanced {out[1]}" if out[0] else "fixed") == split
