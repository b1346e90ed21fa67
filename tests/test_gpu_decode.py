"""GPU parity of ecokv_decode (attention of one new query per head over the
compressed cache, Sec. 3) against the oracle on seeded synthetic caches:
packed Kc / Vc rows with ragged per-unit counts, as ecokv_select and
ecokv_compact lay them out.

Tolerance (fp32 accumulation of bf16 / fp32 inputs against fp64):
|O_g - O_o| <= 1e-4 * max |Vc| over the unit's rows, |lse_g - lse_o| <= 1e-4 * max(1, |lse_o|).
"""
import sys

import numpy as np
import pytest
import torch

import oracle
from parity_utils import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_06663_amd  # noqa: F401  (fails loudly if the library is not built)
    oracle.build(force=False)


def say(msg):
    print(f"[gpu-decode] {msg}", file=sys.stderr, flush=True)


def make_cache(seed, L, Hq, Hkv, B, D, counts, dtype, kscale=1.0):
    r = np.random.default_rng(seed)
    counts = np.asarray(counts, np.int32).reshape(L, Hkv, B)
    offsets = np.concatenate([[0], np.cumsum(counts.reshape(-1))[:-1]]).reshape(L, Hkv, B).astype(np.int32)
    n = int(counts.sum())

    def arr(shape, scale):
        x = (r.standard_normal(shape) * scale).astype(np.float32)
        if dtype == "bf16":
            return (x.view(np.uint32) >> 16).astype(np.uint16)  # truncation: any bf16 values will do
        return x

    return dict(Q=arr((L, Hq, B, D), 1.0), Kc=arr((n, D), kscale), Vc=arr((n, D), 1.0), counts=counts,
                offsets=offsets)


def run(c, L, Hq, Hkv, B, D, dtype, max_count=None):
    import paper_2609_06663_amd as P
    shape = P.Shape(L, Hq, Hkv, D, 1, [0] + list(np.cumsum([2] * B)))
    mc = int(c["counts"].max()) if max_count is None else max_count
    O = torch.full((L, Hq, B, D), -7.0, device="cuda")
    lse = torch.full((L, Hq, B), -7.0, device="cuda")
    P.ecokv_decode(dev(c["Q"], dtype), dev(c["Kc"], dtype), dev(c["Vc"], dtype), shape,
                   torch.from_numpy(c["counts"].reshape(-1)).cuda(), torch.from_numpy(c["offsets"].reshape(-1)).cuda(),
                   mc, O, lse)
    torch.cuda.synchronize()
    return O.cpu().numpy(), lse.cpu().numpy()


def check(c, O, lse, L, Hq, Hkv, B, D, dtype):
    Oo, lo = oracle.decode(c["Q"], c["Kc"], c["Vc"], L, Hq, Hkv, B, D, c["counts"], c["offsets"])
    G = Hq // Hkv
    V = c["Vc"].astype(np.float32) if dtype == "f32" else (c["Vc"].astype(np.uint32) << 16).view(np.float32)
    for l in range(L):
        for q in range(Hq):
            for s in range(B):
                o, n = c["offsets"][l, q // G, s], c["counts"][l, q // G, s]
                vmax = float(np.abs(V[o:o + n]).max())
                err = np.abs(O[l, q, s] - Oo[l, q, s]).max()
                assert err <= 1e-4 * vmax, f"O (l={l}, q={q}, s={s}, n={n}): error {err:.3e}, max|V| {vmax:.3e}"
                assert abs(lse[l, q, s] - lo[l, q, s]) <= 1e-4 * max(1.0, abs(lo[l, q, s])), (l, q, s)


@pytest.mark.parametrize("dtype,D,Hq,Hkv", [("bf16", 128, 28, 4), ("bf16", 64, 8, 8), ("f32", 128, 8, 4),
                                            ("f32", 64, 12, 4), ("bf16", 128, 32, 2), ("bf16", 128, 24, 2)])
def test_decode_ragged(dtype, D, Hq, Hkv):
    # G = 7, 1, 2, 3, 16 (two blocks of 8 query heads), 12 (8 + 4); counts from
    # one row to a few chunks
    L, B = 2, 3
    r = np.random.default_rng(100 + Hq)
    counts = r.integers(1, 2600, size=(L, Hkv, B))
    counts.reshape(-1)[0] = 1                     # one row
    counts.reshape(-1)[-1] = 1024                 # whole tiles
    if counts.size > 2:
        counts.reshape(-1)[1] = 257               # one row past whole tiles
    c = make_cache(7, L, Hq, Hkv, B, D, counts, dtype, kscale=2.0)
    say(f"{dtype} D={D} Hq={Hq} Hkv={Hkv}: ragged counts up to {int(counts.max())}")
    O, lse = run(c, L, Hq, Hkv, B, D, dtype)
    check(c, O, lse, L, Hq, Hkv, B, D, dtype)


def test_decode_large_logits_and_a_loose_max_count():
    # keys scaled up: logits span hundreds, the online maxima move often; a
    # max_count far above every count only adds empty chunks
    L, Hq, Hkv, B, D = 1, 8, 2, 2, 128
    counts = [[[3000, 77], [1, 2049]]]
    c = make_cache(8, L, Hq, Hkv, B, D, counts, "bf16", kscale=30.0)
    say("large logits, max_count 9000")
    O, lse = run(c, L, Hq, Hkv, B, D, "bf16", max_count=9000)
    check(c, O, lse, L, Hq, Hkv, B, D, "bf16")


def test_decode_count_above_max_count_is_nan():
    L, Hq, Hkv, B, D = 1, 4, 2, 1, 64
    c = make_cache(9, L, Hq, Hkv, B, D, [[[100], [300]]], "f32")
    say("a unit with more rows than max_count")
    O, lse = run(c, L, Hq, Hkv, B, D, "f32", max_count=200)
    assert np.isnan(O[0, 2:]).all() and np.isnan(lse[0, 2:]).all()   # KV head 1's query heads
    Oo, lo = oracle.decode(c["Q"], c["Kc"], c["Vc"], L, Hq, Hkv, B, D, c["counts"], c["offsets"])
    np.testing.assert_allclose(O[0, :2], Oo[0, :2], atol=1e-4 * np.abs(c["Vc"][:100]).max())


def test_decode_stack28_sized_cache():
    # the compressed cache of the 28-layer benchmark stack at 20 %: 6553 rows per head
    L, Hq, Hkv, B, D = 28, 28, 4, 1, 128
    counts = np.full((L, Hkv, B), 6553)
    c = make_cache(10, L, Hq, Hkv, B, D, counts, "bf16")
    say("28 layers x 4 KV heads x 6553 rows, 28 query heads")
    O, lse = run(c, L, Hq, Hkv, B, D, "bf16")
    check(c, O, lse, L, Hq, Hkv, B, D, "bf16")


def test_decode_many_units_ragged():
    # 224 units of up to 6000 rows (more blocks than the device holds at once);
    # the counts are ragged, so chunks and 16-row tiles end inside and past units
    L, Hq, Hkv, B, D = 28, 28, 4, 2, 128
    r = np.random.default_rng(11)
    counts = r.integers(1, 6000, size=(L, Hkv, B))
    counts.reshape(-1)[3] = 6000
    counts.reshape(-1)[4] = 1
    counts.reshape(-1)[7] = 16
    counts.reshape(-1)[8] = 17
    c = make_cache(12, L, Hq, Hkv, B, D, counts, "bf16")
    say(f"224 units, ragged counts up to 6000, {int(counts.sum())} rows")
    O, lse = run(c, L, Hq, Hkv, B, D, "bf16", max_count=6000)
    check(c, O, lse, L, Hq, Hkv, B, D, "bf16")


# The last entry is the split that the call takes with its full workspace: fixed
# chunks, or a balanced plan of so many rows per wave (test_decode_plan.py
# checks these).
PLAN_CASES = [
    # fixed chunks of 32 rows per wave (few units), their edges and one row past
    ("bf16", 128, 28, 4, 1, [128, 129, 6553, 2049], 6553, "fixed"),
    ("f32", 128, 14, 2, 1, [1, 4097], 4097, "fixed"),
    # the balanced plan: one round, two rounds, past two (fixed chunks again); units without rows
    ("bf16", 128, 28, 4, 4, [4000, 1, 0, 9000, 127, 128, 129, 2500, 16, 17, 640, 1536, 768, 769, 3000, 5], 9000, "balanced 32"),
    ("f32", 64, 32, 16, 4, list(range(60, 60 + 64 * 113, 113)), 9001, "balanced 128"),
    ("bf16", 64, 8, 8, 8, [6144 + 31 * i for i in range(64)], 12000, "balanced 192"),
    ("bf16", 64, 8, 8, 8, [12000 - i for i in range(64)], 12000, "fixed"),
    # two groups of query heads in fixed chunks; one unit more than a plan takes
    ("bf16", 64, 48, 4, 1, [3000, 20, 900, 1700], 3000, "fixed"),
    ("f32", 64, 257, 257, 1, [1600 + i % 7 for i in range(257)], 1606, "fixed"),
    # balanced plans whose chunks take two, three and eight groups of query heads
    ("f32", 64, 32, 2, 2, [6553, 1, 7000, 6000], 7000, "balanced 48"),
    ("bf16", 64, 64, 4, 4, [19660 - 700 * i for i in range(16)], 19660, "balanced 192"),
    ("bf16", 128, 96, 4, 1, [19660, 19001, 19659, 3], 19660, "balanced 96"),
    ("bf16", 64, 64, 1, 1, [60000], 90000, "balanced 192"),
    # units that do not fill the last lane's four
    ("bf16", 64, 10, 5, 3, [4000 - 211 * i for i in range(15)], 4000, "balanced 48"),
    ("f32", 64, 1, 1, 1, [40000], 40000, "balanced 48"),
    # the same rows in units nearly all full: fixed chunks
    ("bf16", 64, 64, 4, 4, [15000 - 7 * i for i in range(16)], 15000, "fixed"),
    ("f32", 128, 64, 64, 4, [1600 - i % 5 for i in range(256)], 1600, "fixed"),
]


@pytest.mark.parametrize("dtype,D,Hq,Hkv,B,counts,max_count", [c[:7] for c in PLAN_CASES])
def test_decode_plans(dtype, D, Hq, Hkv, B, counts, max_count):
    """The same outputs however the rows are split: with the workspace that the
    call asks for and with the least it takes.  Both are sums of the same
    products, each row's weight rounded a few times: 2e-6 of max |Vc| apart at most."""
    import ctypes
    import paper_2609_06663_amd as P
    from paper_2609_06663_amd import ecokv as E
    say(f"{dtype} D={D} Hq={Hq} Hkv={Hkv} B={B}: {len(counts)} units of up to {max(counts)} rows, max_count {max_count}")
    c = make_cache(14, 1, Hq, Hkv, B, D, counts, dtype, kscale=1.5)
    shape = P.Shape(1, Hq, Hkv, D, 1, [0] + list(np.cumsum([2] * B)))
    Q, Kc, Vc = dev(c["Q"], dtype), dev(c["Kc"], dtype), dev(c["Vc"], dtype)
    # (what follows the counts and offsets in memory is not read as theirs)
    n, off = (torch.full((len(counts) + 8,), 9999, dtype=torch.int32, device="cuda")[:len(counts)] for _ in range(2))
    n.copy_(torch.from_numpy(c["counts"].reshape(-1)))
    off.copy_(torch.from_numpy(c["offsets"].reshape(-1)))
    full = P.ecokv_decode_workspace_size(shape, max_count)
    least = 4 * Hq * B * ((max_count + 767) // 768) * (D + 2)
    assert full >= least
    outs = []
    for size in (full, least):
        O = torch.full((1, Hq, B, D), -7.0, device="cuda")
        lse = torch.full((1, Hq, B), -7.0, device="cuda")
        ws = torch.full((max(size, 256),), 0xAB, dtype=torch.uint8, device="cuda")  # no initial contents needed
        p = lambda t: ctypes.c_void_p(t.data_ptr())
        rc = E.lib.ecokv_decode(p(Q), p(Kc), p(Vc), 0 if dtype == "bf16" else 1, ctypes.byref(shape.c), p(n), p(off),
                                max_count, p(O), p(lse), p(ws), size, None)
        assert rc == 0
        torch.cuda.synchronize()
        outs.append((O.cpu().numpy(), lse.cpu().numpy()))
    assert E.lib.ecokv_decode(p(Q), p(Kc), p(Vc), 0 if dtype == "bf16" else 1, ctypes.byref(shape.c), p(n), p(off),
                              max_count, p(O), p(lse), p(ws), least - 1, None) == -2
    V = np.abs(c["Vc"].astype(np.float32) if dtype == "f32" else (c["Vc"].astype(np.uint32) << 16).view(np.float32)).max()
    np.testing.assert_allclose(outs[0][0], outs[1][0], atol=2e-6 * V, rtol=0)
    empty = np.repeat(c["counts"].reshape(Hkv, B), Hq // Hkv, axis=0) == 0  # [Hq][B]
    assert (outs[0][0][0][empty] == 0).all() and np.isneginf(outs[0][1][0][empty]).all()
    keep = ~empty
    np.testing.assert_allclose(outs[0][1][0][keep], outs[1][1][0][keep], atol=1e-5, rtol=1e-6)
    if not empty.any():
        check(c, *outs[0], 1, Hq, Hkv, B, D, dtype)


@pytest.mark.parametrize("units", [256, 257])
def test_decode_loose_max_count_of_many_blocks(units):
    # a bound of 50 million rows: 65 600 chunks per unit, more blocks in all
    # (16.8 million) than one grid dimension of 2^32 threads holds.  One long
    # unit, whose fixed chunks reach past the blocks that such a dimension
    # wraps round to (256 units would take a balanced plan for fewer rows)
    L, D, max_count = 1, 64, 768 * 65600
    counts = [1 + i % 9 for i in range(units)]
    counts[units // 2] = 600_000
    c = make_cache(21, L, units, units, 1, D, counts, "bf16")
    say(f"{units} units, max_count {max_count}")
    O, lse = run(c, L, units, units, 1, D, "bf16", max_count=max_count)
    check(c, O, lse, L, units, units, 1, D, "bf16")


def test_decode_many_query_rows():
    # 16.8 million query rows: more blocks of the merge than one grid dimension
    # holds.  Every unit reads the same row, whose V is then every output
    import paper_2609_06663_amd as P
    L, Hq, Hkv, B, D = 4097, 64, 1, 64, 64
    say(f"{L * Hq * B} query rows")
    shape = P.Shape(L, Hq, Hkv, D, 1, [2 * s for s in range(B + 1)])
    Q = torch.zeros(L, Hq, B, D, dtype=torch.bfloat16, device="cuda")
    Kc, Vc = (torch.arange(D, dtype=torch.bfloat16, device="cuda").view(1, D) + x for x in (1, 2))
    n = torch.ones(shape.units, dtype=torch.int32, device="cuda")
    O = torch.full((L, Hq, B, D), -7.0, device="cuda")
    lse = torch.full((L, Hq, B), -7.0, device="cuda")
    P.ecokv_decode(Q, Kc, Vc, shape, n, torch.zeros_like(n), 1, O, lse)
    assert bool((O == Vc[0].float()).all()) and bool((lse == 0).all())


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("where", ["one tile", "everywhere"])
def test_decode_rows_of_weight_zero(dtype, D, where):
    # rows whose logit is -inf, wherever a wave or a chunk may begin: whole tiles,
    # the first rows of every 32, whole chunks; the others' attention as if they
    # were not there
    import paper_2609_06663_amd as P
    Hq, Hkv = 28, 4
    counts = [6553, 40, 1700, 3000]
    c = make_cache(23, 1, Hq, Hkv, 1, D, counts, dtype)
    Q, Kc, Vc = dev(c["Q"], dtype), dev(c["Kc"], dtype), dev(c["Vc"], dtype)
    off = c["offsets"].reshape(-1)
    dead = torch.zeros(len(Kc), dtype=torch.bool, device="cuda")
    dead[off[0] + 32:off[0] + 48] = True
    if where == "everywhere":
        dead[off[0] + 200:off[0] + 1100] = True
        dead[off[1] + 16:off[1] + 32] = True
        j = torch.arange(counts[2], device="cuda")
        dead[off[2]:off[2] + counts[2]] = (j % 32 < 16) & (j >= 32)
        dead[off[3] + 2900:off[3] + 3000] = True
    Q[..., 0] = 1.0
    Kc[dead, 0] = -float("inf")
    say(f"{dtype} D={D}, {where}: {int(dead.sum())} of {len(Kc)} rows with logit -inf")
    shape = P.Shape(1, Hq, Hkv, D, 1, [0, 2])
    n, o = (torch.from_numpy(c[k].reshape(-1)).cuda() for k in ("counts", "offsets"))
    O = torch.full((1, Hq, 1, D), -7.0, device="cuda")
    lse = torch.full((1, Hq, 1), -7.0, device="cuda")
    P.ecokv_decode(Q, Kc, Vc, shape, n, o, 6553, O, lse)
    for q in range(Hq):
        u = q // (Hq // Hkv)
        rows = slice(off[u], off[u] + counts[u])
        x = (Kc[rows].double().masked_fill(dead[rows, None], 0.0) @ Q[0, q, 0].double()) / D ** 0.5
        x.masked_fill_(dead[rows], -float("inf"))
        ref = x.softmax(0) @ Vc[rows].double()
        assert (O[0, q, 0] - ref).abs().max() <= 1e-4 * Vc[rows].abs().max(), (u, q)
        assert (lse[0, q, 0] - x.logsumexp(0)).abs() <= 1e-4 * max(1.0, float(x.logsumexp(0).abs())), (u, q)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rows", [(0, 128), (40, 41), (0, 6553)])
def test_decode_nan_rows_reach_the_output(dtype, rows):
    # NaN keys in one unit, down to a whole chunk of them: its outputs are NaN
    # however the rows are split, the other units' finite
    import paper_2609_06663_amd as P
    Hq, Hkv, D = 28, 4, 128
    c = make_cache(24, 1, Hq, Hkv, 1, D, [2000, 6553, 40, 3000], dtype)
    Kc = dev(c["Kc"], dtype)
    Kc[2000 + rows[0]:2000 + rows[1], 5] = float("nan")
    say(f"{dtype}: NaN in rows {rows} of unit 1")
    shape = P.Shape(1, Hq, Hkv, D, 1, [0, 2])
    n, o = (torch.from_numpy(c[k].reshape(-1)).cuda() for k in ("counts", "offsets"))
    O = torch.full((1, Hq, 1, D), -7.0, device="cuda")
    lse = torch.full((1, Hq, 1), -7.0, device="cuda")
    P.ecokv_decode(dev(c["Q"], dtype), Kc, dev(c["Vc"], dtype), shape, n, o, 6553, O, lse)
    bad = torch.zeros(Hq, dtype=torch.bool, device="cuda")
    bad[7:14] = True
    assert bool(O[0, bad].isnan().all()) and bool(lse[0, bad].isnan().all())
    assert bool(O[0, ~bad].isfinite().all()) and bool(lse[0, ~bad].isfinite().all())


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 7])
def test_decode_fp32_logits_round_no_oftener_than_a_tree(D, G):
    # Units of one row: lse is the logit.  Its error against float64 beside that
    # of a tree of runs of four products in numpy's float32, then the scale (base
    # 2) and the natural logarithm's constant: as large, but for the order of the
    # dimensions.  Root mean squares of 4096 G errors leave 1.1 % / sqrt(G) each
    Hkv, B = 8, 64
    f32 = lambda v: v.astype(np.float32).astype("f8")  # (a fused product and sum, rounded once)
    err, tree = [], []
    for seed in range(8):
        c = make_cache(seed, 1, Hkv * G, Hkv, B, D, [1] * (Hkv * B), "f32", kscale=6.0)
        _, lse = run(c, 1, Hkv * G, Hkv, B, D, "f32")
        p = c["Kc"].astype("f8").reshape(Hkv, 1, B, D) * c["Q"].astype("f8").reshape(Hkv, G, B, D)
        x = (p.sum(-1) / np.sqrt(D)).ravel()
        t = p.reshape(-1, D // 4, 4)
        t = f32(t[..., 3] + f32(t[..., 2] + f32(t[..., 1] + f32(t[..., 0]))))
        while t.shape[1] > 1:
            t = f32(t[:, 0::2] + t[:, 1::2])
        scale = np.float32(np.float32(1.4426950408889634) / np.sqrt(np.float32(D)))
        t = f32(f32(t[:, 0] * float(scale)) * float(np.float32(0.69314718055994531)))
        err.append(lse.astype("f8").ravel() - x)
        tree.append(t - x)
    rms, bound = (float(np.sqrt((np.concatenate(e) ** 2).mean())) for e in (err, tree))
    say(f"fp32 D={D} G={G}: logit error {rms:.3e}, tree {bound:.3e}")
    assert rms <= (1 + 0.05 / np.sqrt(G)) * bound, (rms, bound)  # (three standard deviations of the ratio)
