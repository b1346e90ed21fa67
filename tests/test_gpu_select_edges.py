"""The one-block and two-stage selections at the edges of their sizes: groups
of one key to a full block's registers and just past it, one key, nearly all
keys or all but one kept, scores on one octave, over many and all the same,
ties that the budget cuts, NaN and infinities.  Whole numbers: bit for bit
against the oracle."""
import sys

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_06663_amd  # noqa: F401  (fails loudly if the library is not built)
    oracle.build(force=False)


def scores(kind, n, rng):
    if kind == "octave":  # one exponent: the first digit spreads it
        return (1.0 + rng.random(n)).astype(np.float32)
    if kind == "wide":  # both signs, many octaves, subnormal numbers, infinities
        s = (np.exp(rng.uniform(-60, 60, n)) * rng.choice([-1.0, 1.0], n)).astype(np.float32)
        i = rng.integers(0, n, max(1, n // 3))
        s[i] = (rng.integers(-9, 10, i.size) * 1e-42).astype(np.float32)
        s[rng.integers(0, n, max(1, n // 50))] = np.inf
        s[rng.integers(0, n, max(1, n // 50))] = -np.inf
        return s
    if kind == "same":
        return np.full(n, 0.75, np.float32)
    if kind == "two":  # neighbours in the last bit
        return np.where(rng.random(n) < 0.5, np.float32(1.5), np.nextafter(np.float32(1.5), np.float32(2))).astype(np.float32)
    s = rng.integers(0, 5, n).astype(np.float32) - 2  # ties, both zeros, NaN
    s[rng.integers(0, n, max(1, n // 10))] = np.nan
    s[rng.integers(0, n, max(1, n // 10))] = -0.0
    return s


@pytest.mark.parametrize("kind", ["octave", "wide", "same", "two", "ties"])
@pytest.mark.parametrize("n", [1, 2, 63, 1025, 8192, 8193, 16384, 16385, 32767, 32768, 32769])
@pytest.mark.parametrize("mode", ["per_head", "layer_flat"])
def test_edges(kind, n, mode):
    import paper_2609_06663_amd as P
    rng = np.random.default_rng(n * 7 + len(kind))
    w, L, Hkv = 2, 1, 2
    flat = mode == "layer_flat"
    S = np.stack([scores(kind, n, rng) for _ in range(Hkv)])[None]
    cu = [0, n + w]
    shape = P.Shape(L, Hkv, Hkv, 128, w, cu)
    ks = sorted({1, n // 5, n // 2, n - 1} - {0, -1})
    for k in [x for x in ks if 0 < x < n] or [0]:
        print(f"[gpu-select] {kind} {mode} n={n} k={k}", file=sys.stderr, flush=True)
        budget = [k + w]
        m = P.ecokv_index_count(shape, budget)
        idx = torch.full((m,), -7, dtype=torch.int32, device="cuda")
        counts = torch.full((L * Hkv,), -7, dtype=torch.int32, device="cuda")
        offsets = torch.full_like(counts, -7)
        P.ecokv_select(torch.from_numpy(S).cuda(), shape, P.LAYER_FLAT if flat else P.PER_HEAD, budget, idx, counts,
                       offsets)
        torch.cuda.synchronize()
        ref = oracle.select(S.astype(np.float64), L, Hkv, cu, w, budget, oracle.LAYER_FLAT if flat else oracle.PER_HEAD)
        for got, want in zip((idx, counts, offsets), ref):
            np.testing.assert_array_equal(got.cpu().numpy(), want.reshape(-1))


@pytest.mark.parametrize("kind", ["octave", "wide", "same", "two", "ties"])
@pytest.mark.parametrize("n", [1023, 1024, 2047, 2048, 2049, 4095, 4096, 4097])
@pytest.mark.parametrize("mode", ["per_head", "layer_flat"])
def test_edges_of_small_groups(kind, n, mode):
    # two and four keys a thread (up to 2048 and 4096 keys of a group), and just past
    test_edges(kind, n, mode)


def test_one_workspace_for_shapes_of_many_sizes():
    # multi-block and two-stage selections of more and fewer groups, longer and
    # shorter, in turn on one workspace sized for the largest
    import paper_2609_06663_amd as P
    rng = np.random.default_rng(77)
    w = 4
    for mode, shapes in ((P.PER_HEAD, [(6, 4, 41000), (1, 2, 33000), (6, 4, 40000), (2, 1, 36000), (3, 4, 41000)]),
                         (P.LAYER_FLAT, [(30, 4, 12000), (1, 4, 9000), (30, 4, 11000), (2, 4, 12000), (7, 4, 8500)])):
        make = lambda L, H, n: P.Shape(L, H, H, 128, w, [0, n + w])
        ws = torch.zeros(max(P.ecokv_select_workspace_size(make(*s), mode) for s in shapes), dtype=torch.uint8,
                         device="cuda")
        for rnd, share in enumerate((0.6, 0.05, 0.6, 0.05)):
            for L, H, n in shapes:
                shape = make(L, H, n)
                S = torch.from_numpy(rng.integers(0, 900, size=(L, H, n)).astype(np.float32)).cuda()
                budget = [int(share * n) + w]
                print(f"[gpu-select] mode {mode}, round {rnd}: {L} x {H} x {n}, {budget[0]} kept", file=sys.stderr, flush=True)
                got = []
                for work in (ws, torch.zeros_like(ws)):  # the shared one, a fresh one
                    idx = torch.full((P.ecokv_index_count(shape, budget),), -7, dtype=torch.int32, device="cuda")
                    counts = torch.full((L * H,), -7, dtype=torch.int32, device="cuda")
                    offsets = torch.full_like(counts, -7)
                    P.ecokv_select(S, shape, mode, budget, idx, counts, offsets, work)
                    got.append((idx, counts, offsets))
                torch.cuda.synchronize()
                assert all(torch.equal(a, b) for a, b in zip(*got))
                if L <= 2:
                    ref = oracle.select(S.cpu().numpy().astype(np.float64), L, H, [0, n + w], w, budget,
                                        oracle.LAYER_FLAT if mode == P.LAYER_FLAT else oracle.PER_HEAD)
                    for a, b in zip(got[0], ref):
                        np.testing.assert_array_equal(a.cpu().numpy(), b.reshape(-1))
