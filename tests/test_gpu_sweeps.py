"""The sweeps over K of every dtype, head_dim and number of window rows, at the
edges of their tiles: 16-key tiles and 16-row window tiles, batches of 16 to
64 keys, blocks of 128 to 2048.

  sums    ecokv_prefill_write's key sums against float64.  A sum over T keys
          is at most 32 + 4 + 4 additions per lane, wave and block and
          T / 128 / 16 + 4 over the blocks, each rounding by 2^-24 of at most
          the column's absolute mass: 2^-24 (44 + T / 2048) of it; the sum of
          k / |k| adds a few roundings per term (|k|^2 over D / 4 + 2 terms,
          halved by the square root, and the bf16 streaming form's 1 / |k| in
          two bf16 parts, 2^-17): 2^-16 of the mass in all.
  lse     the window rows' log-sum-exp against float64: a logit is a sum of D
          products, each of its roundings at most 2^-24 of |q| |k| / sqrt(D).
  scores  the whole call against the oracle (parity_utils' tolerances).
"""
import math
import sys

import pytest
import torch

import oracle
import workloads as W
from parity_utils import gpu_pass
from test_gpu_parity import check_per_head

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_06663_amd  # noqa: F401  (fails loudly if the library is not built)
    oracle.build(force=False)


def say(msg):
    print(f"[gpu-sweeps] {msg}", file=sys.stderr, flush=True)


def make(dtype, L, Hkv, G, D, w, lens, seed=0, offset_elems=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    cu = [0]
    for t in lens:
        cu.append(cu[-1] + t)
    k = torch.randn(L, Hkv, cu[-1], D, generator=g, device="cuda") + torch.randn(L, Hkv, 1, D, generator=g, device="cuda")
    q = torch.randn(L, Hkv * G, len(lens), w, D, generator=g, device="cuda")
    out = []
    for x in (k, q):
        buf = torch.empty(x.numel() + offset_elems, dtype=dtype, device="cuda")
        v = buf[offset_elems:].view(x.shape)
        v.copy_(x)
        out.append(v)
    return cu, out[0], out[1]


def scores(shape, K, Q):
    import paper_2609_06663_amd as P
    S = torch.full((shape.score_numel(),), math.nan, device="cuda")
    lam = torch.full((shape.units,), math.nan, device="cuda")
    st = torch.full((shape.units, P.NSTATS), math.nan, device="cuda")
    P.ecokv_score(K, Q, shape, P.Params(), S, lam, st)
    torch.cuda.synchronize()
    return S, lam, st


@pytest.mark.parametrize("dtype,D", [("f32", 128), ("f32", 64), ("bf16", 128), ("bf16", 64)])
@pytest.mark.parametrize("G,w", [(1, 1), (4, 4), (1, 17), (8, 4), (3, 11), (8, 8)])
@pytest.mark.parametrize("lens", [[18, 33, 128], [129, 255, 257, 1027]])
def test_sums_and_scores_at_tile_edges(dtype, D, G, w, lens):
    import paper_2609_06663_amd as P
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    L, Hkv, R = 1, 2, G * w
    say(f"{dtype} D={D} R={R} T={lens}: sums")
    cu, K, Q = make(tdt, L, Hkv, G, D, w, lens, seed=R)
    shape = P.Shape(L, G * Hkv, Hkv, D, w, cu)
    Kc = torch.zeros_like(K)
    pre = torch.full((shape.units, 2 * D + 2 * R), math.nan, device="cuda")
    P.ecokv_prefill_write(K.transpose(1, 2).contiguous(), None, Q, shape, P.Params(), Kc, None, pre)
    assert torch.equal(Kc, K)
    for h in range(Hkv):
        for s, T in enumerate(lens):
            p = pre[h * len(lens) + s].double()
            k = K[0, h, cu[s]:cu[s + 1]].double()
            kh = k / k.norm(dim=1, keepdim=True)
            u = 2.0 ** -24
            assert ((p[:D] - k.sum(0)).abs() <= u * (44 + T / 2048) * k.abs().sum(0)).all(), (h, s)
            assert ((p[D:2 * D] - kh.sum(0)).abs() <= 2.0 ** -16 * kh.abs().sum(0)).all(), (h, s)
            q = Q[0, h * G:(h + 1) * G, s].reshape(R, D).double()
            x = q @ k.t() / math.sqrt(D)
            j = torch.arange(R, device="cuda") % w
            x.masked_fill_(torch.arange(T, device="cuda")[None] > (T - w + j)[:, None], -math.inf)
            tol = 2 * u * D * (q.norm(dim=1) * k.norm(dim=1).max()) / math.sqrt(D) + 16 * u
            err = (p[2 * D:2 * D + R] + p[2 * D + R:].log() - x.logsumexp(1)).abs()
            assert (err <= tol).all(), (h, s, float((err / tol).max()))
    say("  scores")
    wl = W.custom(7 + R, L=1, Hq=G * Hkv, Hkv=Hkv, D=D, w=w, seqlens=lens, dtype=dtype,
                  budget=[max(w, t // 4) for t in lens], group=16)
    check_per_head(wl, gpu_pass(wl))


@pytest.mark.parametrize("dtype,D,T", [("f32", 64, 4100), ("f32", 128, 4100), ("bf16", 64, 8200), ("bf16", 128, 8200)])
def test_longest_blocks(dtype, D, T):
    # 64 units: enough keys for the longest blocks (1024 fp32 keys, 2048 bf16),
    # the last of each unit nearly empty; w 8 and G 5, 40 window rows
    wl = W.custom(31, L=8, Hq=40, Hkv=8, D=D, w=8, seqlens=[T], dtype=dtype, budget=[T // 5], group=256)
    say(f"{dtype} D={D} T={T}: longest blocks")
    check_per_head(wl, gpu_pass(wl))


@pytest.mark.parametrize("D", [64, 128])
def test_keys_at_any_element(D):
    # a view at an odd element: the same scores, bit for bit
    import paper_2609_06663_amd as P
    say(f"D={D}: keys and queries at 2-byte alignment")
    lens = [700, 90]
    cu, K, Q = make(torch.bfloat16, 2, 2, 4, D, 4, lens, seed=5)
    cu, K1, Q1 = make(torch.bfloat16, 2, 2, 4, D, 4, lens, seed=5, offset_elems=1)
    assert K1.data_ptr() % 4 == 2 and torch.equal(K, K1)
    shape = P.Shape(2, 8, 2, D, 4, cu)
    for a, b in zip(scores(shape, K, Q), scores(shape, K1, Q1)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64)])
def test_attention_below_the_least_normal(dtype, D):
    # keys whose attention falls by half from one to the next, past 2^-126 (the
    # least normal float) to 2^-149 (the least of all).  With lambda 0 and no
    # pooling the score is the attention itself.  The base-2 logits, up to 150,
    # round by 2^-24 of themselves a few times (1e-4 of the weight at most); a
    # subnormal weight rounds to multiples of 2^-149 a few times on its way
    import paper_2609_06663_amd as P
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    T, step = 240, 0.69921875
    say(f"{dtype} D={D}: subnormal attention")
    t = -torch.arange(T, dtype=torch.float64)
    K = torch.zeros(1, 1, T, D, dtype=torch.float64)
    K[..., 0], K[..., 1] = t, 1.0
    Q = torch.zeros(1, 1, 1, 1, D, dtype=torch.float64)
    Q[..., 0] = step * math.sqrt(D)  # (bf16, 64 dimensions: 5.59375, exact)
    shape = P.Shape(1, 1, 1, D, 1, [0, T])
    S = torch.full((T - 1,), math.nan, device="cuda")
    P.ecokv_score(K.to(tdt).cuda(), Q.to(tdt).cuda(), shape, P.Params(lambda_override=0.0, pool_kernel=1), S)
    x = step * t
    ref = (x - x.logsumexp(0)).exp()[:T - 1].numpy()
    err = abs(S.cpu().numpy().astype("f8") - ref)
    assert (err <= 1e-4 * ref + 4 * 2.0 ** -149).all(), int((err / (1e-4 * ref + 4 * 2.0 ** -149)).argmax())


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64)])
def test_lengths_are_rounded_not_approximated(dtype, D):
    # Keys of components 1, a, b, whose squared length is exact in fp32.
    #  * Two equal keys: their sum of k / |k| at the component 1 is 2 / |k|.  Its
    #    error is that of a square root and a quotient (2^-24 of the value each at
    #    most) and evens out over the lengths: 4096 errors of 0.5 x 2^-24 leave a
    #    mean of 0.008, 0.05 is six times that.
    #  * k, -k and a window key of 0: their centroid is 0 and d_E = |k|, the
    #    rounded square root (a last Newton step may miss it by a hair).
    import numpy as np
    import paper_2609_06663_amd as P
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    L, Hkv, G, B = 4, 16, 4, 64
    U = L * Hkv * B
    rng = np.random.default_rng(5)
    ab = rng.integers(1, 256, size=(U, 2)) / 128.0
    length = np.sqrt(1.0 + (ab ** 2).sum(1))
    k = np.zeros((U, D))
    k[:, 7], k[:, 20], k[:, D - 1] = 1.0, ab[:, 0], ab[:, 1]
    Q = torch.zeros(L, Hkv * G, B, 1, D, dtype=tdt, device="cuda")
    say(f"{dtype} D={D}: 1 / |k| and |k|")

    def keys(*rows):
        return torch.from_numpy(np.ascontiguousarray(np.stack(rows, 1).reshape(L, Hkv, len(rows) * B, D))).to(tdt).cuda()

    K = keys(k, k)
    shape = P.Shape(L, Hkv * G, Hkv, D, 1, [2 * s for s in range(B + 1)])
    pre = torch.full((U, 2 * D + 2 * G), math.nan, device="cuda")
    P.ecokv_prefill_write(K.transpose(1, 2).contiguous(), None, Q, shape, P.Params(), torch.zeros_like(K), None, pre)
    err = (pre[:, D + 7].double().cpu().numpy() / 2 * length - 1) * 2.0 ** 24
    assert abs(err).max() <= 2 and abs(err.mean()) <= 0.05, (abs(err).max(), err.mean())
    shape = P.Shape(L, Hkv * G, Hkv, D, 1, [3 * s for s in range(B + 1)])
    S = torch.full((shape.score_numel(),), math.nan, device="cuda")
    st = torch.full((U, P.NSTATS), math.nan, device="cuda")
    P.ecokv_score(keys(k, -k, 0 * k), Q, shape, P.Params(), S, None, st)
    d = st[:, [P.STAT["dmin"], P.STAT["dmax"]]].double().cpu().numpy()
    ulp = np.spacing(length.astype(np.float32)).astype(np.float64)
    off = abs(d - length[:, None]) / ulp[:, None]
    assert off.max() <= 0.501, off.max()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [7, 28, 56])
def test_fp32_logits_round_no_oftener_than_a_tree(D, G):
    # Keys k and -k: a window row's largest logit, the reference that the cache
    # write hands over, is |q.k| / sqrt(D).  Its error against float64 beside that
    # of 16 runs of D / 16 products added by a tree in numpy's float32, then the
    # scale (base 2) and back: as large, but for the order of the dimensions
    import numpy as np
    import paper_2609_06663_amd as P
    Hkv, B = 8, 64
    f32 = lambda v: v.astype(np.float32).astype("f8")  # (a fused product and sum, rounded once)
    rng = np.random.default_rng(G + D)
    k = (6 * rng.standard_normal((Hkv, B, D))).astype(np.float32)
    q = rng.standard_normal((Hkv, G, B, D)).astype(np.float32)
    shape = P.Shape(1, Hkv * G, Hkv, D, 1, [2 * s for s in range(B + 1)])
    K = torch.from_numpy(np.ascontiguousarray(np.stack([k, -k], 2).reshape(1, Hkv, 2 * B, D))).cuda()
    pre = torch.full((Hkv, B, 2 * D + 2 * G), math.nan, device="cuda")
    P.ecokv_prefill_write(K.transpose(1, 2).contiguous(), None, torch.from_numpy(q).cuda(), shape, P.Params(),
                          torch.zeros_like(K), None, pre)
    got = pre[..., 2 * D:2 * D + G].cpu().numpy().astype("f8").transpose(0, 2, 1).ravel()
    p = k.astype("f8")[:, None] * q.astype("f8")
    x = np.abs(p.sum(-1) / np.sqrt(D)).ravel()
    t = p.reshape(-1, 16, D // 16)
    s = f32(t[..., 0])
    for j in range(1, D // 16):
        s = f32(t[..., j] + s)
    while s.shape[1] > 1:
        s = f32(s[:, 0::2] + s[:, 1::2])
    scale = np.float32(1 / np.sqrt(np.float32(D))) * np.float32(1.4426950408889634)
    s = f32(f32(np.abs(s[:, 0]) * float(scale)) * float(np.float32(1 / np.float32(1.4426950408889634))))
    rms, tree = (float(np.sqrt((e ** 2).mean())) for e in (got - x, s - x))
    say(f"fp32 D={D} R={G}: logit error {rms:.3e}, tree {tree:.3e}")
    assert rms <= (1 + 0.2 / np.sqrt(G)) * tree, (rms, tree)  # (512 G errors: 3 % / sqrt(G) each; four deviations)
