"""The binding's checks with GPU tensors of the wrong type or size (refused
before any launch), and the workspace status after a bounded wait that the
host makes give up at once (every kernel still ends normally)."""
import sys

import numpy as np
import pytest
import torch

import workloads as W
from parity_utils import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_06663_amd  # noqa: F401  (fails loudly if the library is not built)


def say(msg):
    print(f"[gpu-binding] {msg}", file=sys.stderr, flush=True)


def test_wrong_types_and_sizes_are_refused():
    import paper_2609_06663_amd as P
    say("binding checks: wrong element types and short buffers")
    s = P.Shape(2, 8, 2, 128, 4, [0, 300])
    K = torch.zeros(2 * 2 * 300 * 128, dtype=torch.bfloat16, device="cuda")
    Q = torch.zeros(2 * 8 * 4 * 128, dtype=torch.bfloat16, device="cuda")
    S = torch.zeros(2 * 2 * 296, dtype=torch.float32, device="cuda")
    with pytest.raises(ValueError, match="K has"):
        P.ecokv_score(K[:-1], Q, s, None, S)
    with pytest.raises(ValueError, match="Q_win has"):
        P.ecokv_score(K, Q[:-128], s, None, S)
    with pytest.raises(ValueError, match="scores has"):
        P.ecokv_score(K, Q, s, None, S[:-1])
    with pytest.raises(TypeError, match="scores must be float32"):
        P.ecokv_score(K, Q, s, None, S.to(torch.bfloat16))
    with pytest.raises(ValueError, match="workspace has"):
        P.ecokv_score(K, Q, s, None, S, workspace=torch.zeros(1024, dtype=torch.uint8, device="cuda"))
    n = P.ecokv_index_count(s, [40])
    idx = torch.zeros(n, dtype=torch.int32, device="cuda")
    with pytest.raises(ValueError, match="idx has"):
        P.ecokv_select(S, s, P.PER_HEAD, [40], idx[:-1])
    with pytest.raises(TypeError, match="idx must be int32"):
        P.ecokv_select(S, s, P.PER_HEAD, [40], idx.to(torch.int64))
    with pytest.raises(ValueError, match="counts is required"):
        P.ecokv_select(S, s, P.LAYER_FLAT, [40], idx)
    Kc = torch.zeros(n * 128, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ValueError, match="Vc has"):
        P.ecokv_compact(K, K, s, P.PER_HEAD, [40], idx, None, None, Kc, Kc[:-1])
    torch.cuda.synchronize()


@pytest.mark.parametrize("held_units,units,max_count", [(6, 6, 2400), (257, 256, 2304)])
def test_decode_with_a_workspace_of_its_least_size(held_units, units, max_count):
    # the header's least: one chunk for every 768 rows of max_count.  A caller
    # may hold such a workspace, or one sized for a shape with more units (256
    # units ask for more than 257 do); one byte less is refused
    import paper_2609_06663_amd as P
    D, G = 64, 2
    say(f"decode of {units} units, max_count {max_count}, in a workspace for {held_units}")
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    rows = 900
    Kc, Vc = (torch.randn(rows, D, generator=g, device="cuda", dtype=torch.float32) for _ in range(2))
    Q = torch.randn(1, G * units, 1, D, generator=g, device="cuda", dtype=torch.float32)
    n = torch.full((units,), rows, dtype=torch.int32, device="cuda")  # every unit the same rows
    off = torch.zeros(units, dtype=torch.int32, device="cuda")
    shape = P.Shape(1, G * units, units, D, 1, [0, 2])
    held = P.Shape(1, G * held_units, held_units, D, 1, [0, 2])
    least = 4 * G * units * ((max_count + 767) // 768) * (D + 2)
    size = least if held_units == units else P.ecokv_decode_workspace_size(held, max_count)
    assert least <= size < P.ecokv_decode_workspace_size(shape, max_count)
    O = torch.full((1, G * units, 1, D), -7.0, device="cuda")
    P.ecokv_decode(Q, Kc, Vc, shape, n, off, max_count, O, workspace=torch.zeros(size, dtype=torch.uint8, device="cuda"))
    ref = torch.softmax(Q[0, :, 0].double() @ Kc.double().t() / 8.0, 1) @ Vc.double()
    assert (O[0, :, 0] - ref).abs().max() <= 1e-4 * Vc.abs().max()
    with pytest.raises(ValueError, match="workspace has"):
        P.ecokv_decode(Q, Kc, Vc, shape, n, off, max_count, O,
                       workspace=torch.zeros(least - 1, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()


def test_forced_wait_timeout_is_reported(monkeypatch):
    import paper_2609_06663_amd as P
    from paper_2609_06663_amd.pipeline import EvictionPass
    # 8996 non-window keys: four blocks of 4096 keys per unit, which exchange sums
    wl = W.custom(41, L=1, Hq=8, Hkv=2, D=128, w=4, seqlens=[9000], dtype="bf16", budget=[900])
    shape = P.Shape(wl.L, wl.Hq, wl.Hkv, wl.D, wl.w, wl.cu_seqlens)
    ep = EvictionPass(shape, wl.budget, P.PER_HEAD, P.Params(), torch.bfloat16)
    K, V, Q = dev(wl.K, "bf16"), dev(wl.V, "bf16"), dev(wl.Q, "bf16")
    say("split epilogue with a spin limit of 0: its wait gives up at once")
    monkeypatch.setenv("ECOKV_SPIN_LIMIT", "0")
    ep.score(K, Q)
    with pytest.raises(P.EcoKVError) as e:
        ep.check()
    assert e.value.code == P.ETIMEOUT
    lam = ep.lambda_.cpu().numpy()
    assert np.isnan(lam).all() and np.isnan(ep.scores.cpu().numpy()).all()
    say("the query cleared the record; a normal call then reports nothing")
    monkeypatch.delenv("ECOKV_SPIN_LIMIT")
    ep.check()
    ep.score(K, Q)
    ep.check()
    assert np.isfinite(ep.lambda_.cpu().numpy()).all() and np.isfinite(ep.scores.cpu().numpy()).all()


def test_forced_wait_timeout_long_units(monkeypatch):
    # units of 32769 to 65536 non-window keys: eight blocks of 8192 keys per unit exchange sums
    import paper_2609_06663_amd as P
    from paper_2609_06663_amd.pipeline import EvictionPass
    wl = W.custom(42, L=1, Hq=4, Hkv=1, D=128, w=4, seqlens=[40000], dtype="bf16", budget=[4000])
    shape = P.Shape(wl.L, wl.Hq, wl.Hkv, wl.D, wl.w, wl.cu_seqlens)
    ep = EvictionPass(shape, wl.budget, P.PER_HEAD, P.Params(), torch.bfloat16)
    K, Q = dev(wl.K, "bf16"), dev(wl.Q, "bf16")
    say("eight-block epilogue with a spin limit of 0: its waits give up at once")
    monkeypatch.setenv("ECOKV_SPIN_LIMIT", "0")
    ep.score(K, Q)
    with pytest.raises(P.EcoKVError) as e:
        ep.check()
    assert e.value.code == P.ETIMEOUT
    assert np.isnan(ep.lambda_.cpu().numpy()).all() and np.isnan(ep.scores.cpu().numpy()).all()
    monkeypatch.delenv("ECOKV_SPIN_LIMIT")
    ep.score(K, Q)
    ep.check()
    assert np.isfinite(ep.lambda_.cpu().numpy()).all() and np.isfinite(ep.scores.cpu().numpy()).all()
