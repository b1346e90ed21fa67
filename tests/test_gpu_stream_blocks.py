"""The streaming sweeps at block lengths that are no power of two (a wave's
32-key groups then no multiple of its register ring), on odd and ragged
lengths: the whole call against the oracle (parity_utils' tolerances)."""
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


@pytest.mark.parametrize("L,Hkv,lens", [
    (1, 4, [40001]),             # about 313 keys for each of 512 blocks: 512-key blocks
    (1, 4, [61003, 33]),         # 480
    (1, 8, [39999, 257, 4097]),  # 695
    (2, 8, [36001, 5]),          # 1126
    (4, 8, [30011, 6007]),       # 2251: 2048-key blocks
])
def test_block_lengths(L, Hkv, lens):
    print(f"[gpu-blocks] L={L} Hkv={Hkv} T={lens}", file=sys.stderr, flush=True)
    wl = W.custom(11 + L, L=L, Hq=2 * Hkv, Hkv=Hkv, D=128, w=4, seqlens=lens, dtype="bf16",
                  budget=[max(4, t // 5) for t in lens], group=256)
    check_per_head(wl, gpu_pass(wl))


@pytest.mark.parametrize("dtype,D,L,lens", [("bf16", 64, 12, [16391]), ("f32", 128, 8, [9001, 4097])])
def test_one_round_of_row_blocks(dtype, D, L, lens):
    # 4 heads: the longest blocks (2048 bf16 keys, 1024 fp32) leave places of one round free
    print(f"[gpu-blocks] {dtype} D={D} L={L} T={lens}", file=sys.stderr, flush=True)
    wl = W.custom(17, L=L, Hq=8, Hkv=4, D=D, w=4, seqlens=lens, dtype=dtype,
                  budget=[t // 5 for t in lens], group=256)
    check_per_head(wl, gpu_pass(wl))
