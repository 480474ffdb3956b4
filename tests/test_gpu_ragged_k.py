"""bf16 GEMMs whose contraction length is no multiple of 64: the last K-tile is
loaded clamped and zeroed past the end.  Blocks against the oracle with
ragged token counts (the weight gradients contract over them), hidden and FFN
widths (every other GEMM does), last K-tiles of 1 to 63 rows or 8 to 56
columns, whole and K-split launches."""
import pytest

from paper_2402_15627_amd import pblock as pb
from paper_2402_15627_amd.inputs import BlockShape
from tests.parity_util import TOL, compare, case, run_gpu, run_oracle

SHAPES = [
    BlockShape("k1", 1, 65, 200, 1, 64, 72, 20, "bf16"),       # last K-tile: 1 token, 8 columns
    BlockShape("k63", 1, 127, 248, 2, 64, 248, 64, "bf16"),    # 63 tokens, 56 columns
    BlockShape("k_short", 1, 3, 72, 1, 64, 8, 2, "bf16"),      # K below one tile
    # dW_in 9216 x 2048 over 300 tokens: 288 tiles, 256 of them whole
    BlockShape("k_whole", 1, 300, 2048, 16, 128, 3072, 150, "bf16"),
    # dh 2 x 5 tiles split along K = 4872 (77 K-tiles, the last of 8)
    BlockShape("k_split", 1, 300, 1096, 4, 128, 3336, 100, "bf16", gelu_tanh=False),
]


def test_ragged_plans():
    p = pb.pblock_gemm_plan(pb.PB_BF16, 300, 1096, 4872)
    assert (p.tiles, p.n_full, p.tail) == (10, 0, 10) and p.splits > 1
    p = pb.pblock_gemm_plan(pb.PB_BF16, 9216, 2048, 300)
    assert (p.tiles, p.n_full, p.tail, p.splits) == (288, 256, 32, 5)
    assert pb.pblock_backward_pairs(pb.config_from_shape(SHAPES[0])) == (False, False)


@pytest.mark.gpu
@pytest.mark.parametrize("s", SHAPES, ids=[s.name for s in SHAPES])
def test_ragged_contractions_match_oracle(s):
    print(f"[gpu] ragged K {s}", flush=True)
    inp = case(s, seed=1)
    errs, bad = compare(s, run_gpu(s, inp), run_oracle(s, inp))
    print("      " + ", ".join(f"{k}={v:.2e}" for k, v in errs.items()), flush=True)
    assert not bad, f"over tolerance {TOL['bf16']}: {bad}"
