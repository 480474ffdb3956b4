"""The 64 x 64-tile bf16 GEMMs of small grids (K split over a workgroup's waves):
where the plan takes them, and blocks on them against the oracle, at tile edges,
contractions that fill no slice of 32 or leave waves without one, ragged and
whole token counts (separate and shared backward launches, db_in formed in
both), both GeLU forms and every head dim.  What of a block runs on other kernels
is asserted too: a GEMM of one 256 x 256 tile and at most four K-tiles keeps that
tile, and dh + dW_in with a long dh is cut along K instead."""
import pytest

from paper_2402_15627_amd import pblock as pb
from paper_2402_15627_amd.inputs import BlockShape
from tests.parity_util import TOL, compare, case, run_gpu, run_oracle

SHAPES = [
    BlockShape("small_one_token", 1, 1, 64, 1, 64, 64, 1, "bf16"),
    BlockShape("small_edges", 1, 65, 136, 1, 64, 200, 30, "bf16"),
    BlockShape("small_d96", 2, 127, 264, 2, 96, 72, 64, "bf16", gelu_tanh=False),
    BlockShape("small_pair", 2, 64, 320, 2, 64, 512, 40, "bf16"),
    BlockShape("small_pair_erf", 3, 64, 576, 3, 128, 1088, 192, "bf16", gelu_tanh=False),
    BlockShape("small_pair_d96_erf", 3, 64, 320, 2, 96, 448, 192, "bf16", gelu_tanh=False),
    BlockShape("small_smoke", 1, 256, 512, 4, 128, 1024, 96, "bf16"),
]


# the backward's pairs, and the GEMMs that keep one 256 x 256 tile
PAIRS = {"small_pair": ("small", "small"), "small_pair_d96_erf": ("small", "small"),
         "small_pair_erf": ("small", "split"), "small_smoke": ("small", "split")}


def _plans(s):
    for M, N, K in ((s.tokens, s.n_in, s.hidden), (s.tokens, s.hidden, s.k_out),
                    (s.tokens, s.k_out, s.hidden), (s.hidden, s.k_out, s.tokens),
                    (s.tokens, s.hidden, s.n_in), (s.n_in, s.hidden, s.tokens)):
        yield M, N, K, pb.pblock_gemm_plan(pb.PB_BF16, M, N, K)


@pytest.mark.parametrize("s", SHAPES, ids=[s.name for s in SHAPES])
def test_blocks_take_small_tiles(s):
    c = pb.config_from_shape(s)
    kinds = tuple(k for k, _ in pb.pblock_backward_launches(c))
    assert kinds == PAIRS.get(s.name, ("apart", "apart"))
    for M, N, K, p in list(_plans(s))[:2 if s.name in PAIRS else 6]:
        if M <= 256 and N <= 256 and K <= 256 and p.tiles == 1:
            assert s.name == "small_one_token"
        else:
            assert p.tiles == -(-M // 64) * -(-N // 64), (M, N, K)


@pytest.mark.parametrize("M,N,K,small", [
    (128, 256, 512, True), (256, 2560, 512, True), (1, 8, 640, True),
    (333, 1280, 256, True), (512, 2048, 2048, True),
    (128, 256, 256, False),       # one 256 x 256 tile of four K-tiles
    (128, 1024, 7168, False),     # a long K is split over workgroups instead
    (1024, 2048, 2048, False), (2048, 10752, 12288, False),
])
def test_plan(M, N, K, small):
    p = pb.pblock_gemm_plan(pb.PB_BF16, M, N, K)
    side = 64 if small else 256
    assert p.tiles == -(-M // side) * -(-N // side)
    if small:
        assert (p.n_full, p.tail, p.splits, p.workgroups) == (p.tiles, 0, 1, p.tiles)


@pytest.mark.gpu
@pytest.mark.parametrize("s", SHAPES, ids=[s.name for s in SHAPES])
def test_small_blocks_match_oracle(s):
    print(f"[gpu] small GEMMs {s}", flush=True)
    c = pb.config_from_shape(s)
    assert pb.pblock_workspace_bytes(c, pb.WS_FORWARD) == 0  # no 256 x 256 tile is split
    inp = case(s, seed=3)
    errs, bad = compare(s, run_gpu(s, inp), run_oracle(s, inp))
    print("      " + ", ".join(f"{k}={v:.2e}" for k, v in errs.items()), flush=True)
    assert not bad, f"over tolerance {TOL['bf16']}: {bad}"
