"""The fp32 GEMM's launches (64 x 64 tiles, whole or split along K, and 16 x 64
tiles): the plan that picks one, and the block against the oracle at sizes
where each is taken with remainders in every dimension (rows, columns and a
contraction length that is no multiple of a K-tile or a slice), with each
epilogue, with the split workspace and without it."""
import pytest

from paper_2402_15627_amd import pblock as pb
from paper_2402_15627_amd.inputs import BlockShape
from tests.parity_util import TOL, case, compare, normwise, run_gpu, run_oracle

# (M, N, K): tiles, workgroups, threads, splits
PLANS = [
    (2048, 2048, 2048, 1024, 1024, 256, 1),   # 64 x 64 tiles, four to a CU
    (333, 2824, 520, 945, 945, 512, 1),       # 16 x 64
    (1, 8, 8, 1, 1, 512, 1),
    (333, 520, 2824, 54, 486, 256, 9),        # 54 tiles of 64 x 64 in 9 slices of K
    (128, 256, 1792, 8, 112, 256, 14),
]

SHAPES = [
    # in-projection 333 x 2824 in 16-row tiles, out-projection 333 x 520 and
    # dh split along K, dW_in 2824 x 520 over K = 333 tokens
    BlockShape("f32_tiles_in", 1, 333, 520, 4, 64, 2056, 100, "f32", gelu_tanh=False),
    # 1100 x 1032 outputs: whole 64-row tiles, the last column group 8 wide;
    # dW_out 1032 x 136 takes K = 1100
    BlockShape("f32_tiles_dh", 2, 550, 1032, 1, 64, 72, 33, "f32"),
    # every GEMM's last K-slice is ragged and the rows fill no tile
    BlockShape("f32_tiles_k", 1, 70, 328, 2, 64, 1544, 40, "f32"),
]


@pytest.mark.parametrize("M,N,K,tiles,workgroups,threads,splits", PLANS)
def test_f32_plan(M, N, K, tiles, workgroups, threads, splits):
    p = pb.pblock_gemm_plan(pb.PB_F32, M, N, K)
    assert (p.tiles, p.workgroups, p.threads, p.splits) == (tiles, workgroups, threads, splits)
    blocks = -(-M // 256) * -(-N // 256)
    assert (p.n_full, p.tail) == ((0, blocks) if splits > 1 else (tiles, 0))


@pytest.mark.gpu
@pytest.mark.parametrize("s", SHAPES, ids=[s.name for s in SHAPES])
def test_f32_launches_match_oracle(s):
    import torch
    print(f"[gpu] fp32 GEMM launches {s}", flush=True)
    inp = case(s, seed=0)
    ref = run_oracle(s, inp)
    gpu, blk = run_gpu(s, inp, with_block=True)
    errs, bad = compare(s, gpu, ref)
    print("      " + ", ".join(f"{k}={v:.2e}" for k, v in errs.items()), flush=True)
    assert not bad, f"over tolerance {TOL['f32']}: {bad}"
    # without the optional partial results' space
    t = blk.t
    y2 = torch.empty_like(blk.y)
    pb.pblock_forward(blk.cfg, t["x"], t["gamma"], t["beta"], t["w_in"], t["b_in"], t["w_out"],
                      t["b_out"], y2, blk.saved, None)
    torch.cuda.synchronize()
    y2 = y2.cpu().numpy().astype(float)
    assert normwise(y2.reshape(-1), ref["y"].reshape(-1)) <= TOL["f32"]
