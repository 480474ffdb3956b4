"""Shared backward launches whose first GEMM (dC or dh: few tiles, a long K) is
split along K: the blocks against the oracle, and against the same call with a
workspace that leaves no room for the slices (whole tiles)."""
import numpy as np
import pytest

from paper_2402_15627_amd.inputs import BlockShape
from tests.parity_util import GRAD_NAMES, TOL, compare, case, normwise, run_oracle, to_device

pytestmark = pytest.mark.gpu

SHAPES = [
    # dh: four tiles of 9728 / 64 = 152 K-tiles
    BlockShape("pair_split_dh", 1, 128, 1024, 4, 128, 8192, 96, "bf16"),
    # ragged tile edges, several batch rows, heads of 64
    BlockShape("pair_split_d64", 3, 128, 2112, 8, 64, 4160, 50, "bf16"),
    BlockShape("pair_split_erf", 1, 384, 2048, 8, 128, 4096, 128, "bf16", gelu_tanh=False),
]


@pytest.mark.parametrize("s", SHAPES, ids=[s.name for s in SHAPES])
def test_split_shared_launch(s):
    import torch
    from paper_2402_15627_amd import pblock as pb
    print(f"[gpu] split shared launches {s}", flush=True)
    cfg = pb.config_from_shape(s)
    assert pb.pblock_backward_pairs(cfg) == (True, True)
    inp = case(s, seed=2)
    blk = pb.ParallelBlock(cfg, to_device(s, inp))
    blk.forward()
    blk.backward()
    torch.cuda.synchronize()
    get = lambda: {n: blk.grads[n].float().cpu().numpy().astype(np.float64)  # noqa: E731
                   for n in GRAD_NAMES}
    split = get()
    blk.ws = blk.ws[:-1]  # one byte short of the optional split region: whole tiles
    blk.backward()
    torch.cuda.synchronize()
    whole = get()
    ref = run_oracle(s, inp)
    for got in (split, whole):
        errs, bad = compare(s, got, ref, GRAD_NAMES)
        assert not bad, f"over tolerance {TOL['bf16']}: {bad}"
    for n in GRAD_NAMES:
        assert normwise(split[n], whole[n]) <= 1e-2, n
    # the split did happen: its sums round differently
    assert any((split[n] != whole[n]).any() for n in GRAD_NAMES)
