"""How the backward's shared launches are cut (host only): the rule against the
end of the items in the order in which they start, simulated here."""
import heapq
import random

import pytest

from paper_2402_15627_amd import pblock as pb

CUS = 256


def _tiles(m, n):
    return -(-m // 256) * -(-n // 256)


def _end(n1, a, n2, b):
    """n1 items of a, then n2 of b, each to the CU that is free first."""
    free = [0.0] * CUS
    for t in [a] * n1 + [b] * n2:
        heapq.heapreplace(free, free[0] + t)
    return max(free)


def _config(tokens, hidden, a, ffn, head_dim=128):
    return pb.make_config(1, tokens, hidden, a // head_dim, head_dim, ffn, tokens, "bf16", 1e-5,
                          True)


def _pairs(tokens, hidden, a, ffn):
    """Tiles and K-tiles of dC, dW_out and of dh, dW_in."""
    n_in, k_out = 3 * a + ffn, a + ffn
    return ((_tiles(tokens, k_out), hidden // 64, _tiles(hidden, k_out), tokens // 64),
            (_tiles(tokens, hidden), n_in // 64, _tiles(n_in, hidden), tokens // 64))


# tokens, hidden, A, FFN and the kinds measured fastest (dC + dW_out, dh + dW_in)
@pytest.mark.parametrize("shape,kinds", [
    # long T: 54, 63 and 75 tiles of the weight gradient bound the launch, and
    # cutting the first GEMM delays them
    ((7296, 2176, 256, 1088), ("whole", "whole")),
    ((7744, 768, 768, 3072), ("whole", "whole")),
    ((6336, 1152, 512, 2304), ("whole", "whole")),
    ((3584, 640, 640, 2560), ("whole", None)),
    ((4224, 1664, 384, 1664), ("whole", "whole")),
    # few tokens: the first GEMM's few long tiles bound it
    ((128, 1024, 512, 4096), (None, "split")),
    ((512, 2048, 1024, 8192), (None, "split")),
    ((1024, 4096, 2048, 16384), ("whole", "split")),
    ((192, 8320, 8320, 33280), (None, "split")),
    # the headline workload
    ((2048, 12288, 1536, 6144), ("whole", "whole")),
    # the smallest
    ((256, 256, 256, 1024), ("small", "small")),
])
def test_kinds(shape, kinds):
    got = pb.pblock_backward_launches(_config(*shape))
    assert all(want in (None, kind) for want, (kind, _) in zip(kinds, got)), got


def test_no_cut_makes_a_launch_longer():
    rng = random.Random(3)
    cut = 0
    for _ in range(300):
        tokens = 64 * rng.randint(1, 128)
        a, ffn = 128 * rng.randint(1, 32), 64 * rng.randint(1, 256)
        shape = (tokens, 64 * rng.randint(1, 96), a, ffn)
        cfg = _config(*shape)
        for (t1, k1, t2, k2), (kind, s) in zip(_pairs(*shape), pb.pblock_backward_launches(cfg)):
            if kind != "split":
                assert s == 1
                continue
            cut += 1
            # a tile's stores cost more than nothing; the partial tiles' sum, 1/17 each
            whole = _end(t1, k1, t2, k2 + 1.5)
            assert _end(t1 * s, -(-k1 // s), t2, k2 + 1.5) + t1 * s / 17 < whole, (shape, s)
    assert cut > 50


def test_without_split_region():
    cfg = _config(512, 2048, 1024, 8192)
    full = pb.pblock_workspace_bytes(cfg, pb.WS_BACKWARD)
    assert pb.pblock_backward_launches(cfg, ws_bytes=full)[1][0] == "split"
    assert pb.pblock_backward_launches(cfg, ws_bytes=full - 1)[1] == ("whole", 1)
    ragged = pb.make_config(1, 333, 512, 4, 128, 1024, 333, "bf16", 1e-5, True)
    assert [k for k, _ in pb.pblock_backward_launches(ragged, "serial")] == ["apart"] * 4
