"""Where the bf16 attention splits a block's tiles over several workgroups (a
host-only plan, seen through the workspace sizes): long blocks of few heads are
split, short windows stay whole, and the allocation-free entry point's limit
does not depend on that choice."""
import ctypes

import pytest

from paper_2402_15627_amd import pblock as pb

FAKE = 1 << 40


def ws(S, heads, d, W, batch=1):
    c = pb.make_config(batch, S, 64, heads, d, 64, W)
    size = lambda mode: pb.pblock_swattn_workspace_bytes(c, mode)  # noqa: E731
    return size(pb.ATTN_WS_FORWARD) > 0, size(pb.ATTN_WS_BACKWARD) > size(pb.ATTN_WS_BACKWARD_MIN)


@pytest.mark.parametrize("B,S,heads,d,W,fwd", [
    # us split, us whole
    (4, 1396, 7, 96, 1396, True),   # 34.0, 38.9
    (2, 1359, 16, 96, 1359, True),  # 31.5, 38.5
    (2, 677, 2, 96, 384, True),     # 12.9, 14.5
    (2, 870, 10, 64, 870, True),    # 17.6, 21.6
    (3, 510, 1, 128, 177, True),    # 12.6, 13.5
    (2, 1192, 12, 96, 238, False),  # 22.0, 13.9
    (3, 675, 16, 128, 300, False),  # 24.4, 17.4
    (1, 5770, 5, 128, 342, False),  # 30.7, 20.9
])
def test_split_plan_of_batches(B, S, heads, d, W, fwd):
    assert ws(S, heads, d, W, B)[0] == fwd


@pytest.mark.parametrize("S,heads,d,W,fwd,bwd", [
    (2048, 12, 128, 2048, True, False),  # the backward's two roles fill the chip
    (4544, 3, 128, 4544, True, True),
    (1024, 8, 128, 1024, True, True),
    # forward 14.5 us split, 15.9 whole; backward 30.6 and 25.7
    (512, 8, 128, 512, True, False),
    (1024, 16, 96, 512, False, False),
    (4096, 4, 128, 256, False, False),
    (256, 4, 128, 96, False, False),
    (1, 1, 64, 1, False, False),
    (8192, 40, 128, 1024, False, False),
])
def test_split_plan(S, heads, d, W, fwd, bwd):
    assert ws(S, heads, d, W) == (fwd, bwd)


def test_noalloc_limit_is_that_of_the_finest_split():
    # 256 forward blocks of 6 tiles: kept whole, yet two chunks would take
    # 2 x 8192 x 4 x 128 fp32 partials and their row terms, over 32 MiB
    c = pb.make_config(1, 8192, 64, 4, 128, 64, 256)
    assert pb.pblock_swattn_workspace_bytes(c, pb.ATTN_WS_FORWARD) == 0
    st = pb.load_library().pblock_swattn_forward_noalloc(
        ctypes.byref(c), FAKE, FAKE, FAKE, 512, FAKE, 512, FAKE, None)
    assert st == 2 and "scratch" in pb.pblock_last_error()
