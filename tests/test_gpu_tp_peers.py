"""The pipelined all-gather and reduce-scatter between buffers of two processes:
a second process holds the shards (and the places the chunks go to), which this
one opens by IPC handles, as a tensor-parallel rank opens its peers' buffers.

Such copies belong to the DMA engines, though an opened pointer reads as device
memory like any other; own buffers take the copy kernel.  Both must give the same bits, alone
and mixed in one call."""
import sys

import numpy as np
import pytest

from paper_2402_15627_amd.inputs import BlockShape, make_inputs

pytestmark = pytest.mark.gpu

S = BlockShape("tp_peers", 1, 640, 512, 4, 64, 1000, 64, "bf16", w_std=0.05)
TP, RANK = 8, 3


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _peer(shape, seed, out, done):
    """Holds TP shards of [shape] drawn from the seed, and as many places for
    chunks, until told to go."""
    import torch
    gen = torch.Generator().manual_seed(seed)
    shards = [torch.randn(shape, generator=gen).to(torch.bfloat16).cuda() for _ in range(TP)]
    places = [torch.zeros(shape, dtype=torch.bfloat16, device="cuda") for _ in range(TP)]
    torch.cuda.synchronize()
    out.put((shards, places))
    done.wait(100)


@pytest.fixture(scope="module")
def peer():
    import torch
    import torch.multiprocessing as mp
    ctx = mp.get_context("spawn")
    out, done = ctx.Queue(), ctx.Event()
    torch.zeros(1, device="cuda")
    p = ctx.Process(target=_peer, args=((S.tokens // TP, S.hidden), 4, out, done), daemon=True)
    p.start()
    shards, places = out.get(timeout=90)
    yield shards, places
    torch.cuda.synchronize()
    del shards, places
    done.set()
    p.join(30)


def _weights(seed=1):
    import torch
    inp = make_inputs(S, seed)
    z = np.random.default_rng(seed).standard_normal((S.tokens, S.n_in)).astype(np.float32)
    return (torch.from_numpy(inp["w_out"]).to(torch.bfloat16).cuda(),
            torch.from_numpy(z).to(torch.bfloat16).cuda())


def test_routes(peer):
    import torch
    from paper_2402_15627_amd import pblock as pb
    _say("[gpu] copy routes")
    own = torch.zeros(1024, dtype=torch.bfloat16, device="cuda")
    pinned = torch.zeros(1024, dtype=torch.bfloat16).pin_memory()
    with pb.TpContext(TP) as ctx:
        assert ctx.copies_by_kernel(own, own[512:])
        for other in (peer[0][0], peer[1][TP - 1], pinned):
            assert not ctx.copies_by_kernel(other, own)
            assert not ctx.copies_by_kernel(own, other)


@pytest.mark.parametrize("per,n_comm,own", [(1, 1, ()), (2, 3, (1, 4, 5)), (8, 2, (0,))])
def test_all_gather_of_a_peers_shards(peer, per, n_comm, own):
    """own: shards that are copied here first (in mixed calls the launches with
    a peer's shard among them go to the DMA engines)."""
    import torch
    from paper_2402_15627_amd import pblock as pb
    _say(f"[gpu] ag dC from a peer per={per} n_comm={n_comm} own={own}")
    cfg = pb.config_from_shape(S)
    w_out, z = _weights()
    n = pb.pblock_ag_dc_workspace_bytes(cfg, TP, per)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None

    def run(shards):
        new = lambda w: torch.zeros((S.tokens, w), dtype=torch.bfloat16, device="cuda")  # noqa: E731
        dy, d_o, dz = new(S.hidden), new(S.attn_width), new(S.n_in)
        comm = [torch.cuda.Stream() for _ in range(n_comm)]
        with pb.TpContext(TP) as ctx:
            pb.pblock_ag_dc(cfg, TP, RANK, shards, dy, w_out, z, d_o, dz, per, ws,
                            torch.cuda.current_stream(), comm, ctx)
        torch.cuda.synchronize()
        return dy, d_o, dz
    local = [s.clone() for s in peer[0]]
    want = run(local)
    assert torch.equal(want[0], torch.cat(local))
    got = run([local[j] if j in own else s for j, s in enumerate(peer[0])])
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("per,n_comm,own", [(1, 2, ()), (2, 1, (2, 3)), (8, 3, ())])
def test_reduce_scatter_into_a_peers_buffers(peer, per, n_comm, own):
    import torch
    from paper_2402_15627_amd import pblock as pb
    _say(f"[gpu] rs out-projection to a peer per={per} n_comm={n_comm} own={own}")
    cfg = pb.config_from_shape(S)
    w_out, _ = _weights()
    gen = torch.Generator().manual_seed(9)
    c = torch.randn((S.tokens, S.k_out), generator=gen).to(torch.bfloat16).cuda()
    n = pb.pblock_rs_out_proj_workspace_bytes(cfg, TP, per)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None

    def run(dst):
        partial = torch.zeros((S.tokens, S.hidden), dtype=torch.bfloat16, device="cuda")
        for d in dst:
            d.zero_()
        comm = [torch.cuda.Stream() for _ in range(n_comm)]
        with pb.TpContext(TP) as ctx:
            pb.pblock_rs_out_proj(cfg, TP, RANK, c, w_out, partial, dst, per, ws,
                                  torch.cuda.current_stream(), comm, ctx)
        torch.cuda.synchronize()
        assert torch.equal(torch.cat([d.clone() for d in dst]), partial)
        return partial
    local = [torch.empty_like(d) for d in peer[1]]
    want = run(local)
    got = run([local[j] if j in own else d for j, d in enumerate(peer[1])])
    assert torch.equal(got, want)
