"""The bf16 epilogues' GeLU and GeLU' at every bf16 value, through calls whose
products are exact: pblock_ag_dc with dC = 1 writes dU = GeLU'(U) for any U,
pblock_ag_in_proj with h = 0 writes GeLU(b_in).

Bounds: half a bf16 step of the float64 value, and an absolute term for the
fp32 evaluation (a few roundings of numbers of size 1, 2.5e-7; in the tails
this dwarfs the value).  NaN stays NaN."""
import numpy as np
import pytest

from paper_2402_15627_amd.inputs import round_to_bf16

pytestmark = pytest.mark.gpu


def _all_bf16():
    return (np.arange(65536, dtype=np.uint32) << 16).view(np.float32)


def _step(ref):
    """bf16 spacing at ref (normal numbers)."""
    return 2.0 ** (np.floor(np.log2(np.maximum(np.abs(ref), 1e-37))) - 7)


def _grad_reference(u):
    """GeLU' of the tanh form in float64; beyond |u| = 30 it is 0 or 1 to well
    below 1e-100."""
    v = np.clip(u.astype(np.float64), -30, 30)
    k = np.sqrt(2 / np.pi)
    a = k * (v + 0.044715 * v ** 3)
    a = np.clip(a, -300, 300)
    s, s1 = 1 / (1 + np.exp(-2 * a)), 1 / (1 + np.exp(2 * a))
    return s + 2 * v * s * s1 * k * (1 + 3 * 0.044715 * v * v)


def _gelu_grad_gpu(u, tokens, hidden):
    """dU of a call in which every element of dC is 1."""
    import torch
    from paper_2402_15627_amd import pblock as pb
    F = u.size // tokens
    cfg = pb.make_config(1, tokens, hidden, 1, 64, F, 1, "bf16", 1e-5, True)
    new = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    dy, w_out, z, d_o, dz = (new(tokens, hidden), new(hidden, 64 + F), new(tokens, 192 + F),
                             new(tokens, 64), new(tokens, 192 + F))
    dy[:, 0] = 1
    w_out[0] = 1
    z[:, 192:] = torch.from_numpy(u.reshape(tokens, F)).cuda().to(torch.bfloat16)
    n = pb.pblock_ag_dc_workspace_bytes(cfg, 1, 1)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
    with pb.TpContext(1) as ctx:
        pb.pblock_ag_dc(cfg, 1, 0, [dy], dy, w_out, z, d_o, dz, 1, ws,
                        torch.cuda.current_stream(), [torch.cuda.Stream()], ctx)
    torch.cuda.synchronize()
    return dz[:, 192:].float().cpu().numpy().reshape(-1)


@pytest.mark.parametrize("tokens,hidden,tile", [(64, 8, 64), (2048, 2048, 256)])
def test_tanh_gelu_grad_of_every_value(tokens, hidden, tile):
    from paper_2402_15627_amd import pblock as pb
    u = np.tile(_all_bf16(), max(1, tokens * 1024 // 65536))
    print(f"[gpu] GeLU' tanh, {tile} x {tile} tiles", flush=True)
    p = pb.pblock_gemm_plan(pb.PB_BF16, tokens, 64 + u.size // tokens, hidden)
    assert p.tiles == -(-tokens // tile) * -(-(64 + u.size // tokens) // tile)
    got = _gelu_grad_gpu(u, tokens, hidden)
    fin = np.isfinite(u)
    assert np.isfinite(got[fin]).all(), f"first at u = {u[fin][~np.isfinite(got[fin])][0]}"
    assert np.isnan(got[np.isnan(u)]).all()
    ref = _grad_reference(u[fin])
    over = np.abs(got[fin] - ref) - 0.5 * _step(ref) - 2.5e-7
    assert over.max() <= 0, (u[fin][over.argmax()], over.max())


def test_erf_gelu_is_correctly_rounded():
    """u in (-4, 8): there no float64 value lies closer to a rounding boundary
    than the fp32 evaluation's error (device erff to an ulp), so each result is
    the bf16 value nearest to it."""
    import torch
    from scipy.special import erfc
    from paper_2402_15627_amd import pblock as pb
    print("[gpu] GeLU erf", flush=True)
    u, T, H = _all_bf16(), 8, 8
    cfg = pb.make_config(1, T, H, 1, 64, u.size, 1, "bf16", 1e-5, False)
    new = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    h, w_in, z, c = new(T, H), new(192 + u.size, H), new(T, 192 + u.size), new(T, 64 + u.size)
    b_in = new(192 + u.size)
    b_in[192:] = torch.from_numpy(u).cuda().to(torch.bfloat16)
    n = pb.pblock_ag_in_proj_workspace_bytes(cfg, 1, 1)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
    with pb.TpContext(1) as ctx:
        pb.pblock_ag_in_proj(cfg, 1, 0, [h], h, w_in, b_in, z, c, 1, ws,
                             torch.cuda.current_stream(), [torch.cuda.Stream()], ctx)
    torch.cuda.synchronize()
    got = c[:, 64:].float().cpu().numpy()
    ok = (u > -4) & (u < 8) & (np.abs(u) > 1e-30)
    v = u[ok].astype(np.float64)
    want = round_to_bf16((v * 0.5 * erfc(-v / np.sqrt(2))).astype(np.float32))
    for row in got:
        assert np.array_equal(row[ok], want), u[ok][row[ok] != want]
    assert np.isnan(got[:, np.isnan(u)]).all()
