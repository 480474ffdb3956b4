"""The fp32 attention kernels (16-row blocks whose 16-row tiles are dealt to
four waves) against the one-head float64 oracle, at sequence lengths and
windows around the block, the tile and the four-tile round, with padded rows;
and non-finite inputs, which reach the rows that see them and no others."""
import numpy as np
import pytest

from oracle import pblock_oracle as orc

pytestmark = pytest.mark.gpu


def run(B, S, nh, d, W, q, k, v, do):
    import torch
    from paper_2402_15627_amd import pblock as pb
    ld = q.shape[-1]
    cfg = pb.make_config(B, S, 64, nh, d, 64, W, "f32")
    q, k, v, do = (torch.from_numpy(a).cuda() for a in (q, k, v, do))
    o, dq, dk, dv = (torch.zeros_like(q) for _ in range(4))
    lse = torch.zeros((B, nh, S), device="cuda")
    pb.pblock_swattn_forward(cfg, q, k, v, ld, o, ld, lse)
    ws = torch.empty(pb.pblock_swattn_workspace_bytes(cfg, pb.ATTN_WS_BACKWARD),
                     dtype=torch.uint8, device="cuda")
    pb.pblock_swattn_backward(cfg, q, k, v, ld, o, ld, do, ld, lse, dq, dk, dv, ld, ws)
    torch.cuda.synchronize()
    return {n: t.cpu().numpy() for n, t in zip(("o", "lse", "dq", "dk", "dv"),
                                               (o, lse, dq, dk, dv))}


def normal(rng, *shape):
    return rng.standard_normal(shape).astype(np.float32)


@pytest.mark.parametrize("S,W", [(1, 1), (15, 16), (16, 1), (17, 2), (64, 64), (65, 17),
                                 (131, 33), (300, 64), (300, 100000)])
@pytest.mark.parametrize("d", [64, 96, 128])
def test_matches_oracle(S, W, d):
    B, nh = 2, 2
    print(f"[gpu] fp32 attention S={S} W={W} d={d}", flush=True)
    rng = np.random.default_rng(S * 1000 + W + d)
    A = nh * d
    q, k, v, do = (normal(rng, B, S, A + 8) for _ in range(4))
    got = run(B, S, nh, d, W, q, k, v, do)
    for n in ("o", "dq", "dk", "dv"):
        assert not got[n][..., A:].any()  # padding columns are never written
    for b in range(B):
        for h in range(nh):
            sl = slice(h * d, (h + 1) * d)
            a = [t[b, :, sl].astype(np.float64) for t in (q, k, v, do)]
            o, lse = orc.swa_head_forward(*a[:3], W)
            ref = dict(zip(("o", "dq", "dk", "dv"), (o, *orc.swa_head_backward(*a, W))))
            np.testing.assert_allclose(got["lse"][b, h], lse, rtol=0, atol=1e-5)
            for n, r in ref.items():
                # S = 1 (or W = 1) has dq = dk = 0: compared against the
                # size of the terms that cancel there, about 1
                scale = max(np.abs(r).max(), 1.0)
                assert np.abs(got[n][b, :, sl] - r).max() <= 1e-5 * scale, (b, h, n)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_non_finite_values_stay_in_their_window(bad):
    """An infinite or NaN value in V (key 40, window 20) reaches the outputs of
    queries 40 .. 59 only, and through dP the gradients of the keys those
    queries see; a NaN query 90 reaches its own row and keys 71 .. 90."""
    B, S, nh, d, W = 1, 128, 1, 64, 20
    print(f"[gpu] fp32 attention with {bad}", flush=True)
    rng = np.random.default_rng(5)
    q, k, v, do = (normal(rng, B, S, d) for _ in range(4))
    clean = run(B, S, nh, d, W, q, k, v, do)
    v2, q2 = v.copy(), q.copy()
    v2[0, 40, 7] = bad
    q2[0, 90, 3] = np.nan
    got = run(B, S, nh, d, W, q2, k, v2, do)
    hit = {"o": [range(40, 60), [90]], "dq": [range(40, 60), [90]],
           "dk": [range(21, 60), range(71, 91)], "dv": [range(71, 91)]}
    for n, ranges in hit.items():
        rows = np.zeros(S, bool)
        for r in ranges:
            rows[list(r)] = True
        finite = np.isfinite(got[n][0]).all(-1)
        assert (finite == ~rows).all(), (n, np.flatnonzero(finite == rows))
        scale = np.abs(clean[n]).max()
        assert np.abs(got[n][0][~rows] - clean[n][0][~rows]).max() <= 1e-5 * scale, n
    # the infinity itself is kept where the definition gives one
    if np.isinf(bad):
        assert (got["o"][0, 40:60, 7] == bad).all()


def test_large_logits():
    """Logits of 64 rms, lse around 150: lse itself is rounded to 2^-17 there, rms
    4.4e-6 of every probability that the backward forms from it, so dV, a sum
    of probabilities times dO, may be 4e-6 off; products with log2 e rounded on
    top (half a unit in the last place of 216, twice) would take it to 5e-6."""
    B, S, nh, d, W = 1, 333, 12, 64, 150
    print("[gpu] fp32 attention, large logits", flush=True)
    rng = np.random.default_rng(8)
    q, k, v, do = (normal(rng, B, S, nh * d) for _ in range(4))
    q *= 8
    k *= 8
    got = run(B, S, nh, d, W, q, k, v, do)
    diff, size = 0.0, 0.0
    for h in range(nh):
        sl = slice(h * d, (h + 1) * d)
        a = [t[0, :, sl].astype(np.float64) for t in (q, k, v, do)]
        dv = orc.swa_head_backward(*a, W)[2]
        diff += np.square(got["dv"][0, :, sl] - dv).sum()
        size += np.square(dv).sum()
    print(f"      dV {np.sqrt(diff / size):.2e}", flush=True)
    assert np.sqrt(diff / size) <= 4e-6
