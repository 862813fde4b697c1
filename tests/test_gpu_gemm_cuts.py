"""The projection GEMM at the edges of its tile choices.

A product of T tiles of 256 x 256 runs as 64 x 64 tiles (T <= 20), or as whole
tiles with the last round's R cut into quarters (R <= 64), halves (R <= 128) or
left whole; K runs in 64-wide stages through rings two or four stages deep, so
K = 64 .. 320 covers every fill and drain.  Feature widths past the 32-bit
offsets of the tile loads take whole addresses.

Tolerance: the exact product of bfloat16 operands, accumulated in float32 (at
most sqrt(K) 2^-24 of the terms' norm, below 1e-5 of values of unit scale) and
rounded once to bfloat16 (2^-9 relative): 2^-8 |v| + 1e-4.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def run_project(d, h, T_vis, T_txt, d_text, seed):
    from paper_2609_13804_amd import binding as sp
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rnd = lambda *s, scale=1.0: (torch.randn(s, generator=g, device="cuda") * scale).to(torch.bfloat16)
    X, W = rnd(T_vis, d), rnd(3 * h, d, scale=d ** -0.5)
    E, Wt = rnd(max(1, T_txt), d_text), rnd(h, d_text, scale=d_text ** -0.5)
    ss, st = rnd(d), rnd(d)
    off = torch.tensor([0, T_txt], dtype=torch.int32, device="cuda")
    dm = sp.dims(d, d_text, h, sp.SP_BF16)
    n = sp.stepprune_workspace_bytes(sp.STAGE_PROJECT, dm, T_vis, T_txt, 1, 0, 0, 0)
    ws = torch.zeros(n, dtype=torch.uint8, device="cuda")
    # a guard row past the output: no tile may write it
    KQV = torch.full((T_vis + 3, 3 * h), 7.0, dtype=torch.bfloat16, device="cuda")
    ctx = torch.empty((1, h), dtype=torch.float32, device="cuda")
    sp.stepprune_project(dm, X, T_vis, ss, st, W, E, off, 1, T_txt, Wt, 1.0, 1e-5, KQV, ctx, ws, n)
    torch.cuda.synchronize()
    assert sp.stepprune_read_device_error(ws) == 0
    return torch.cat([X, ss[None], st[None]]), W, E[:T_txt], Wt, KQV, ctx


def check(rows, W, E, Wt, KQV, ctx):
    ref = torch.zeros((rows.shape[0], W.shape[0]), dtype=torch.float64, device="cuda")
    for k in range(0, W.shape[1], 1 << 20):
        ref += rows[:, k:k + (1 << 20)].double() @ W[:, k:k + (1 << 20)].double().t()
    got = KQV[:-1].double()
    assert bool(((got - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-4).all())
    assert bool((KQV[-1] == 7.0).all())
    if E.shape[0]:
        c = torch.nn.functional.layer_norm(E.double() @ Wt.double().t(), (W.shape[0] // 3,), eps=1e-5).mean(0)
        assert float((ctx[0].double() - c).abs().max()) <= 1e-5
    else:
        assert bool((ctx == 0).all())


@pytest.mark.parametrize("T_vis,h,T_txt", [
    (1, 64, 1),            # one tile of 64 x 64 parts
    (255, 448, 70),        # 12 + 2 tiles, ragged columns (1344 = 5 x 256 + 64)
    (430, 768, 3),         # 18 + 3: quarters, the first product past the 64 x 64 tiles
    (1180, 1024, 300),     # 60 + 8: halves, text rows in a second panel
    (1537, 1024, 0),       # 84: halves, START alone in the last panel's second row
    (2600, 1024, 129),     # 132 + 4: whole tiles, one round
    (5375, 1024, 31),      # 264 + 4: a whole round and 12 tiles in quarters
    (7000, 1024, 20),      # 336 + 4: a whole round and 84 tiles in halves
])
@pytest.mark.parametrize("d", [64, 192, 320])
def test_cuts(T_vis, h, T_txt, d):
    check(*run_project(d, h, T_vis, T_txt, 128, seed=T_vis + d))


@pytest.mark.parametrize("d", [576, 1024])
def test_deep_k(d):
    """Rings that wrap several times, on quarters and on whole tiles."""
    check(*run_project(d, 1024, 900, 40, d, seed=d))
    check(*run_project(d, 1024, 4000, 40, d, seed=d + 1))


def test_wide_features():
    """d past the 32-bit tile offsets (4,194,304): whole addresses."""
    check(*run_project((1 << 22) + 64, 64, 3, 2, 64, seed=9))
