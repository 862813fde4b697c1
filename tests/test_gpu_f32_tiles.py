"""The float32 projection and text products at the edges of their tile choices.

Projections of up to 400 tiles of 64 x 64 take 32 x 64 tiles, larger ones 64 x 64;
the text product's tiles, split over K, follow in the same launch.  K runs in
64-wide stages through a ring of three (two) buffers, so K = 64, 128 and 192 are
the fills and drains shorter than, equal to and longer than it.

Tolerance: a float32 sum of K products is off by at most K roundings of 2^-24 of
the terms' magnitudes; independent roundings add up to about sqrt(K) of that, and
4 sqrt(K) leaves a factor of four.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T_vis,d,h,T_txt,d_text", [
    (1, 64, 64, 1, 64),             # three rows, one stage
    (30, 128, 64, 33, 128),         # exactly one row of tiles; two text tiles
    (31, 192, 128, 32, 64),         # one row past it
    (574, 1024, 256, 31, 1024),     # 18 x 12 tiles and a split text product
    (2110, 128, 256, 40, 192),      # 33 x 12 = 396 of 64 x 64: the last in 32 x 64
    (2111, 128, 256, 40, 192),      # 34 x 12 = 408: the first in 64 x 64, one row in the last
    (2300, 64, 256, 0, 64),         # no text, one stage through two buffers
    (200, 320, 512, 1100, 256),     # more text than tokens
    (1700, 192, 512, 2100, 128),
])
def test_f32_products(gpu_lib, T_vis, d, h, T_txt, d_text):
    from paper_2609_13804_amd import binding as sp
    g = torch.Generator(device="cuda")
    g.manual_seed(T_vis + d)
    rnd = lambda *s, scale=1.0: torch.randn(s, generator=g, device="cuda") * scale
    X, W = rnd(T_vis, d), rnd(3 * h, d, scale=d ** -0.5)
    E, Wt = rnd(max(1, T_txt), d_text), rnd(h, d_text, scale=d_text ** -0.5)
    ss, st = rnd(d), rnd(d)
    off = torch.tensor([0, T_txt], dtype=torch.int32, device="cuda")
    dm = sp.dims(d, d_text, h, sp.SP_F32)
    n = sp.stepprune_workspace_bytes(sp.STAGE_PROJECT, dm, T_vis, T_txt, 1, 0, 0, 0)
    ws = torch.zeros(n + 256, dtype=torch.uint8, device="cuda")
    ws[n:] = 7                       # guards past the outputs: no tile may write them
    KQV = torch.full((T_vis + 3, 3 * h), 7.0, device="cuda")
    ctx = torch.empty((1, h), dtype=torch.float32, device="cuda")
    sp.stepprune_project(dm, X, T_vis, ss, st, W, E, off, 1, T_txt, Wt, 1.0, 1e-5, KQV, ctx, ws, n)
    torch.cuda.synchronize()
    assert sp.stepprune_read_device_error(ws) == 0
    rows = torch.cat([X, ss[None], st[None]]).double()
    ref, mag = rows @ W.double().t(), rows.abs() @ W.double().abs().t()
    assert bool(((KQV[:-1].double() - ref).abs() <= mag * (4 * d ** 0.5) * 2.0 ** -24).all())
    assert bool((KQV[-1] == 7.0).all()) and bool((ws[n:] == 7).all())
    if T_txt:
        c = torch.nn.functional.layer_norm(E.double() @ Wt.double().t(), (h,), eps=1e-5).mean(0)
        assert float((ctx[0].double() - c).abs().max()) <= 1e-5
