"""The Gram blocks of the selection against the exact products.

The bfloat16 products run in tiles of 128 x 256, 256 x 192 or 128 x 192 (chosen
by the rounds of workgroups they take) with the rows of START and the context and
the columns of STOP and START as strips; SP_GRAM_ONLY leaves a group's block in
the workspace after its 256-byte header: rows of float32 with stride
ld = max_group + 2 rounded up to 4, A of the tokens, A of START, B of the tokens,
B of START, three rows that sum to the context's.

Tolerance: float32 accumulation of h exact products rounds at most h times, each
by 2^-24 of a partial sum no larger than the sum of magnitudes; the matrix cores
round once per 16 products or less often, so h / 16 + 4 roundings bound it.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu


def gram(sizes, h, dtype, seed=1, imgs=None):
    from paper_2609_13804_amd import binding as sp
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    G, T, mg = len(sizes), sum(sizes), max(sizes)
    dm = sp.dims(64, 64, h, sp.SP_F32 if dtype == torch.float32 else sp.SP_BF16)
    KQV = torch.randn((T + 2, 3 * h), generator=g, device="cuda").to(dtype)
    ctx = torch.randn((G, h), generator=g, device="cuda")
    off = [0]
    for n in sizes:
        off.append(off[-1] + n)
    I = lambda a: torch.tensor(a, dtype=torch.int32, device="cuda")
    o, img, cap, ko = I(off), I(list(range(G))), I([1] * G), I(list(range(G + 1)))
    nb = sp.stepprune_workspace_bytes(sp.STAGE_SELECT, dm, T, 0, G, G, mg, 1)
    ws = torch.zeros(nb, dtype=torch.uint8, device="cuda")
    kept, cnt = I([0] * G), I([0] * G)
    sp.stepprune_select(dm, KQV, ctx, T, o, G, o, img, cap, G, mg, 1, ko, 0.0, 1, sp.SP_GRAM_ONLY,
                        kept, cnt, None, None, 0, ws, nb)
    torch.cuda.synchronize()
    assert sp.stepprune_read_device_error(ws) == 0
    ld = (mg + 2 + 3) // 4 * 4
    rows = 2 * (mg + 1) + 3
    blocks = ws[256:256 + 4 * G * rows * ld].view(torch.float32).view(G, rows, ld)
    return KQV, ctx, off, blocks


def check_group(KQV, c, a, n, blk, h):
    R = KQV.double()
    start, stop = R[-2], R[-1]
    tok = R[a:a + n]
    K, Q, V = tok[:, :h], tok[:, h:2 * h], tok[:, 2 * h:]
    keys = torch.cat([K, stop[None, :h], start[None, :h]])
    left = torch.cat([Q, start[None, h:2 * h], V, start[None, 2 * h:], c.double()[None]])
    ref, mag = left @ keys.t(), left.abs() @ keys.abs().t()
    got = blk[:2 * n + 2, :n + 2].double()
    got = torch.cat([got, blk[2 * n + 2:2 * n + 5, :n + 2].double().sum(0, keepdim=True)])
    tol = mag * (h / 16 + 4) * 2.0 ** -24
    tol[-1] += mag[-1] * 2.0 ** -22           # the context's three-part split
    bad = (got - ref).abs() > tol
    # v . START's key is no term of the method: its column is not compared
    bad[n + 1:2 * n + 2, n + 1] = False
    assert not bool(bad.any()), (n, bad.nonzero()[:4].tolist())


@pytest.mark.parametrize("sizes,h", [
    ([1], 64), ([191, 0, 192, 193], 128), ([255, 256, 7], 256), ([257, 384], 192), ([575, 576], 1024),
    ([577, 96, 95], 448), ([1022], 512), ([64] * 9, 64),
    ([256] * 300, 256),                          # many rounds of 128 x 256
    ([576] * 60 + [300, 1, 0, 530], 320),        # and of 256 x 192, ragged
    ([384] * 96, 1024),
])
def test_bf16_blocks(sizes, h):
    KQV, ctx, off, blocks = gram(sizes, h, torch.bfloat16)
    picks = range(len(sizes)) if len(sizes) <= 10 else [0, 1, len(sizes) // 2, len(sizes) - 4,
                                                        len(sizes) - 3, len(sizes) - 2, len(sizes) - 1]
    for g in picks:
        check_group(KQV, ctx[g], off[g], sizes[g], blocks[g], h)


@pytest.mark.parametrize("sizes,h", [([1, 0, 63], 64), ([64, 65, 200], 256), ([576] * 12, 128)])
def test_f32_blocks(sizes, h):
    KQV, ctx, off, blocks = gram(sizes, h, torch.float32)
    for g in range(len(sizes)):
        check_group(KQV, ctx[g], off[g], sizes[g], blocks[g], h)
