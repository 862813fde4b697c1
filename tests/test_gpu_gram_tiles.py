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


def gram(sizes, h, dtype, seed=1, rows=None, ctx=None):
    from paper_2609_13804_amd import binding as sp
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    G, T, mg = len(sizes), sum(sizes), max(sizes)
    dm = sp.dims(64, 64, h, sp.SP_F32 if dtype == torch.float32 else sp.SP_BF16)
    KQV = torch.randn((T + 2, 3 * h), generator=g, device="cuda").to(dtype) if rows is None else rows
    ctx = torch.randn((G, h), generator=g, device="cuda") if ctx is None else ctx
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


@pytest.mark.parametrize("h", [64, 640, 1024])
def test_bf16_blocks_do_not_depend_on_the_batch(h):
    """A group's block has the same bits alone and in batches that take the other
    tiles (h 1024, groups of 512: 128 x 192 alone, 128 x 256 for 11 of them, 256 x
    192 for 20; and among groups of other sizes)."""
    n, most = 512, 20
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    rows = torch.randn((most * 576, 3 * h), generator=g, device="cuda").bfloat16()
    ends = torch.randn((2, 3 * h), generator=g, device="cuda").bfloat16()
    ctx = torch.randn((most, h), generator=g, device="cuda")
    want = None
    for sizes in ([n], [n] * 11, [n] * 20, [n, 576, 30], [n] + [576] * 19):
        KQV = torch.cat([rows[:sum(sizes)], ends])
        blocks = gram(sizes, h, torch.bfloat16, rows=KQV, ctx=ctx)[3]
        got = blocks[0][:2 * n + 5, :n + 2].contiguous()
        want = got if want is None else want
        same = got.view(torch.int32) == want.view(torch.int32)
        same[n + 1:, n + 1] = True            # v . START's key is no term of the method
        assert bool(same.all()), (len(sizes), (~same).nonzero()[:4].tolist())


@pytest.mark.parametrize("sizes,h,limit", [([256] * 5, 640, 6.5e-8), ([512] * 3, 512, 6.1e-8), ([512] * 20, 1024, 6.8e-8),
                                           ([768] * 8, 1024, 6.8e-8), ([256] * 300, 1024, 6.7e-8)])
def test_strips_are_as_close_as_lane_sums(sizes, h, limit):
    """START's and the context's rows and STOP's column against 64 bits, 2-norm: no
    further than dot products summed over 64 lanes (the limits, measured on these
    sizes; a sum over 64 lanes rounds h / 64 times at a lane's share and 6 times in
    the tree).  One float32 chain over K is 1.8e-7 off at h 1024."""
    KQV, ctx, off, blocks = gram(sizes, h, torch.bfloat16)
    R = KQV.double()
    start, stop = R[-2], R[-1]
    num = den = 0.0
    for i in range(0, len(sizes), max(1, len(sizes) // 6)):
        n, b = sizes[i], blocks[i].double()
        tok = R[off[i]:off[i] + n]
        keys = torch.cat([tok[:, :h], stop[None, :h]])
        got = [b[n, :n + 1], b[2 * n + 1, :n + 1], b[2 * n + 2:2 * n + 5, :n + 1].sum(0), b[:n, n], b[n + 1:2 * n + 1, n]]
        ref = [keys @ start[h:2 * h], keys @ start[2 * h:], keys @ ctx[i].double(), tok[:, h:2 * h] @ stop[:h],
               tok[:, 2 * h:] @ stop[:h]]
        num += sum(float((x - y).square().sum()) for x, y in zip(got, ref))
        den += sum(float(y.square().sum()) for y in ref)
    print(f"strips {sizes[0]} x {len(sizes)}, h {h}: {(num / den) ** 0.5:.2e}")
    assert (num / den) ** 0.5 <= limit
