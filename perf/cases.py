"""The work that a program has this library do, as a list of measurable cases.

Every case goes through the public calls (``paper_2609_13804_amd.binding``),
with tensors of the caller's own on the GPU, as a serving or a training program
holds them.  Sizes follow the settings in ``paper_2609_13804_amd/workloads.py``:
one image of a few hundred tokens up to 64 images of 3328; feature widths 1024
to 4096; hidden widths 256 to 1024; bfloat16 and float32; one and five tokens
per round; padded and packed prefill buffers; one-image requests and batches,
even and ragged.

    listed()              the fixed cases
    draw(rng)             one more case of the same ranges
    prepare(case, seed)   inputs, weights, outputs and workspaces on the GPU
    run(state)            one pass, its outputs
    work(case)            the bytes and operations that a pass cannot do without
    tolerance(case)       how far another correct implementation may be
    exact(case, seed)     the computed values in 64 bits, in plain torch
"""
import math
import random

import torch

from paper_2609_13804_amd import binding as sp
from paper_2609_13804_amd import workloads as W

CLUSTERS = 48          # visual tokens: centres plus noise, so near-duplicates exist
NOISE = 0.05
CAUSAL = "causal"


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # A single request at its smallest: one 576-token image, float32, the
        # whole path (project, select, compact).  Latency and launches count.
        dict(name="step_one_image_f32", kind="step", dtype="f32", images=1, lo=576, hi=576, mult=1,
             text=32, d=1024, h=256, split="single", group=0, cap=64, g=1, layout="padded", keep=0.11),
        # The benchmark's batch, the whole path: 16 LLaVA-1.5-shaped images into
        # a padded 576 + 64 prefill buffer.
        dict(name="step_llava15", kind="step", dtype="bf16", images=16, lo=576, hi=576, mult=1,
             text=64, d=4096, h=1024, split="single", group=0, cap=192, g=1, layout="padded", keep=0.111),
        # Serving one dynamic-resolution image (an odd number of tokens): the
        # projection of a single request.
        dict(name="project_one_image", kind="project", dtype="bf16", images=1, lo=1037, hi=1037, mult=1,
             text=96, d=3584, h=1024),
        # Projection of the LLaVA-NeXT-shaped batch: 8 images of 5 x 576 tokens.
        dict(name="project_llavanext", kind="project", dtype="bf16", images=8, lo=2880, hi=2880, mult=1,
             text=128, d=4096, h=1024),
        # Selection over one image's tiles (5 groups of 576), one token a round:
        # the latency of a high-resolution request.
        dict(name="select_one_image", kind="select", dtype="bf16", images=1, lo=2880, hi=2880, mult=1,
             text=128, h=1024, split="fixed", group=576, cap=64, g=1, keep=0.056),
        # Selection of the Qwen2.5-VL-shaped ragged batch, balanced groups.
        dict(name="select_qwen25vl", kind="select", dtype="bf16", images=32, lo=256, hi=4096, mult=4,
             text=96, h=1024, split="balanced", group=576, cap=0.25, g=1, keep=0.111),
        # Selection of the InternVL3-shaped batch, 832 groups of 256 tokens, five
        # tokens per round (the high-resolution setting).
        dict(name="select_internvl3_g5", kind="select", dtype="bf16", images=64, lo=3328, hi=3328, mult=1,
             text=512, h=1024, split="fixed", group=256, cap=7, g=5, keep=0.1),
        # Training: trajectory sums over the full rollout of a 16-image batch.
        dict(name="trajectory_llava15", kind="trajectory", dtype="bf16", images=16, lo=576, hi=576, mult=1,
             text=64, h=1024, split="single", group=0, cap=192, g=1, keep=0.111, tau=1.0, beta=0.9),
        # Gather of the InternVL3-shaped batch's kept tokens and text into a
        # packed prefill buffer.
        dict(name="compact_internvl3", kind="compact", dtype="bf16", images=64, lo=3328, hi=3328, mult=1,
             text=512, d=3584, layout="packed", keep=0.1),
        # The input encoder on one ragged request of narrow features, causal.
        dict(name="encode_one_image_causal", kind="encode", images=1, lo=1037, hi=1037, mult=1, text=40,
             d=1024, attention=CAUSAL),
        # The input encoder on the benchmark's batch.
        dict(name="encode_llava15", kind="encode", images=16, lo=576, hi=576, mult=1, text=64, d=4096,
             attention="both"),
        # Training: the noise gate and denoiser on the benchmark's batch.
        dict(name="denoise_llava15", kind="denoise", tokens=9216, d=4096),
    ]


def _log(rng, lo, hi):
    """An integer from lo to hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "project", "select", "trajectory", "compact", "encode", "denoise"])
    if kind == "denoise":
        d = 64 * rng.randint(8, 64)
        return dict(kind=kind, tokens=_log(rng, 256, 9216), d=d)
    if kind == "encode":
        d = 128 * rng.randint(4, 32)
        images = _log(rng, 1, 16)
        hi = rng.randint(256, 640)
        return dict(kind=kind, images=images, lo=rng.randint(128, hi), hi=hi, mult=1,
                    text=rng.randint(16, 96), d=d, attention=rng.choice(["both", CAUSAL]))
    f32 = rng.random() < 0.25
    dtype = "f32" if f32 else "bf16"
    images = _log(rng, 1, 8 if f32 else 64)
    hi = rng.randint(256, 1100 if f32 else 3328)
    lo = hi if rng.random() < 0.4 else rng.randint(128, hi)
    c = dict(kind=kind, dtype=dtype, images=images, lo=lo, hi=hi, mult=rng.choice([1, 4]),
             text=rng.randint(16, 512 if images > 8 else 128))
    if kind == "compact":
        c.update(d=64 * rng.randint(16, 64), layout=rng.choice(["padded", "packed"]),
                 keep=round(rng.uniform(0.05, 0.34), 3))
        return c
    c["h"] = 64 * rng.randint(4, 8) if f32 else 64 * rng.randint(4, 16)
    if kind == "project":
        c["d"] = 64 * rng.randint(16, 24 if f32 else 64)
        return c
    if kind == "step":
        c["d"] = 64 * rng.randint(16, 24 if f32 else 64)
        c["layout"] = rng.choice(["padded", "packed"])
        c["images"] = min(c["images"], 16)
    group = rng.choice([256, 384, 576, 576, 1000])
    g = 5 if kind != "trajectory" and rng.random() < 0.35 else 1
    c.update(split=rng.choice(["fixed", "balanced"]), group=group, g=g, keep=round(rng.uniform(0.05, 0.15), 3))
    c["cap"] = max(4, int(group * (0.05 if g == 5 else 0.25)))
    if kind == "trajectory":
        c.update(images=min(c["images"], 16), tau=round(rng.uniform(0.5, 2.0), 2), beta=round(rng.uniform(0.8, 1.0), 2))
    return c


# ---------------------------------------------------------------- shapes

def _sizes(c):
    """Visual tokens of every image: the case alone decides them."""
    r = random.Random(c["lo"] * 7919 + c["hi"] * 31 + c["images"])
    m = c["mult"]
    lo, hi = -(-c["lo"] // m), max(c["hi"] // m, -(-c["lo"] // m))
    return [m * r.randint(lo, hi) for _ in range(c["images"])]


def _layout(c):
    sizes = _sizes(c)
    frac = isinstance(c.get("cap"), float)
    w = W.Workload("case", 0, batch=c["images"], d=c.get("d", 64), d_text=c.get("d", 64), h=c.get("h", 64),
                   dtype=c["dtype"], text_len=c["text"], tokens=tuple(sizes), grouping=c.get("split", "single"),
                   group_size=c.get("group", 0), cap=0 if frac else c.get("cap", 0),
                   cap_frac=c.get("cap", 0.0) if frac else 0.0, g=c.get("g", 1), layout=c.get("layout", "padded"))
    return W.make_layout(w)


def _dtype(c):
    return torch.float32 if c.get("dtype") == "f32" else torch.bfloat16


def _code(c):
    return sp.SP_F32 if c.get("dtype") == "f32" else sp.SP_BF16


def _expected_kept(c):
    """About how many tokens each group keeps: the share the STOP bias is set for, within the cap."""
    lay = _layout(c)
    out = []
    for g in range(lay.groups):
        n = int(lay.grp_off[g + 1] - lay.grp_off[g])
        out.append((n, min(c["keep"] * n, int(lay.grp_cap[g]) * c["g"], n)))
    return out


# ---------------------------------------------------------------- inputs

class _Rand:
    """Seeded normal values, drawn on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(1000003 * (seed + 1))

    def normal(self, shape, scale=1.0, dtype=torch.float32):
        return torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32).mul_(scale).to(dtype)

    def uniform(self, shape):
        return torch.rand(shape, generator=self.g, device="cuda")

    def tokens(self, sizes, width, dtype):
        """Rows of every image: a centre of the image plus noise."""
        out = torch.empty((sum(sizes), width), device="cuda", dtype=dtype)
        at = 0
        for n in sizes:
            centres = self.normal((CLUSTERS, width))
            pick = torch.randint(0, CLUSTERS, (n,), generator=self.g, device="cuda")
            out[at:at + n] = centres[pick].add_(self.normal((n, width), NOISE)).to(dtype)
            at += n
        return out


def _ints(a):
    return torch.tensor([int(v) for v in a], dtype=torch.int32, device="cuda")


def _ws(which, dm, T_vis, T_txt, B, G, max_group, max_cap):
    n = sp.stepprune_workspace_bytes(which, dm, T_vis, T_txt, B, G, max_group, max_cap)
    return torch.zeros(n, dtype=torch.uint8, device="cuda"), n


def _project_inputs(c, r):
    sizes, dt, d, h = _sizes(c), _dtype(c), c["d"], c["h"]
    return dict(X=r.tokens(sizes, d, dt), E=r.normal((c["images"] * c["text"], d), 1.0, dt),
                W_kqv=r.normal((3 * h, d), d ** -0.5, dt), W_text=r.normal((h, d), d ** -0.5, dt),
                s_start=r.normal((d,), 1.0, dt), s_stop=r.normal((d,), 1.0, dt))


def _select_inputs(c, r):
    """Projected rows and contexts as the projection leaves them: the features'
    clusters carried through a random linear map, START and STOP rows last, and
    the mean of an image's normalised text rows."""
    h, dt = c["h"], _dtype(c)
    KQV = torch.cat([r.tokens(_sizes(c), 3 * h, dt), r.normal((2, 3 * h), 1.0, dt)])
    ctx = torch.stack([torch.nn.functional.layer_norm(r.normal((c["text"], h)), (h,)).mean(0)
                       for _ in range(c["images"])])
    return dict(KQV=KQV, ctx=ctx)


def _block(r, d, wide, names):
    """A pre-norm block's parameters; ``wide``: output widths of the matrices."""
    out = {}
    for name in names:
        if name.startswith("W_"):
            n_out, n_in = wide[name]
            out[name] = r.normal((n_out, n_in), n_in ** -0.5, torch.bfloat16)
        elif name.startswith("ln") and name.endswith("_g"):
            out[name] = 1.0 + r.normal((d,), 0.1)
        elif name.startswith("ln"):
            out[name] = r.normal((d,), 0.1)
        else:
            out[name] = r.normal((wide.get("W_" + name[2:], (d, d))[0],), 0.02)
    return out


def _encode_inputs(c, r):
    d = c["d"]
    wide = {"W_qkv": (3 * d, d), "W_o": (d, d), "W_1": (4 * d, d), "W_2": (d, 4 * d)}
    return dict(X=r.tokens(_sizes(c), d, torch.bfloat16),
                E=r.normal((c["images"] * c["text"], d), 1.0, torch.bfloat16),
                W_p=r.normal((d, d), d ** -0.5, torch.bfloat16),
                blocks=[_block(r, d, wide, W.ENCODER_FIELDS) for _ in range(2)])


def _denoise_inputs(c, r):
    d, T = c["d"], c["tokens"]
    wide = {"W_v": (d, d), "W_o": (d, d), "W_1": (4 * d, d), "W_2": (d, 4 * d)}
    return dict(X=r.tokens([T], d, torch.bfloat16), alpha=r.uniform((T,)),
                eps=r.normal((T, d), 1.0, torch.bfloat16), p=_block(r, d, wide, W.DENOISER_FIELDS))


def _compact_inputs(c, r):
    """Every image keeps a random ascending subset of its tokens."""
    dt, d = _dtype(c), c["d"]
    X = r.tokens(_sizes(c), d, dt)
    E = r.normal((c["images"] * c["text"], d), 1.0, dt)
    kept = []
    for n in _sizes(c):
        k = max(1, int(round(c["keep"] * n)))
        kept.append(torch.sort(torch.randperm(n, generator=r.g, device="cuda")[:k]).values.to(torch.int32))
    return dict(X=X, E=E, kept=kept)


# ---------------------------------------------------------------- prepare

class _State:
    pass


def prepare(case, seed):
    s = _State()
    c = s.case = dict(case)
    r = _Rand(seed)
    kind = c["kind"]
    if kind == "denoise":
        _prepare_denoise(s, c, r)
    elif kind == "encode":
        _prepare_encode(s, c, r)
    elif kind == "compact":
        _prepare_compact(s, c, r)
    else:
        _prepare_path(s, c, r)
    return s


def _prepare_path(s, c, r):
    kind, dt, h = c["kind"], _dtype(c), c["h"]
    d = c.get("d", 1024)
    lay = _layout(c)
    s.B, s.T_vis, s.T_txt = lay.batch, int(lay.img_off[-1]), int(lay.text_off[-1])
    s.dm = sp.dims(d, d, h, _code(c))
    s.img_off, s.text_off = _ints(lay.img_off), _ints(lay.text_off)
    if kind in ("step", "project"):
        s.__dict__.update(_project_inputs(c, r))
        s.KQV = torch.empty((s.T_vis + 2, 3 * h), dtype=dt, device="cuda")
        s.ctx = torch.empty((s.B, h), dtype=torch.float32, device="cuda")
        s.ws_p = _ws(sp.STAGE_PROJECT, s.dm, s.T_vis, s.T_txt, s.B, 0, 0, 0)
    else:
        s.__dict__.update(_select_inputs(c, r))
    if kind == "project":
        return
    g = s.g = c["g"]
    n = [int(lay.grp_off[i + 1] - lay.grp_off[i]) for i in range(lay.groups)]
    s.G, s.max_group = lay.groups, max(n)
    s.max_cap = max(1, max(min(int(k) * g, m) for k, m in zip(lay.grp_cap, n)))
    s.grp_off, s.grp_img, s.grp_cap = _ints(lay.grp_off), _ints(lay.grp_img), _ints(lay.grp_cap)
    s.kept_off = _ints(lay.kept_off)
    s.kept_idx = torch.full((int(lay.kept_off[-1]),), -1, dtype=torch.int32, device="cuda")
    s.kept_cnt = torch.zeros(s.B, dtype=torch.int32, device="cuda")
    s.grp_cnt = torch.zeros(s.G, dtype=torch.int32, device="cuda")
    s.ws_s = _ws(sp.STAGE_SELECT, s.dm, s.T_vis, s.T_txt, s.B, s.G, s.max_group, s.max_cap)
    if kind == "step":
        s.layout = sp.SP_LAYOUT_PADDED if c["layout"] == "padded" else sp.SP_LAYOUT_PACKED
        s.rows = lay.rows_per_image if c["layout"] == "padded" else 0
        s.out = torch.zeros((lay.out_rows, d), dtype=dt, device="cuda")
        s.seq = torch.zeros(s.B + (c["layout"] == "packed"), dtype=torch.int32, device="cuda")
        s.ws_c = _ws(sp.STAGE_COMPACT, s.dm, s.T_vis, s.T_txt, s.B, s.G, s.max_group, s.max_cap)
        _project(s)
    if kind == "trajectory":
        s.s = torch.zeros(s.T_vis, dtype=torch.float32, device="cuda")
        s.kbar = torch.zeros(s.G, dtype=torch.float32, device="cuda")
        s.pstop = torch.empty((s.G, int(max(lay.grp_cap))), dtype=torch.float32, device="cuda")
    # The STOP bias is a weight of the selector, trained to a retention: take the
    # one at which this batch keeps its share of the tokens.
    total = sum(k for _, k in _expected_kept(c))
    lo, hi = -12.0, 12.0
    for _ in range(14):
        s.b_stop = 0.5 * (lo + hi)
        _select(s)
        if int(s.grp_cnt.sum()) > total:
            lo = s.b_stop
        else:
            hi = s.b_stop
    s.kept_idx.fill_(-1)


def _prepare_compact(s, c, r):
    lay = _layout(c)
    d = c["d"]
    s.__dict__.update(_compact_inputs(c, r))
    s.B, s.T_vis, s.T_txt = lay.batch, int(lay.img_off[-1]), int(lay.text_off[-1])
    s.dm = sp.dims(d, d, 64, _code(c))
    s.img_off, s.text_off = _ints(lay.img_off), _ints(lay.text_off)
    cnt = [int(k.numel()) for k in s.kept]
    off = [0]
    for k in cnt:
        off.append(off[-1] + k)
    s.kept_idx, s.kept_cnt, s.kept_off = torch.cat(s.kept), _ints(cnt), _ints(off)
    packed = c["layout"] == "packed"
    s.layout = sp.SP_LAYOUT_PACKED if packed else sp.SP_LAYOUT_PADDED
    s.rows = 0 if packed else max(cnt) + c["text"]
    rows = off[-1] + s.T_txt if packed else s.B * s.rows
    s.out = torch.zeros((rows, d), dtype=_dtype(c), device="cuda")
    s.seq = torch.zeros(s.B + packed, dtype=torch.int32, device="cuda")
    s.ws_c = _ws(sp.STAGE_COMPACT, s.dm, s.T_vis, s.T_txt, s.B, 0, 0, 0)


def _prepare_encode(s, c, r):
    d = c["d"]
    lay = _layout(dict(c, dtype="bf16"))
    s.__dict__.update(_encode_inputs(c, r))
    s.B, s.T_vis, s.T_txt = lay.batch, int(lay.img_off[-1]), int(lay.text_off[-1])
    s.dm = sp.dims(d, d, 1024, sp.SP_BF16)
    s.img_off, s.text_off = _ints(lay.img_off), _ints(lay.text_off)
    s.max_seq = max(_sizes(c)) + c["text"]
    s.flags = sp.SP_ENC_CAUSAL if c["attention"] == CAUSAL else 0
    s.blk = sp.encoder_blocks(s.blocks)
    s.H = torch.empty((s.T_vis, d), dtype=torch.bfloat16, device="cuda")
    s.ws_e = _ws(sp.STAGE_ENCODE, s.dm, s.T_vis, s.T_txt, s.B, 0, s.max_seq, 0)


def _prepare_denoise(s, c, r):
    d, T = c["d"], c["tokens"]
    s.__dict__.update(_denoise_inputs(c, r))
    s.dm = sp.dims(d, d, 1024, sp.SP_BF16)
    s.params = sp.denoiser(**s.p)
    s.out = torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
    s.ws_g = _ws(sp.STAGE_GATE, s.dm, T, 0, 1, 0, 0, 0)


# ---------------------------------------------------------------- run

def _project(s):
    sp.stepprune_project(s.dm, s.X, s.T_vis, s.s_start, s.s_stop, s.W_kqv, s.E, s.text_off, s.B, s.T_txt,
                         s.W_text, 1.0, 1e-5, s.KQV, s.ctx, s.ws_p[0], s.ws_p[1])


def _select(s):
    sp.stepprune_select(s.dm, s.KQV, s.ctx, s.T_vis, s.img_off, s.B, s.grp_off, s.grp_img, s.grp_cap, s.G,
                        s.max_group, s.max_cap, s.kept_off, s.b_stop, s.g, 0, s.kept_idx, s.kept_cnt,
                        s.grp_cnt, None, 0, s.ws_s[0], s.ws_s[1])


def _compact(s):
    sp.stepprune_compact(s.dm, s.X, s.img_off, s.E, s.text_off, s.kept_idx, s.kept_off, s.kept_cnt, s.B,
                         s.layout, s.rows, s.out.shape[0], s.out, s.seq, s.ws_c[0], s.ws_c[1])


def run(s):
    kind = s.case["kind"]
    if kind == "project":
        _project(s)
        return {"KQV": s.KQV, "ctx": s.ctx}
    if kind == "select":
        _select(s)
        return {"kept_idx": s.kept_idx, "kept_cnt": s.kept_cnt, "grp_cnt": s.grp_cnt}
    if kind == "step":
        _project(s)
        _select(s)
        _compact(s)
        return {"KQV": s.KQV, "ctx": s.ctx, "kept_idx": s.kept_idx, "kept_cnt": s.kept_cnt,
                "grp_cnt": s.grp_cnt, "out": s.out, "seq": s.seq}
    if kind == "trajectory":
        tj = sp.trajectory(s.case["tau"], s.case["beta"], s.s, s.kbar, s.pstop, int(s.pstop.shape[1]))
        sp.stepprune_select_trajectory(s.dm, s.KQV, s.ctx, s.T_vis, s.img_off, s.B, s.grp_off, s.grp_img,
                                       s.grp_cap, s.G, s.max_group, s.max_cap, s.kept_off, s.b_stop, s.g,
                                       sp.SP_FULL_ROLLOUT, s.kept_idx, s.kept_cnt, s.grp_cnt, None, 0, tj,
                                       s.ws_s[0], s.ws_s[1])
        return {"kept_idx": s.kept_idx, "kept_cnt": s.kept_cnt, "grp_cnt": s.grp_cnt, "s": s.s,
                "kbar": s.kbar, "pstop": s.pstop}
    if kind == "compact":
        _compact(s)
        return {"out": s.out, "seq": s.seq}
    if kind == "encode":
        sp.stepprune_encode(s.dm, s.X, s.T_vis, s.img_off, s.B, s.E, s.text_off, s.T_txt, s.W_p, 1.0, s.blk,
                            s.max_seq, s.flags, s.H, s.ws_e[0], s.ws_e[1])
        return {"H": s.H}
    sp.stepprune_gate_denoise(s.dm, s.X, s.case["tokens"], s.alpha, s.eps, s.params, s.out, s.ws_g[0], s.ws_g[1])
    return {"out": s.out}


# ---------------------------------------------------------------- work

def _project_work(c):
    T, L, d, h = sum(_sizes(c)), c["images"] * c["text"], c["d"], c["h"]
    e = 4 if c["dtype"] == "f32" else 2
    return {"bytes": e * ((T + 2) * d + 4 * h * d + L * d + (T + 2) * 3 * h) + 4 * c["images"] * h,
            "flops": 2.0 * (T + 2) * d * 3 * h + 2.0 * L * d * h}


def _select_work(c):
    """Every projected row read once, and per step the newest entry's query and
    value against every key of the group and the weighted sum over the history."""
    e = 4 if c["dtype"] == "f32" else 2
    by = e * (sum(_sizes(c)) + 2) * 3 * c["h"] + 4 * c["images"] * c["h"]
    fl = 0.0
    full = c["kind"] == "trajectory"
    lay = _layout(c)
    for g, (n, k) in enumerate(_expected_kept(c)):
        k = min(int(lay.grp_cap[g]) * c["g"], n) if full else k
        by += 4 * k + (4 * n if full else 0)
        fl += 4.0 * n * c["h"] * (k + 1) + n * k * k / c["g"]
    return {"bytes": by, "flops": fl}


def _compact_work(c, kept):
    e = 4 if c["dtype"] == "f32" else 2
    return {"bytes": 2 * e * c["d"] * (kept + c["images"] * c["text"]) + 4 * kept, "flops": 0}


def work(c):
    kind = c["kind"]
    if kind == "project":
        return _project_work(c)
    if kind in ("select", "trajectory"):
        return _select_work(c)
    if kind == "compact":
        return _compact_work(c, sum(max(1, int(round(c["keep"] * n))) for n in _sizes(c)))
    if kind == "step":
        p, q = _project_work(c), _select_work(c)
        z = _compact_work(c, sum(k for _, k in _expected_kept(c)))
        return {"bytes": p["bytes"] + q["bytes"] + z["bytes"], "flops": p["flops"] + q["flops"]}
    d = c["d"]
    if kind == "denoise":
        T = c["tokens"]
        return {"bytes": 2 * (3 * T * d + 10 * d * d) + 4 * T, "flops": 20.0 * T * d * d}
    sizes, L = _sizes(c), c["text"]
    S = sum(sizes) + len(sizes) * L
    half = 0.5 if c["attention"] == CAUSAL else 1.0
    attn = sum(4.0 * (n + L) ** 2 * d * half for n in sizes)
    return {"bytes": 2 * (2 * sum(sizes) * d + len(sizes) * L * d + 25 * d * d),
            "flops": 2.0 * len(sizes) * L * d * d + 2 * (24.0 * S * d * d + attn)}


# ---------------------------------------------------------------- tolerance

def tolerance(c):
    kind = c["kind"]
    if kind == "compact":
        return "exact"                       # a copy
    if kind == "select":
        # decisions in float32: a different order of its sums moves a logit by
        # about 1e-7 of its scale, and only a near-tie within that can turn
        return {"rel": 1e-5, "differ": 0.01}
    if kind == "trajectory":
        # float32 sums over up to a few hundred steps of float32 softmaxes: up to
        # 5e-7 from 64 bits
        return {"rel": 3e-6, "max": 3e-4, "differ": 0.01}
    if kind == "project" and c["dtype"] == "f32":
        # 6e-7 from 64 bits
        return {"rel": 3e-6, "max": 1e-4}
    if kind == "step" and c["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-4, "differ": 0.01}
    if kind in ("project", "step"):
        # stored bfloat16: 1.7e-3 from the exact product, whichever way it is summed
        return {"rel": 7e-3, "max": 0.02, "differ": 0.01}
    # blocks of bfloat16 products, each operand and result rounded once: about
    # 3.5e-3 from the exact block
    return {"rel": 1.2e-2, "max": 0.15}


# ---------------------------------------------------------------- exact values

def exact(c, seed):
    r = _Rand(seed)
    kind = c["kind"]
    with torch.no_grad():
        if kind in ("project", "step"):
            out = _exact_project(c, _project_inputs(c, r))
            if kind == "step":
                out.update(kept_idx=None, kept_cnt=None, grp_cnt=None, out=None, seq=None)
            return out
        if kind == "trajectory":
            return _exact_trajectory(c, seed)
        if kind == "encode":
            return {"H": _exact_encode(c, _encode_inputs(c, r))}
        if kind == "denoise":
            return {"out": _exact_denoise(c, _denoise_inputs(c, r))}
    return None                              # whole numbers and copies


def _exact_project(c, i):
    Wk = i["W_kqv"].double().t().contiguous()
    T, h = i["X"].shape[0], c["h"]
    KQV = torch.empty((T + 2, 3 * h), dtype=torch.float64, device="cuda")
    for at in range(0, T, 16384):
        KQV[at:min(T, at + 16384)] = i["X"][at:at + 16384].double() @ Wk
    KQV[T] = i["s_start"].double() @ Wk
    KQV[T + 1] = i["s_stop"].double() @ Wk
    t = torch.nn.functional.layer_norm(i["E"].double() @ i["W_text"].double().t(), (h,), eps=1e-5)
    return {"KQV": KQV, "ctx": t.view(c["images"], c["text"], h).mean(1)}


def _exact_trajectory(c, seed):
    """The rollout and its sums, group by group, from the same projected rows."""
    s = prepare(c, seed)
    lay = _layout(c)
    h, tau, beta = c["h"], c["tau"], c["beta"]
    sig = h ** -0.5
    T = int(lay.img_off[-1])
    start, stop = s.KQV[T].double(), s.KQV[T + 1].double()
    out_s = torch.zeros(T, dtype=torch.float64, device="cuda")
    kbar = torch.zeros(lay.groups, dtype=torch.float64, device="cuda")
    pstop = torch.full((lay.groups, int(max(lay.grp_cap))), float("nan"), dtype=torch.float64, device="cuda")
    for g in range(lay.groups):
        a, b = int(lay.grp_off[g]), int(lay.grp_off[g + 1])
        n = b - a
        rows = torch.cat([s.KQV[a:b].double(), start[None]])            # row n: START
        K, Q, V = rows[:, :h], rows[:, h:2 * h], rows[:, 2 * h:]
        keys = torch.cat([K[:n], stop[None, :h]])                        # column n: STOP
        A, Bv, cK = Q @ keys.t(), V @ keys.t(), keys @ s.ctx[int(lay.grp_img[g])].double()
        H = Q @ K.t()                                                    # query against history key
        hist = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        hist[0] = n
        gone = torch.zeros(n + 1, dtype=torch.bool, device="cuda")
        al, bt, size = torch.ones((), dtype=torch.float64, device="cuda"), 1.0, 1
        for t in range(min(int(lay.grp_cap[g]), n + 1)):
            e = hist[size - 1]
            w = torch.softmax(sig * H[e].index_select(0, hist[:size]), 0)
            l = sig * (cK + A[e] + w @ Bv.index_select(0, hist[:size]))
            l[n] += s.b_stop
            l = l.masked_fill(gone, float("-inf"))
            p = torch.softmax(l / tau, 0)
            bt *= beta
            out_s[a:b] += al * bt * p[:n]
            kbar[g] += al * (1.0 - p[n])
            pstop[g, t] = p[n]
            al = al * (1.0 - p[n])
            if t >= n:
                break
            pick = torch.argmax(l[:n])
            gone[pick] = True
            hist[size] = pick
            size += 1
    return {"kept_idx": None, "kept_cnt": None, "grp_cnt": None, "s": out_s, "kbar": kbar, "pstop": pstop}


def _ln(x, g, b):
    return torch.nn.functional.layer_norm(x, (x.shape[-1],), g.double(), b.double(), 1e-6)


def _mlp(x, p):
    y = torch.nn.functional.gelu(_ln(x, p["ln2_g"], p["ln2_b"]) @ p["W_1"].double().t() + p["b_1"].double())
    return x + y @ p["W_2"].double().t() + p["b_2"].double()


def _exact_encode(c, i):
    d, L = c["d"], c["text"]
    E = torch.nn.functional.layer_norm(i["E"].double() @ i["W_p"].double().t(), (d,), eps=1e-5)
    out, at = [], 0
    for b, n in enumerate(_sizes(c)):
        x = torch.cat([i["X"][at:at + n].double(), E[b * L:(b + 1) * L]])
        at += n
        S = n + L
        for p in i["blocks"]:
            qkv = _ln(x, p["ln1_g"], p["ln1_b"]) @ p["W_qkv"].double().t() + p["b_qkv"].double()
            q, k, v = (t.contiguous() for t in qkv.view(S, 3, d // 128, 128).permute(1, 2, 0, 3))
            sc = torch.matmul(q, k.transpose(1, 2).contiguous()) * 128 ** -0.5
            if c["attention"] == CAUSAL:
                sc = sc.masked_fill(torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
            o = torch.matmul(torch.softmax(sc, -1), v).permute(1, 0, 2).reshape(S, d)
            x = _mlp(x + o @ p["W_o"].double().t() + p["b_o"].double(), p)
        out.append(x[:n])
    return torch.cat(out)


def _exact_denoise(c, i):
    p, out = i["p"], []
    for at in range(0, c["tokens"], 4096):
        a = i["alpha"][at:at + 4096].double()[:, None]
        x = a.sqrt() * i["X"][at:at + 4096].double() + (1 - a).sqrt() * i["eps"][at:at + 4096].double()
        u = _ln(x, p["ln1_g"], p["ln1_b"]) @ p["W_v"].double().t() + p["b_v"].double()
        out.append(_mlp(x + u @ p["W_o"].double().t() + p["b_o"].double(), p))
    return torch.cat(out)
