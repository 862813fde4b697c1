"""Trajectory sums over every launch shape of one token a round: one, two and
three segments of the register-only recurrence, each with and without second
columns, at its edges, and the general kernel past them (8 waves, 8 waves with
second columns, 16 waves).

The untraced run, which a training program makes, is compared with the oracle
along the traced run's actions (tests/parity.py, check_trajectory), the traced
run likewise; a second untraced run gives the same bits.
"""
import math

import numpy as np
import pytest
import torch

from paper_2609_13804_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

INF = math.inf
CASES = [
    # (name, tokens per image, round caps, dtype, STOP bias, full rollout): one launch each
    ("one_segment", (1, 1, 15, 16, 17, 63, 64, 100, 512), (1, 5, 20, 16, 15, 64, 64, 63, 64), "f32", -INF, False),
    ("two_segments", (64, 65, 128, 130, 447), (65, 66, 128, 127, 113), "f32", 0.5, True),
    ("three_segments", (129, 160, 192, 192, 512), (140, 129, 192, 250, 177), "f32", -INF, False),
    ("three_segments_bf16", (512, 300, 65), (192, 192, 192), "bf16", 0.3, False),
    ("second_columns_64", (576, 513, 520, 575, 40), (64, 63, 16, 17, 64), "f32", -INF, False),
    ("second_columns_128", (576, 514), (128, 100), "f32", 0.5, True),
    ("second_columns_192", (576, 513, 20), (192, 161, 192), "bf16", 0.3, True),
    ("past_the_registers", (193, 200), (193, 250), "f32", -INF, False),
    ("second_columns_deep", (576, 530), (193, 300), "f32", 0.5, True),
    ("past_the_columns", (577, 30, 700), (40, 64, 120), "f32", 0.5, True),
]


@pytest.mark.parametrize("name,tokens,caps,dtype,b_stop,full", CASES, ids=[c[0] for c in CASES])
def test_sums(gpu_lib, name, tokens, caps, dtype, b_stop, full):
    from paper_2609_13804_amd import binding as sp
    from paper_2609_13804_amd.runner import DeviceRun
    tau, beta = 0.8, 0.97
    w = W.Workload(name, 500 + len(name), batch=len(tokens), d=128, d_text=128, h=64, dtype=dtype, text_len=4,
                   tokens=tokens, cap=max(caps), layout="padded")
    lay = W.make_layout(w)
    caps = np.asarray(caps, np.int32)
    steps = int(max(min(int(c), n + 1) for c, n in zip(caps, tokens)))
    run = DeviceRun(w, W.make_inputs(w), lay, b_stop, trace_steps=steps, caps=caps)
    run.project()
    flags = sp.SP_FULL_ROLLOUT if full else 0

    def sums(extra):
        out = run.select_trajectory(tau, beta, flags=flags | extra, pstop_steps=steps + 2)
        torch.cuda.synchronize()
        assert run.device_errors() == [0, 0, 0]
        return [t.cpu().numpy() for t in out], run.kept_lists()

    plain, kept = sums(0)
    again, _ = sums(0)
    for a, b in zip(plain, again):
        assert np.array_equal(a, b, equal_nan=True)
    traced, kept_traced = sums(sp.SP_TRACE)
    assert kept_traced == kept
    actions = run.trace_actions()
    for s, kbar, pstop in (plain, traced):
        parity.check_trajectory(run.KQV.double().cpu().numpy(), run.ctx.double().cpu().numpy(), lay.grp_off,
                                lay.grp_img, caps, b_stop, w.h, actions, s, kbar, pstop, tau, beta,
                                ignore_stop=full)
