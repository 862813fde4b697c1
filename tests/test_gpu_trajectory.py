"""Trajectory sums of the training surrogate on the GPU (Eqs. 5-7 along the
pointer trajectory; stepprune_select_trajectory), against the oracle with the
staged, teacher-forced protocol of tests/parity.py (check_trajectory for the
sums, check_selection for the decisions), with and without the full rollout
(SP_FULL_ROLLOUT): traced runs of the paper-shaped workloads and of histories
past every tier.  The untraced kernels and the other launch shapes are in
test_gpu_trajectory_shapes.py.
"""
import math

import numpy as np
import pytest
import torch

from paper_2609_13804_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

CASES = [
    # (workload, tau, beta, full rollout)
    ("tiny_f32", 1.0, 0.9, False),
    ("tiny_f32", 0.5, 1.0, True),
    ("tiny_bf16", 2.0, 0.95, False),
    ("small_packed_bf16", 1.0, 0.9, True),
    ("mid_bf16", 1.0, 0.9, False),
    ("mid_bf16", 0.7, 0.98, True),
]


def _run(name, tau, beta, full, caps=None, b_stop=None):
    from paper_2609_13804_amd import binding as sp
    from paper_2609_13804_amd.runner import DeviceRun
    w = W.WORKLOADS[name]
    lay, inp = W.make_layout(w), W.make_inputs(w)
    c = lay.grp_cap if caps is None else np.asarray(caps, np.int32)
    steps = int(max(min(int(x), int(n)) for x, n in zip(c, np.diff(lay.grp_off)))) + 1
    run = DeviceRun(w, inp, lay, W.stop_bias(w) if b_stop is None else b_stop, trace_steps=steps,
                    caps=c)
    run.project()
    flags = sp.SP_TRACE | (sp.SP_FULL_ROLLOUT if full else 0)
    ts, kb, ps = run.select_trajectory(tau, beta, flags=flags, pstop_steps=steps + 2)
    torch.cuda.synchronize()
    assert run.device_errors() == [0, 0, 0]
    return w, lay, run, ts.cpu().numpy(), kb.cpu().numpy(), ps.cpu().numpy()


@pytest.mark.parametrize("name,tau,beta,full", CASES)
def test_trajectory_sums_match_the_oracle(gpu_lib, name, tau, beta, full):
    w, lay, run, s, kbar, pstop = _run(name, tau, beta, full)
    KQV = run.KQV.double().cpu().numpy()
    ctx = run.ctx.double().cpu().numpy()
    actions = run.trace_actions()
    sel = parity.check_selection(KQV, ctx, lay.grp_off, lay.grp_img, run.caps_host, run.b_stop, w.h,
                                 actions, run.trace.cpu().numpy(), w.dtype, ignore_stop=full)
    rep = parity.check_trajectory(KQV, ctx, lay.grp_off, lay.grp_img, run.caps_host, run.b_stop,
                                  w.h, actions, s, kbar, pstop, tau, beta, ignore_stop=full)
    if full:
        sizes = np.diff(lay.grp_off)
        assert [len(a) for a in actions] == [int(c) if c <= n else int(n) + 1
                                             for c, n in zip(run.caps_host, sizes)]
    print(f"{name} tau={tau} beta={beta} full={full}: {rep.episodes} episodes, "
          f"{sel.exempt_steps} exempt steps, max errors s {rep.max_s_err:.2e}, "
          f"K_bar {rep.max_kbar_err:.2e}, p(STOP) {rep.max_pstop_err:.2e}")


def test_trajectory_run_decides_as_the_plain_selection(gpu_lib):
    """The trajectory kernel takes the plain kernel's decisions."""
    w, lay, run, s, kbar, pstop = _run("mid_bf16", 1.0, 0.9, False)
    kept_traj = run.kept_lists()
    run.select(flags=0)
    torch.cuda.synchronize()
    assert run.kept_lists() == kept_traj


def test_long_full_rollouts_cross_every_history_tier(gpu_lib):
    """Full rollouts of 400 steps on 576-token groups (register, LDS and
    re-read history tiers, second columns)."""
    w0 = W.WORKLOADS["mid_bf16"]
    caps = np.minimum(np.diff(W.make_layout(w0).grp_off), 400)
    w, lay, run, s, kbar, pstop = _run("mid_bf16", 1.0, 0.99, True, caps=caps)
    KQV = run.KQV.double().cpu().numpy()
    ctx = run.ctx.double().cpu().numpy()
    rep = parity.check_trajectory(KQV, ctx, lay.grp_off, lay.grp_img, caps, run.b_stop, w.h,
                                  run.trace_actions(), s, kbar, pstop, 1.0, 0.99, ignore_stop=True)
    print(f"long rollouts: max errors s {rep.max_s_err:.2e}, K_bar {rep.max_kbar_err:.2e}")
