"""The register-only recurrence (one token a round, groups of up to 576 tokens,
caps up to 192) at the edges of its history blocks of 16, its segments of 64 and
its columns, and just past them, where the general kernel takes over.

The traced kernel's every step, with its whole logit vector, is compared with the
oracle (tests/parity.py protocol and tolerances), and the untraced kernel must
keep the same tokens.  A bias of -inf runs every episode to its cap or out of
tokens: a cap above the group's size ends in a STOP with no candidate left.
"""
import math

import numpy as np
import pytest
import torch

from paper_2609_13804_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu

CASES = [
    # (name, tokens per image, round caps, dtype, STOP bias): one launch each
    ("one_segment", (1, 1, 15, 16, 17, 63, 64, 100, 512), (1, 5, 20, 16, 15, 64, 64, 63, 64), "f32", -math.inf),
    ("two_segments", (64, 65, 128, 130, 447), (65, 66, 128, 127, 113), "f32", -math.inf),
    ("three_segments", (129, 160, 191, 192, 192, 512), (140, 129, 300, 192, 250, 177), "f32", -math.inf),
    ("past_the_registers", (193, 200), (193, 250), "f32", -math.inf),
    ("second_columns_64", (576, 513, 520, 575, 40), (64, 63, 16, 17, 64), "f32", -math.inf),
    ("second_columns_128", (576, 514), (128, 100), "f32", -math.inf),
    ("second_columns_192", (576, 513), (192, 161), "f32", -math.inf),
    ("second_columns_deep", (576,), (193,), "f32", -math.inf),
    ("past_the_columns", (577, 30), (40, 64), "f32", -math.inf),
    ("stops_bf16", (576, 300, 513, 20, 64), (192, 192, 192, 192, 192), "bf16", 0.3),
]


@pytest.mark.parametrize("name,tokens,caps,dtype,b_stop", CASES, ids=[c[0] for c in CASES])
def test_edges(gpu_lib, name, tokens, caps, dtype, b_stop):
    from paper_2609_13804_amd import binding as sp
    from paper_2609_13804_amd.runner import DeviceRun
    w = W.Workload(name, 400 + len(name), batch=len(tokens), d=128, d_text=128, h=64, dtype=dtype, text_len=4,
                   tokens=tokens, cap=max(caps), layout="padded")
    lay = W.make_layout(w)
    caps = np.asarray(caps, np.int32)
    steps = int(max(min(int(c), n + 1) for c, n in zip(caps, tokens)))
    run = DeviceRun(w, W.make_inputs(w), lay, b_stop, trace_steps=steps, caps=caps, logits=True)
    run.project()
    run.select(flags=0)
    torch.cuda.synchronize()
    assert run.device_errors() == [0, 0, 0]
    plain = run.kept_lists()
    run.select(flags=sp.SP_TRACE | sp.SP_LOGITS)
    torch.cuda.synchronize()
    assert run.device_errors() == [0, 0, 0]
    assert run.kept_lists() == plain
    actions = run.trace_actions()
    parity.check_selection(run.KQV.double().cpu().numpy(), run.ctx.double().cpu().numpy(), lay.grp_off,
                           lay.grp_img, caps, b_stop, w.h, actions, run.trace.cpu().numpy(), w.dtype,
                           logits=run.trace_logits())
    assert plain == parity.kept_from_actions(actions, lay.grp_off, lay.grp_img, lay.img_off, lay.batch)


def test_exact_ties_go_to_the_lowest_column(gpu_lib):
    """Two tokens tie above the rest and the rest tie exactly, at huge logits."""
    from paper_2609_13804_amd.runner import DeviceRun
    w = W.Workload("ties", 431, batch=1, d=128, d_text=128, h=64, dtype="f32", text_len=4, tokens=(70,), cap=8,
                   layout="padded")
    lay = W.make_layout(w)
    run = DeviceRun(w, W.make_inputs(w), lay, -math.inf)
    run.project()
    run.KQV[:70, :64] = 0.0
    run.KQV[:70, 0] = -1.0
    run.KQV[[9, 33], 0] = 1.0
    run.KQV[71, :64] = 0.0                   # STOP's key
    run.ctx.zero_()
    run.KQV[:, 64:128] = 0.0                 # queries add nothing
    run.KQV[:, 128:] = 0.0
    run.ctx[0, 0] = 1e30
    run.select(flags=0)
    torch.cuda.synchronize()
    kept = run.kept_lists()[0]
    assert len(kept) == 8 and 9 in kept and 33 in kept
    # ties beyond them go to the lowest index
    assert kept == sorted([9, 33] + [0, 1, 2, 3, 4, 5])
