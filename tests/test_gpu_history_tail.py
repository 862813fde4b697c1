"""One token a round with histories past the registers and the LDS rows: the
entries read again from the Gram buffer, sixteen at a time, on the 16-wave and
the 8-wave launch, with remainders of 0, 1 and 15 in the last sixteen and an
episode that takes every token.  Checked step by step as in
test_gpu_seq_select.py.
"""
import math

import pytest
import torch

from paper_2609_13804_amd import workloads as W
from tests import test_gpu_seq_select as seq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,tokens,caps", [
    ("sixteen_waves", (1000, 577, 830, 640), (300, 250, 85, 101)),
    ("sixteen_waves_to_the_end", (600,), (700,)),
    ("eight_waves", (512, 500, 449), (400, 330, 450)),
])
def test_history_tail(gpu_lib, name, tokens, caps):
    seq.test_edges(gpu_lib, name, tokens, caps, "f32", -math.inf)


@pytest.mark.parametrize("n,cap", [(600, 100), (512, 400), (576, 192), (70, 40)])
def test_an_overflowed_history_term_stays_infinite(gpu_lib, n, cap):
    """Every value's product with every key overflows to +inf: the logits are
    +inf at each step, however many entries the last sixteen hold, and ties go to
    the lowest column."""
    from paper_2609_13804_amd.runner import DeviceRun
    w = W.Workload("overflow", 441, batch=1, d=128, d_text=128, h=64, dtype="f32", text_len=4, tokens=(n,),
                   cap=cap, layout="padded")
    run = DeviceRun(w, W.make_inputs(w), W.make_layout(w), -math.inf)
    run.project()
    run.KQV.zero_()
    run.KQV[:n, 0] = 1e30                      # keys of the tokens
    run.KQV[:n + 1, 128] = 1e30                # values of the tokens and of START
    run.ctx.zero_()
    run.select(flags=0)
    torch.cuda.synchronize()
    assert run.device_errors() == [0, 0, 0]
    assert run.kept_lists()[0] == list(range(cap))
