"""The waves' partial sums of the trajectory path cross a barrier before they are
read (csrc/select.hip).

Each step of the recurrence writes a wave's partial softmax sum into ``zpart``;
``traj_finish()`` reads every wave's.  In both kernels, going round the step
loop and past its end, a workgroup barrier has to lie between the writes and
the next read.  A read before it may see a slot of two steps ago, which no test
of values shows reliably, so the order of the statements is checked here.
"""
import os
import re

import pytest

from paper_2609_13804_amd import build as B

EVENT = re.compile(r"(?P<write>zpart\[[^;]*\]\s*=[^=])|(?P<barrier>\b(?:lds_barrier|__syncthreads)\(\);)"
                   r"|(?P<read>\btraj_finish\(\);)")


def _block_end(s, at):
    """The index after the brace block that opens at or after ``at``."""
    i = s.index("{", at)
    depth = 0
    while True:
        depth += {"{": 1, "}": -1}.get(s[i], 0)
        i += 1
        if depth == 0:
            return i


def _kernel(name):
    src = open(os.path.join(B.CSRC, "select.hip")).read()
    src = re.sub(r"//[^\n]*", "", src)
    at = re.search(r"void %s\(SelParams p\)" % name, src).end()
    body = src[at:_block_end(src, at)]
    while True:                     # one token a round: the other side of each GROUPED test is not run
        m = re.search(r"if constexpr \(GROUPED\) \{", body)
        if not m:
            return body
        body = body[:m.start()] + body[_block_end(body, m.start()):]


def _events(s):
    return [m.lastgroup for m in EVENT.finditer(s)]


@pytest.mark.parametrize("name,loop", [("select_seq_kernel", r"auto step = "), ("select_kernel", r"for \(int t = 1; t <= cap; \+\+t\) ")])
def test_partial_sums_cross_a_barrier(name, loop):
    body = _kernel(name)
    at = re.search(loop, body).start()
    end = _block_end(body, at)
    step, rest = _events(body[at:end]), _events(body[end:])
    assert step.count("write") == 1 and "read" in step and "read" in rest, (step, rest)
    # the last step is followed by another one or by the end of the episode
    for after in (step, rest):
        seq = step[step.index("write") + 1:] + after
        assert "barrier" in seq[:seq.index("read")], (name, step, rest)
    # a slot's parity is written again two steps on: a barrier after the read, before that write
    again = step[step.index("read") + 1:] + step
    assert "barrier" in again[:len(again) - again[::-1].index("write")], (name, step)
