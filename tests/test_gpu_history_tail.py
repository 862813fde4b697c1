"""One token a round with histories past the registers and the LDS rows: the
entries read again from the Gram buffer, sixteen at a time, on the 16-wave and
the 8-wave launch, with remainders of 0, 1 and 15 in the last sixteen and an
episode that takes every token.  Checked step by step as in
test_gpu_seq_select.py.
"""
import math

import pytest

from tests import test_gpu_seq_select as seq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,tokens,caps", [
    ("sixteen_waves", (1000, 577, 830, 640), (300, 250, 85, 101)),
    ("sixteen_waves_to_the_end", (600,), (700,)),
    ("eight_waves", (512, 500, 449), (400, 330, 450)),
])
def test_history_tail(gpu_lib, name, tokens, caps):
    seq.test_edges(gpu_lib, name, tokens, caps, "f32", -math.inf)
