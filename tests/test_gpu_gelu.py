"""The GELU of the products' epilogue over [-9, 9], against 64 bits.

The denoiser passes a value straight through: zero features, noise and weights,
the bias b_1 as the GELU's argument, and a W_2 that selects a quarter of the
hidden width, so the output is the GELU rounded to bfloat16.

Bound, beside half a unit of bfloat16's last place (eight significant bits: at most
2^-8 of the value, just above a power of two): 3e-6 of the value above -5, where the kernel's exponent is a fit that is good to 2.6e-6;
2.5e-8 below, where the fit's argument stays at 5 (2e-8).  Values that near the
exact ones round to the same bfloat16 but for the share that lies that near a
boundary between two, about 2 x 3e-6 / 2^-8 of them: fewer than 1 %.
"""
import math

import numpy as np
import pytest
import torch

from paper_2609_13804_amd import binding as sp
from paper_2609_13804_amd import workloads as W

pytestmark = pytest.mark.gpu

D = 512


def _gelu(y):
    """The kernel's GELU of 4 D float32 values, through the denoiser."""
    z = lambda *s: torch.zeros(s, dtype=torch.float32, device="cuda")
    zb = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    t = {"ln1_g": z(D), "ln1_b": z(D), "W_v": zb(D, D), "b_v": z(D), "W_o": zb(D, D), "b_o": z(D), "ln2_g": z(D),
         "ln2_b": z(D), "W_1": zb(4 * D, D), "b_1": torch.from_numpy(y).cuda(), "W_2": zb(D, 4 * D), "b_2": z(D)}
    assert set(t) == set(W.DENOISER_FIELDS)
    dm = sp.dims(D, D, 128, sp.SP_BF16)
    T = 4                       # every row is the same
    nb = sp.stepprune_workspace_bytes(sp.STAGE_GATE, dm, T, 0, 1, 0, 0, 0)
    ws = torch.zeros(nb, dtype=torch.uint8, device="cuda")
    got = []
    for k in range(4):
        t["W_2"].zero_()
        t["W_2"][:, k * D:(k + 1) * D] = torch.eye(D, device="cuda").bfloat16()
        out = zb(T, D)
        sp.stepprune_gate_denoise(dm, zb(T, D), T, z(T), zb(T, D), sp.denoiser(**t), out, ws, nb)
        torch.cuda.synchronize()
        assert bool((out == out[:1]).all())
        got.append(out[0].double().cpu().numpy())
    return np.concatenate(got)


@pytest.mark.parametrize("lo,hi", [(-9.0, -5.0), (-5.0, -2.0), (-2.0, 2.0), (2.0, 9.0)])
def test_gelu(gpu_lib, lo, hi):
    rng = np.random.default_rng(int(10 * (lo + 10)))
    y = np.concatenate([[lo, hi], rng.uniform(lo, hi, 4 * D - 2)]).astype(np.float32)
    want = np.array([0.5 * float(v) * math.erfc(-float(v) / math.sqrt(2.0)) for v in y])
    got = _gelu(y)
    tail = y < -5.0
    tol = np.abs(want) * 2.0 ** -8 + np.where(tail, 2.5e-8, 3e-6 * np.abs(want))
    assert np.all(np.abs(got - want) <= tol), y[np.abs(got - want) > tol][:5]
    if not tail.any():
        rounded = torch.from_numpy(want).to(torch.bfloat16).double().numpy()
        assert np.mean(got == rounded) >= 0.99
