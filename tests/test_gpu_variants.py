"""Kernel variants that a rule on sizes, types or alignment chooses between: each at the sizes where it can go wrong,
against the oracle or against the general path."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2407_14417_amd import binding as mm, synth
from tests.gpu_common import dev

pytestmark = pytest.mark.gpu


# ---------------------------------------------------------------- quantizer: 128-bit loads against 2-byte loads

def _quantized(w, bits, shift):
    """Codes, scales and zeros of `w`, read from an address `shift` halves past an aligned one."""
    out, inn = w.shape
    buf = torch.zeros(out * inn + 8, dtype=torch.float16, device="cuda")
    src = buf[shift:shift + out * inn].view(out, inn)
    src.copy_(w)
    codes = torch.zeros((out, inn * bits // 8), dtype=torch.uint8, device="cuda")
    scale, zero = (torch.zeros((out, inn // 64), dtype=torch.float16, device="cuda") for _ in range(2))
    (mm.moe_quantize_int4 if bits == 4 else mm.moe_quantize_int8)(src, codes, scale, zero)
    return codes.cpu().numpy(), scale.cpu().numpy().view(np.uint16), zero.cpu().numpy().view(np.uint16)


def _grid_weights(out, inn):
    """Every group on a grid of half steps of its own scale (quotients that are ties), other groups constant, with
    both zeros, subnormal, at the edge of fp16 or holding infinities and NaN."""
    rng = np.random.default_rng(5)
    w = synth.normal_f16((out, inn), 0.02, 4, 61).astype(np.float32).reshape(-1, 64)
    n = w.shape[0]
    for g in range(n):
        kind = g % 8
        if kind == 1:
            w[g] = (rng.integers(0, 31, 64) * 0.5 - 3) * 2.0 ** rng.integers(-8, 3)
        elif kind == 2:
            w[g] = rng.choice([0.0, -0.0], 64)
        elif kind == 3:
            w[g] = rng.integers(0, 40, 64) * 2.0 ** -24
        elif kind == 4:
            w[g] = rng.choice([-65504.0, 65504.0, 1e-4, 3.0], 64)
        elif kind == 5:
            w[g, rng.integers(0, 64, 3)] = rng.choice([np.inf, -np.inf], 3)
        elif kind == 6:
            w[g, rng.integers(0, 64, 3)] = np.nan
        elif kind == 7:
            w[g] = (rng.integers(0, 511, 64) * 0.5) * 2.0 ** -10
    return w.astype(np.float16).reshape(out, inn)


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("shape", [(1, 64), (3, 64), (33, 2048), (8, 1024), (301, 1088)])
def test_quantizer_wide_loads_equal_narrow_loads(orc, bits, shape):
    for w in (synth.normal_f16(shape, 0.02, 4, 60), _grid_weights(*shape)):
        wide, narrow = _quantized(dev(w), bits, 0), _quantized(dev(w), bits, 1)
        for a, b in zip(wide, narrow):
            assert np.array_equal(a, b)
        if np.isfinite(w.astype(np.float32)).all() and not (w == 0).any():
            ref = orc.quantize_int4(w) if bits == 4 else orc.quantize_int8(w)
            assert np.array_equal(wide[0], ref.data)
            assert np.array_equal(wide[1], ref.scale.view(np.uint16)) and np.array_equal(wide[2], ref.zero.view(np.uint16))
