"""Launches for many rows per expert, each asked from the library (common.launch_forms) before it is run, so that a change of
its rules cannot leave a kernel untested: weights drawn and quantized on the device, tokens sent to chosen experts, a
float64 product with the dequantized weights as the reference."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2407_14417_amd import binding as mm
from tests.common import assert_ffn_close, launch_forms

pytestmark = pytest.mark.gpu

PREC = {"h": mm.PREC_FP16, "q": mm.PREC_INT4G64, "e": mm.PREC_INT8G64}


def _draw(gen, shape, sigma):
    return torch.empty(shape, dtype=torch.float16, device="cuda").normal_(0.0, sigma, generator=gen)


def _expert(gen, d, f, bits):
    """(expert, its three matrices as fp16)"""
    mats, dense = [], []
    for o, i in ((f, d), (f, d), (d, f)):
        w = _draw(gen, (o, i), 0.02)
        if bits == "h":
            mats.append(mm.Mat(w))
        else:
            codes = torch.empty((o, i // 2 if bits == "q" else i), dtype=torch.uint8, device="cuda")
            scale, zero = (torch.empty((o, i // 64), dtype=torch.float16, device="cuda") for _ in range(2))
            (mm.moe_quantize_int4 if bits == "q" else mm.moe_quantize_int8)(w, codes, scale, zero)
            mats.append(mm.Mat(codes, scale, zero))
            (mm.moe_dequant_int4 if bits == "q" else mm.moe_dequant_int8)(mats[-1], o, i, w)
        dense.append(w)
    return mm.Expert(PREC[bits], *mats), dense


def _reference(x, dense):
    w1, w3, w2 = (w.double() for w in dense)
    a = x.double() @ w1.t()
    return ((torch.nn.functional.silu(a) * (x.double() @ w3.t())) @ w2.t()).cpu().numpy()


def _routed(gen, d, E, rows):
    """Tokens of which rows[e] go to expert e (top-1), in mixed order; a gate matrix that reads the choice off their first
    columns."""
    to = torch.cat([torch.full((n,), e) for e, n in enumerate(rows)])
    to = to[torch.randperm(len(to), generator=torch.Generator().manual_seed(len(to)))].cuda()
    x = _draw(gen, (len(to), d), 1.0)
    x[:, :E] *= 0.125
    x[torch.arange(len(to), device="cuda"), to] = 8.0
    gate = torch.zeros((E, d), dtype=torch.float16, device="cuda")
    gate[torch.arange(E), torch.arange(E)] = 1.0
    return x, to, gate


def _block(d, f, gate, experts, x):
    T = x.shape[0]
    out = torch.full((T, d), float("nan"), dtype=torch.float16, device="cuda")
    idx = torch.empty((T, 1), dtype=torch.int32, device="cuda")
    layer = mm.Layer(d, f, 1, gate, experts)
    ws = mm.alloc_workspace(layer, T).fill_(0xFF)
    mm.moe_layer_forward(layer, x, out, ws, idx)
    assert mm.moe_read_status(ws) == 0
    return out, idx[:, 0]


def _check(d, f, gate, experts, dense, x, to):
    out, idx = _block(d, f, gate, experts, x)
    assert torch.equal(idx.long(), to)
    for e in range(len(experts)):
        mine = to == e
        if bool(mine.any()):
            assert_ffn_close(out[mine].cpu().numpy(), _reference(x[mine], dense[e]), f"expert {e}, {int(mine.sum())} rows")


@pytest.fixture(scope="module")
def weights():
    """Experts of a shape and string of precisions, kept until another is asked for."""
    held = {}

    def get(d, f, bits):
        if (d, f, bits) not in held:
            held.clear()
            gen = torch.Generator(device="cuda").manual_seed(d + f)
            held[d, f, bits] = [_expert(gen, d, f, b) for b in bits]
        return [e for e, _ in held[d, f, bits]], [w for _, w in held[d, f, bits]]
    return get


# Workgroups of 8 wavefronts: for each precision every number of 16-row tiles a chunk can have, with one row and with all rows
# in the last one; contractions of 8 steps up and 4 down (walked from different places), of 9 and 3, of 3 and 2 (shorter than
# the LDS rings are deep); tiles of weight rows that end past the matrix (1152, 384).
TILES = [(1, 9, 14), (2, 7, 15), (3, 5, 16), (4, 6, 13), (8, 5, 11), (2, 10, 12)]


@pytest.mark.parametrize("d,f,bits,up_steps,down_steps", [(1024, 4096, "hqe" * 3, 8, 4), (1024, 4096, "hqq" * 3, 8, 4), (1152, 4224, "hqe" * 3, 9, 3),
                                                          (384, 1792, "hqe" * 7, 3, 2)])
@pytest.mark.parametrize("tiles", TILES)
@pytest.mark.parametrize("full", [False, True])
def test_prefill_eight_wavefronts(weights, d, f, bits, up_steps, down_steps, tiles, full):
    experts, dense = weights(d, f, bits)
    E = len(bits)
    rows = [16 * tiles[e // 3 % 3] - (0 if full else 15 if e < 3 else e) for e in range(E)]
    rows[9:] = [100, 1, 128, 90, 110, 127, 16, 128, 113, 100, 97, 128][:E - 9]
    form = launch_forms([PREC[b] for b in bits], d, f, 1, sum(rows))
    assert [m.waves for m in form] == [8, 8] and [m.quant_rows for m in form] == [256, 256]
    assert [m.steps_per_split for m in form] == [up_steps, down_steps]
    x, to, gate = _routed(torch.Generator(device="cuda").manual_seed(sum(rows)), d, E, rows)
    _check(d, f, gate, experts, dense, x, to)


# Workgroups of 4 wavefronts: the same for chunks of up to 8 tiles, with and without 8-bit experts in the block (two kernels).
@pytest.mark.parametrize("bits", ["hqe" * 3, "hqq" * 3])
@pytest.mark.parametrize("d,f", [(640, 384), (1024, 2048)])
@pytest.mark.parametrize("tiles", [(1, 6, 8), (2, 5, 8), (3, 4, 7)])
@pytest.mark.parametrize("full", [False, True])
def test_prefill_four_wavefronts(weights, d, f, bits, tiles, full):
    experts, dense = weights(d, f, bits)
    rows = [16 * tiles[e // 3] - (0 if full else 15 if e < 3 else e) for e in range(9)]
    assert [m.waves for m in launch_forms([PREC[b] for b in bits], d, f, 1, sum(rows))] == [4, 4]
    x, to, gate = _routed(torch.Generator(device="cuda").manual_seed(sum(rows)), d, 9, rows)
    _check(d, f, gate, experts, dense, x, to)


# More rows than a chunk holds: chunks of 256, 192 and 128 rows of quantized experts, split evenly, with as many of 256 of
# 16-bit ones between them.
@pytest.mark.parametrize("rows,quant", [((257, 300, 300, 200, 150, 270, 520, 100, 153), (256, 256)),
                                        ((257, 300, 300, 520, 400, 129, 130, 513, 151), (128, 128)),
                                        ((385, 385, 385, 385, 385, 385, 385, 385, 385), (192, 128)),
                                        ((100, 390, 520, 900, 700, 513, 193, 500, 684), (256, 192))])
def test_prefill_several_chunks(weights, rows, quant):
    d, f, bits = 1024, 4096, "hqe" * 3
    experts, dense = weights(d, f, bits)
    form = launch_forms([PREC[b] for b in bits], d, f, 1, sum(rows))
    assert [m.waves for m in form] == [8, 8] and tuple(m.quant_rows for m in form) == quant
    x, to, gate = _routed(torch.Generator(device="cuda").manual_seed(sum(rows)), d, 9, rows)
    _check(d, f, gate, experts, dense, x, to)


def test_prefill_as_many_experts_as_there_can_be(weights):
    """Chunks are handed out by length over all 32, one of them without tokens."""
    d, f, bits = 256, 1152, "hqeq" * 8
    experts, dense = weights(d, f, bits)
    rows = [9 * (e * 5 % 32) for e in range(32)]
    assert launch_forms([PREC[b] for b in bits], d, f, 1, sum(rows))[0].waves == 8
    x, to, gate = _routed(torch.Generator(device="cuda").manual_seed(1), d, 32, rows)
    _check(d, f, gate, experts, dense, x, to)


# One expert alone on 8 wavefronts: chunks of 128 rows and a rest below two rounds of workgroups, the even split above.
@pytest.mark.parametrize("d,f,n,waves,quant", [(512, 14336, 300, (8, 4), 0), (512, 14336, 540, (8, 4), 256), (512, 14336, 1100, (8, 4), 192),
                                               (4096, 1792, 1100, (4, 8), 0)])
def test_prefill_one_expert_alone(weights, d, f, n, waves, quant):
    experts, dense = weights(d, f, "hqe")
    x = _draw(torch.Generator(device="cuda").manual_seed(n), (n, d), 1.0)
    layer = mm.Layer(d, f, 1, torch.zeros((3, d), dtype=torch.float16, device="cuda"), experts)
    ws = mm.alloc_workspace(layer, n)
    for e in range(3):
        form = launch_forms([PREC[b] for b in "hqe"], d, f, 1, n, e)
        assert tuple(m.waves for m in form) == waves and form[waves.index(8)].quant_rows == quant
        y = torch.full((n, d), float("nan"), dtype=torch.float32, device="cuda")
        mm.moe_expert_ffn_mixed(layer, e, x, y, ws)
        assert_ffn_close(y.cpu().numpy(), _reference(x, dense[e]), f"expert {e}")


# Blocks without 16-bit experts with 33 to 52 rows per expert: the projections that stay with the kernel for few rows, up and
# down, long and short ranges, chunks of every number of tiles.
ROWS = [30, 50, 64, 65, 1, 16, 17, 33, 48, 49, 0, 100, 80, 5, 128, 2]


@pytest.mark.parametrize("d,f,bits,up,down", [(4096, 3712, "q" * 16, 0, 4), (4096, 3712, "qe" * 8, 0, 4), (4096, 3712, "e" * 16, 0, 0),
                                              (1536, 1280, "q" * 16, 4, 0), (1536, 1280, "qe" * 8, 4, 0), (1536, 1280, "e" * 16, 4, 0),
                                              (3584, 1408, "q" * 32, 4, 0), (3584, 1408, "qe" * 16, 4, 0)])
def test_64_row_chunks_outside_the_prefill_kernel(weights, d, f, bits, up, down):
    experts, dense = weights(d, f, bits)
    rows = ROWS * (len(bits) // 16)
    form = launch_forms([PREC[b] for b in bits], d, f, 1, sum(rows))
    assert [(m.waves, m.ct, m.half, m.steps_per_stage) for m in form] == [(w, 4, 0, 0 if w else 1) for w in (up, down)]
    x, to, gate = _routed(torch.Generator(device="cuda").manual_seed(5), d, len(bits), rows)
    _check(d, f, gate, experts, dense, x, to)


def test_64_row_chunks_two_steps_per_stage(weights):
    """Long down-projections of few workgroups, all 8-bit: two 128-column steps per LDS stage; the same bits as in a block of
    more experts, which takes one."""
    d, f = 5376, 3712
    experts, dense = weights(d, f, "e" * 12)
    few, many = (launch_forms([mm.PREC_INT8G64] * E, d, f, 1, sum(ROWS[:E])) for E in (8, 12))
    assert [few[0].waves, many[0].waves] == [4, 4]
    assert [(m[1].waves, m[1].half, m[1].steps_per_stage, m[1].splits) for m in (few, many)] == [(0, 0, 2, 1), (0, 0, 1, 1)]
    x, to, gate = _routed(torch.Generator(device="cuda").manual_seed(5), d, 12, ROWS[:12])
    _check(d, f, gate, experts, dense, x, to)
    out, _ = _block(d, f, gate, experts, x)
    first = to < 8
    some, _ = _block(d, f, gate[:8].contiguous(), experts[:8], x[first].contiguous())
    assert torch.equal(some, out[first])
