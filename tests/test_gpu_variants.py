"""Kernel variants that a rule on sizes, types or alignment chooses between: each at the sizes where it can go wrong,
against the oracle or against the general path."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2407_14417_amd import binding as mm, synth
from tests import common
from tests.common import assert_ffn_close, build_workload, launch_forms
from tests.gpu_common import dev, device_layer

pytestmark = pytest.mark.gpu


# ---------------------------------------------------------------- quantizer: 128-bit loads against 2-byte loads

def _quantized(w, bits, shift=0, code_shift=0):
    """Codes, scales and zeros of `w`, read from an address `shift` halves past an aligned one; codes written
    `code_shift` bytes past one."""
    out, inn = w.shape
    buf = torch.zeros(out * inn + 8, dtype=torch.float16, device="cuda")
    src = buf[shift:shift + out * inn].view(out, inn)
    src.copy_(w)
    n = out * inn * bits // 8
    codes = torch.zeros(n + 8, dtype=torch.uint8, device="cuda")[code_shift:code_shift + n].view(out, -1)
    scale, zero = (torch.zeros((out, inn // 64), dtype=torch.float16, device="cuda") for _ in range(2))
    (mm.moe_quantize_int4 if bits == 4 else mm.moe_quantize_int8)(src, codes, scale, zero)
    return codes.cpu().numpy(), scale.cpu().numpy().view(np.uint16), zero.cpu().numpy().view(np.uint16)


def _grid_weights(out, inn):
    """Groups on a grid of half steps of their own scale (quotients that are ties: kind 1 for 4 bits, kind 7 for 8),
    with both zeros, subnormal, at the edge of fp16 or holding infinities and NaN."""
    rng = np.random.default_rng(5)
    w = synth.normal_f16((out, inn), 0.02, 4, 61).astype(np.float32).reshape(-1, 64)
    n = w.shape[0]
    for g in range(n):
        kind = g % 8
        if kind == 1:
            w[g] = (np.append(rng.integers(0, 31, 62), [0, 30]) * 0.5 - 3) * 2.0 ** rng.integers(-8, 3)
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
            w[g] = (np.append(rng.integers(0, 511, 62), [0, 510]) * 0.5) * 2.0 ** -10
    return w.astype(np.float16).reshape(out, inn)


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("shape", [(1, 64), (3, 64), (33, 2048), (8, 1024), (301, 1088)])
def test_quantizer_wide_loads_equal_narrow_loads(orc, bits, shape):
    for w in (synth.normal_f16(shape, 0.02, 4, 60), _grid_weights(*shape)):
        wide = _quantized(dev(w), bits)
        for narrow in (_quantized(dev(w), bits, shift=1), _quantized(dev(w), bits, code_shift=1),
                       _quantized(dev(w), bits, code_shift=bits // 2)):
            for a, b in zip(wide, narrow):
                assert np.array_equal(a, b)
        # against the definition: every group but those with infinities or NaN, or with both zeros (whose minimum is either)
        g = w.reshape(-1, 64)
        told = np.isfinite(g.astype(np.float32)).all(1) & ~((g.view(np.uint16) == 0).any(1) & (g.view(np.uint16) == 0x8000).any(1))
        assert told.sum() > told.size // 2
        tame = np.where(np.repeat(told, 64).reshape(shape), w, np.float16(1))
        ref = orc.quantize_int4(tame) if bits == 4 else orc.quantize_int8(tame)
        for a, b in zip(wide, (ref.data, ref.scale.view(np.uint16), ref.zero.view(np.uint16))):
            assert np.array_equal(a.reshape(told.size, -1)[told], np.asarray(b).reshape(told.size, -1)[told])


# ---------------------------------------------------------------- gating and grouping

def _routing_layer(wg, k):
    ex = [mm.Expert(mm.PREC_FP16, None, None, None, resident=False) for _ in range(wg.shape[0])]
    return mm.Layer(wg.shape[1], 64, k, dev(wg), ex)


@pytest.mark.parametrize("E,k,T", [(32, 8, 128), (32, 8, 129), (32, 1, 63), (1, 1, 65), (31, 7, 2341)])
def test_permute_runs_of_every_length(orc, E, k, T):
    """16 runs of whole groups of 64 pairs: exactly one group each, one more, a single ragged one, long runs."""
    rng = np.random.default_rng(E * 100 + T)
    idx = rng.integers(0, E, (T, k)).astype(np.int32) if T % 2 else np.sort(rng.integers(0, E, (T, k)), axis=0).astype(np.int32)
    layer = _routing_layer(np.zeros((E, 64), np.float16), k)
    ws = mm.alloc_workspace(layer, T)
    counts, offsets, perm = (torch.empty(n, dtype=torch.int32, device="cuda") for n in (E, E + 1, T * k))
    mm.moe_permute(layer, dev(idx), counts, offsets, perm, ws)
    for got, ref in zip((counts, offsets, perm), orc.permute(idx, E)):
        assert np.array_equal(got.cpu().numpy(), ref)
    assert mm.moe_read_status(ws) == 0


def _selection_passes(logits, k):
    """k passes over the logits, each taking the first of the largest that are left; a NaN never compares larger, so
    it is taken exactly when it is the first one left."""
    left, out = list(range(len(logits))), []
    for _ in range(k):
        best = left[0]
        for e in left[1:]:
            if logits[e] > logits[best]:
                best = e
        left.remove(best)
        out.append(best)
    return out


@pytest.mark.parametrize("T", [1, 3])
@pytest.mark.parametrize("d,E,k", [(64, 32, 8), (2048, 8, 2), (4160, 5, 3), (8192, 13, 4)])
def test_route_infinite_and_nan_logits(T, d, E, k):
    """Router rows with one non-zero column, so that every logit is one product: infinities, NaN and ties."""
    values = np.array([1.0, np.nan, -np.inf, 2.0, np.inf, 2.0, np.nan, -3.0], np.float16)
    wg = np.zeros((E, d), np.float16)
    wg[:, d - 1] = np.resize(values, E)
    x = np.zeros((T, d), np.float16)
    x[:, d - 1] = [1.0, -1.0, 0.5][:T]
    idx = torch.empty((T, k), dtype=torch.int32, device="cuda")
    gate = torch.empty((T, k), dtype=torch.float32, device="cuda")
    mm.moe_route(_routing_layer(wg, k), dev(x), idx, gate)
    for t in range(T):
        assert idx[t].tolist() == _selection_passes((x[t, d - 1].astype(np.float32) * wg[:, d - 1].astype(np.float32)).tolist(), k)


# ---------------------------------------------------------------- blocks

def _run_block(layer, x, k, ws=None):
    T, d = x.shape
    out = torch.full((T, d), float("nan"), dtype=torch.float16, device="cuda")
    idx = torch.empty((T, k), dtype=torch.int32, device="cuda")
    gate = torch.empty((T, k), dtype=torch.float32, device="cuda")
    ws = mm.alloc_workspace(layer, T) if ws is None else ws
    ws.fill_(0xFF)                                                # NaN wherever it is floats
    mm.moe_layer_forward(layer, dev(x), out, ws, idx, gate)
    assert mm.moe_read_status(ws) == 0
    return out.cpu().numpy(), idx.cpu().numpy(), gate.cpu().numpy()


def _check_block(orc, cfg):
    print(cfg.name, flush=True)
    wl = build_workload(cfg, orc)
    out, idx, gate = _run_block(device_layer(wl), wl.x, cfg.k)
    ref, ref_idx, ref_gate = orc.layer_forward(wl.x, wl.wg, wl.experts, cfg.k, bias=wl.bias)
    assert np.array_equal(idx, ref_idx)
    assert np.allclose(gate, ref_gate, rtol=0, atol=2e-6)
    assert_ffn_close(out, ref, cfg.name)


# Contractions that end with half a step of 128 columns (odd multiples of 64): in the up-projection, in the
# down-projection (one range of an odd and of an even number of steps, several ranges of which the last ends early),
# in both; 16, 32, 64 and 128 rows per chunk; every precision.
@pytest.mark.parametrize("d,f", [(320, 512), (512, 320), (448, 960), (320, 1472), (832, 2752), (8128, 256), (256, 16320)])
@pytest.mark.parametrize("T,zipf", [(2, None), (40, None), (75, 1.2), (150, None), (300, 2.0)])
def test_block_widths_of_odd_multiples_of_64(orc, d, f, T, zipf):
    if d * f > 500000 and T != 40:
        return
    _check_block(orc, common.Config(f"half_d{d}_f{f}_T{T}", d, f, 5, 2, T, (0, 3), zipf=zipf, int8_experts=(1, 4)))


# One workspace for several numbers of tokens: sized for more tokens than the call has, and exactly the unsplit call's
# bytes; nothing is written past either, and a byte less than that is refused.
@pytest.mark.parametrize("d,f,E,k,T,T_sized", [(1088, 3008, 8, 2, 39, 40), (832, 2752, 8, 2, 95, 96), (320, 512, 5, 2, 7, 40),
                                               (512, 2880, 4, 2, 1, 2)])
def test_workspace_sized_for_more_tokens(orc, d, f, E, k, T, T_sized):
    cfg = common.Config(f"ws_d{d}_f{f}_T{T}", d, f, E, k, T, tuple(range(0, E, 3)), int8_experts=tuple(range(1, E, 3)))
    wl = build_workload(cfg, orc)
    layer, x = device_layer(wl), dev(wl.x)
    ref, ref_idx, _ = orc.layer_forward(wl.x, wl.wg, wl.experts, k)
    least = common.unsplit_workspace_bytes(d, f, E, k, T)
    idx = torch.empty((T, k), dtype=torch.int32, device="cuda")
    for n in sorted({least, mm.workspace_bytes(layer, T_sized)}):
        room = torch.full((n + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
        out = torch.full((T, d), float("nan"), dtype=torch.float16, device="cuda")
        mm.moe_layer_forward(layer, x, out, room[:n], idx)
        assert mm.moe_read_status(room) == 0 and bool((room[n:] == 0xFF).all())
        assert np.array_equal(idx.cpu().numpy(), ref_idx)
        assert_ffn_close(out.cpu().numpy(), ref, f"{cfg.name} ws={n}")
        swap, swapped = mm.Swap(layer, [None] * E, 1, T), torch.full_like(out, float("nan"))
        assert mm.moe_layer_forward_swap(layer, swap, x, swapped, room[:n]) == 0
        assert torch.equal(swapped, out) and bool((room[n:] == 0xFF).all())
        h = torch.zeros_like(out)
        mm.moe_chain_forward(mm.Chain([layer], [torch.ones(d, dtype=torch.float16, device="cuda")]), 1e-5, h.copy_(x), room[:n])
        assert bool(torch.isfinite(h).all()) and bool((room[n:] == 0xFF).all())
    with pytest.raises(mm.MoeError) as refused:
        mm.moe_layer_forward(layer, x, out, room[:least - 1], idx)
    assert refused.value.code == mm.MOE_EWORKSPACE


def test_static_scratch_at_its_limit_odd_multiples_of_64(orc):
    """As many tokens as the library's own scratch holds unsplit, and where splits still fit: the same bits as with a
    workspace; one token more is refused."""
    d, f, E, k = 832, 2752, 8, 2
    most = max(T for T in range(1, 1000) if common.unsplit_workspace_bytes(d, f, E, k, T) <= mm.moe_static_scratch_bytes())
    cfg = common.Config("static_limit", d, f, E, k, most, (0, 3, 6), int8_experts=(1, 4, 7))
    wl = build_workload(cfg, orc)
    layer, x = device_layer(wl), dev(wl.x)
    for T in (most, 95, 96, 30):
        own, with_ws = (torch.full((T, d), float("nan"), dtype=torch.float16, device="cuda") for _ in range(2))
        mm.moe_layer_forward_static(layer, x[:T], own)
        mm.moe_layer_forward(layer, x[:T], with_ws, mm.alloc_workspace(layer, T))
        assert torch.equal(own, with_ws) and bool(torch.isfinite(own).all())
    more = torch.cat([x, x[:1]])
    with pytest.raises(mm.MoeError) as refused:
        mm.moe_layer_forward_static(layer, more, torch.empty_like(more))
    assert refused.value.code == mm.MOE_EWORKSPACE


# Contractions of whole steps beside a d_model of an odd multiple of 64, a workspace for fewer splits than the plan has: the
# ranges keep one length (20 rows alone and 40 tokens in chunks of up to 32 rows, the rest in prefill launches), an infinity at
# the start of a row of w2 stays in its output.
@pytest.mark.parametrize("T", [10, 40, 95])
def test_smaller_workspace_whole_steps(orc, T):
    d, f = 832, 2816
    cfg = common.Config(f"fewer_{T}", d, f, 4, 2, T, (0, 2), int8_experts=(1,))
    wl = build_workload(cfg, orc)
    layer = device_layer(wl)
    least, full = common.unsplit_workspace_bytes(d, f, 4, 2, T), mm.workspace_bytes(layer, T)
    ref, ref_idx, _ = orc.layer_forward(wl.x, wl.wg, wl.experts, 2)
    rows = np.concatenate([wl.x, wl.x])
    alone = [orc.expert_ffn(e, rows) for e in wl.experts]
    for n in sorted({least, full, *(least + s * 8 * T * d for s in (1, 2, 3, 5) if least + s * 8 * T * d < full)}):
        room = torch.full((n + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
        out, idx, _ = _run_block(layer, wl.x, 2, room[:n])
        assert np.array_equal(idx, ref_idx)
        assert_ffn_close(out, ref, f"{cfg.name} ws={n}")
        for e in range(4):
            y = torch.full((2 * T, d), float("nan"), dtype=torch.float32, device="cuda")
            mm.moe_expert_ffn_mixed(layer, e, dev(rows), y, room[:n])
            assert_ffn_close(y.cpu().numpy(), alone[e], f"{cfg.name} expert {e} ws={n}")
        layer.experts[3].w2.data[7, 0] = float("inf")
        mm.moe_expert_ffn_mixed(layer, 3, dev(rows), y, room[:n])
        layer.experts[3].w2.data[7, 0] = float(wl.experts[3].w2.data[7, 0])
        assert not torch.isfinite(y[:, 7]).any() and torch.isfinite(y[:, torch.arange(d, device="cuda") != 7]).all()
        assert bool((room[n:] == 0xFF).all())


# Up to 16 pairs: ranges of unequal length where the number of steps has no divisor (17, 19, 23, 67 steps, with and without
# half a step at the end, the last range of two and three steps), the same with a workspace for fewer splits and through
# one expert alone.
@pytest.mark.parametrize("d,f", [(704, 2112), (320, 2432), (512, 2880), (320, 8512), (448, 4672)])
@pytest.mark.parametrize("T", [2, 5, 8])
def test_uneven_splits(orc, d, f, T):
    cfg = common.Config(f"uneven_d{d}_f{f}_T{T}", d, f, 3, 2, T, (0,), int8_experts=(1,))
    wl = build_workload(cfg, orc)
    layer = device_layer(wl)
    least, full = common.unsplit_workspace_bytes(d, f, 3, 2, T), mm.workspace_bytes(layer, T)
    assert full > least
    ref, ref_idx, _ = orc.layer_forward(wl.x, wl.wg, wl.experts, 2)
    for n in (full, full - 256, (least + full) // 2, least):
        room = torch.full((n + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
        out, idx, _ = _run_block(layer, wl.x, 2, room[:n])
        assert bool((room[n:] == 0xFF).all())
        assert np.array_equal(idx, ref_idx)
        assert_ffn_close(out, ref, f"{cfg.name} ws={n}")
    for e in range(3):
        y = torch.full((T, d), float("nan"), dtype=torch.float32, device="cuda")
        mm.moe_expert_ffn_mixed(layer, e, dev(wl.x), y, mm.alloc_workspace(layer, T))
        assert_ffn_close(y.cpu().numpy(), orc.expert_ffn(wl.experts[e], wl.x), f"{cfg.name} expert {e}")


# Ranges of four steps of 7 and 19, which ask for scales 128 bits at a time where rows of scales start on 16-byte boundaries:
# these are 28 and 76 bytes apart.
@pytest.mark.parametrize("d,f,T,splits", [(320, 896, 4, 2), (576, 2432, 3, 5)])
def test_uneven_splits_of_whole_fours(orc, d, f, T, splits):
    down = common.launch_forms([mm.PREC_INT4G64] * 3, d, f, 1, T)[1]
    assert (down.half, down.ct, down.splits, down.steps_per_split) == (0, 1, splits, 4)
    cfg = common.Config(f"fours_d{d}_f{f}_T{T}", d, f, 3, 1, T, (0, 1, 2))
    wl = build_workload(cfg, orc)
    ref, ref_idx, _ = orc.layer_forward(wl.x, wl.wg, wl.experts, 1)
    out, idx, _ = _run_block(device_layer(wl), wl.x, 1)
    assert np.array_equal(idx, ref_idx)
    assert_ffn_close(out, ref, cfg.name)


@pytest.mark.parametrize("bits", [4, 8, 16])
def test_half_step_keeps_neighbours_apart(orc, bits):
    """A row's end is the next row's start in memory: infinities at the start of a token, of a hidden row and of a
    weight row stay with their token and their output column."""
    d, f, T = 320, 448, 6
    quant = {4: dict(int4_experts=(0,)), 8: dict(int4_experts=(), int8_experts=(0,)), 16: dict(int4_experts=())}[bits]
    wl = build_workload(common.Config("half_inf", d, f, 1, 1, T, **quant), orc)
    layer = device_layer(wl)
    clean = _run_block(layer, wl.x, 1)[0]
    x = wl.x.copy()
    x[3, 0] = np.inf
    got = _run_block(layer, x, 1)[0]
    keep = np.arange(T) != 3
    assert np.array_equal(got[keep], clean[keep]) and not np.isfinite(got[3]).all()
    w2 = layer.experts[0].w2
    (w2.data if bits == 16 else w2.scale)[7, 0] = float("inf")
    got = _run_block(layer, wl.x, 1)[0]
    cols = np.arange(d) != 7
    assert np.array_equal(got[:, cols], clean[:, cols]) and not np.isfinite(got[:, 7]).any()


# One 8-bit expert alone with more than 64 rows, on workgroups of 4 wavefronts: chunks of up to 128 rows, ragged last tiles, the
# one-tile rest, ranges of 8 steps (up) and of splits of 4 steps (down).
@pytest.mark.parametrize("n", [70, 81, 96, 100, 128, 129, 150, 170, 185, 200, 225, 250, 257])
def test_expert_ffn_8bit_pipelined_body(orc, n):
    cfg = common.Config("steps4_8bit", 1024, 2048, 2, 1, 4, (), int8_experts=(0, 1))
    wl = build_workload(cfg, orc)
    layer = device_layer(wl)
    x = synth.normal_f16((n, cfg.d), 1.0, 9, 77)
    y = torch.full((n, cfg.d), float("nan"), dtype=torch.float32, device="cuda")
    ws = mm.alloc_workspace(layer, n)
    mm.moe_expert_ffn_mixed(layer, 1, dev(x), y, ws)
    assert mm.moe_read_status(ws) == 0
    assert_ffn_close(y.cpu().numpy(), orc.expert_ffn(wl.experts[1], x), f"n={n}")


@pytest.mark.parametrize("T", [139, 150, 170, 185, 200, 215, 230, 256, 257])
@pytest.mark.parametrize("bits", [4, 8])
def test_block_quantized_chunks_in_small_launches(orc, T, bits):
    """Both experts take every token; few workgroups, of 4 wavefronts: chunks of 128 rows and a rest."""
    assert [m.waves for m in launch_forms([mm.PREC_INT4G64 if bits == 4 else mm.PREC_INT8G64] * 2, 1024, 2048, 2, T)] == [4, 4]
    _check_block(orc, common.Config(f"steps4_{bits}bit_T{T}", 1024, 2048, 2, 2, T, (0, 1) if bits == 4 else (),
                                    int8_experts=(0, 1) if bits == 8 else ()))


def _rows_per_chunk(n, E, columns):
    """The library's rule for blocks in which every token reaches all E quantized experts (n rows each), with `columns`
    workgroups per chunk."""
    up = lambda a, b: -(-a // b)
    if columns * E * up(n, 128) <= 256:
        return 128
    best = None
    for cap in (256, 192, 128):
        cost = up(columns * E * up(n, cap), 256) * (40 + 7 * up(n // up(n, cap), 16))
        if best is None or 20 * cost < 19 * best[1]:
            best = cap, cost
    return best[0]


# Launches of more workgroups (in both projections): one chunk of 9 to 16 tiles, two of 9, and five of 10.
@pytest.mark.parametrize("d,f,T,rows", [*((2048, 11264, T, 256) for T in (139, 150, 170, 185, 200, 215, 230, 256, 257)),
                                        (1024, 5120, 800, 192)])
@pytest.mark.parametrize("bits", [4, 8])
def test_block_quantized_chunks_of_more_than_128_rows(d, f, T, rows, bits):
    """Both experts take every token.  Weights are drawn and quantized on the device; the reference is a float64 product
    with the dequantized ones."""
    splits = 11 if f == 11264 else 10
    assert _rows_per_chunk(T, 2, f // 128) == _rows_per_chunk(T, 2, d // 256 * splits) == rows
    form = launch_forms([mm.PREC_INT4G64 if bits == 4 else mm.PREC_INT8G64] * 2, d, f, 2, T)
    assert [(m.waves, m.quant_rows) for m in form] == [(8, rows)] * 2 and form[1].splits == splits
    gen = torch.Generator(device="cuda").manual_seed(T)
    draw = lambda shape, sigma: torch.empty(shape, dtype=torch.float16, device="cuda").normal_(0.0, sigma, generator=gen)
    experts, dense = [], []
    for _ in range(2):
        mats = []
        for o, i in ((f, d), (f, d), (d, f)):
            codes = torch.empty((o, i * bits // 8), dtype=torch.uint8, device="cuda")
            scale, zero = (torch.empty((o, i // 64), dtype=torch.float16, device="cuda") for _ in range(2))
            w = draw((o, i), 0.02)
            (mm.moe_quantize_int4 if bits == 4 else mm.moe_quantize_int8)(w, codes, scale, zero)
            mats.append(mm.Mat(codes, scale, zero))
            (mm.moe_dequant_int4 if bits == 4 else mm.moe_dequant_int8)(mats[-1], o, i, w)
            dense.append(w)
        experts.append(mm.Expert(mm.PREC_INT4G64 if bits == 4 else mm.PREC_INT8G64, *mats))
    x = draw((T, d), 1.0)
    out, idx, gate = _run_block(mm.Layer(d, f, 2, draw((2, d), 0.02), experts), x.cpu().numpy(), 2)
    ref = np.zeros((T, d))
    for e in range(2):
        w1, w3, w2 = (w.double() for w in dense[3 * e:3 * e + 3])
        a = x.double() @ w1.t()
        y = (torch.nn.functional.silu(a) * (x.double() @ w3.t())) @ w2.t()
        ref += (gate * (idx == e)).sum(1, dtype=np.float64)[:, None] * y.cpu().numpy()
    assert_ffn_close(out, ref, f"{bits}-bit T={T}")


# One token at widths that are no multiple of 2048: rows shorter than a wavefront's loads, one load per lane exactly,
# ragged last ones, up to the limits; one, two, three and four or more loads per lane and row in both kernels; few and
# many experts and slots; every precision; the RMSNorm of the chain; one expert alone.
@pytest.mark.parametrize("d,f,E,k", [(64, 64, 3, 2), (192, 320, 4, 2), (1024, 2816, 8, 2), (1088, 3008, 5, 3), (512, 1536, 1, 1),
                                     (2048, 1408, 32, 8), (2112, 960, 6, 4), (4160, 1024, 3, 2), (8192, 192, 2, 1),
                                     (128, 16320, 2, 2), (2880, 2880, 4, 2)])
def test_one_token_any_width(orc, d, f, E, k):
    for seed in range(3):
        low = tuple(range(seed, E, 3))
        _check_block(orc, common.Config(f"one_token_d{d}_f{f}_E{E}_k{k}_{seed}", d, f, E, k, 1, low, seed=seed,
                                        int8_experts=tuple(range((seed + 1) % 3, E, 3)), zipf=1.2 if seed == 1 else None))


@pytest.mark.parametrize("d,f", [(192, 320), (1088, 3008), (2880, 960)])
@pytest.mark.parametrize("bits", [4, 8, 16])
def test_one_row_any_width(orc, d, f, bits):
    """One expert alone; the 16-bit one with most of w2 subnormal (sums of products that are not flushed)."""
    quant = {4: dict(int4_experts=(0,)), 8: dict(int4_experts=(), int8_experts=(0,)), 16: dict(int4_experts=())}[bits]
    wl = build_workload(common.Config(f"one_row_{bits}", d, f, 1, 1, 1, **quant), orc)
    if bits == 16:
        wl.experts[0].w2.data[:] = (wl.experts[0].w2.data.astype(np.float32) * 1e-3).astype(np.float16)
    layer = device_layer(wl)
    y = torch.full((1, d), float("nan"), dtype=torch.float32, device="cuda")
    ws = mm.alloc_workspace(layer, 1)
    mm.moe_expert_ffn_mixed(layer, 0, dev(wl.x), y, ws)
    assert mm.moe_read_status(ws) == 0
    assert_ffn_close(y.cpu().numpy(), orc.expert_ffn(wl.experts[0], wl.x), f"d={d} f={f} bits={bits}")


@pytest.mark.parametrize("d,f", [(192, 320), (1024, 2816), (2880, 960)])
@pytest.mark.parametrize("bits", [4, 8, 16])
def test_one_token_hidden_value_past_the_fp16_range(orc, d, f, bits):
    """One hidden value beyond 65504 is an infinity: every output is that infinity with the sign of its weight, as in
    the multi-token kernels, and no NaN."""
    cfg = common.Config("overflow", d, f, 1, 1, 1, ())
    wl = build_workload(cfg, orc)
    w1, w3, w2 = common.expert_weights_f16(cfg, 0)
    big = f - 5                                                   # in the last pieces of a hidden row
    w1[big] = w3[big] = np.where(wl.x[0] < 0, -4, 4)
    w2[:, big] = np.where(np.arange(d) % 3 == 0, -0.05, 0.05)     # (no dequantized weight there is zero)
    stored = {4: orc.quantize_int4, 8: orc.quantize_int8, 16: orc.Mat}[bits]
    wl.experts[0] = orc.Expert(stored(w1), stored(w3), stored(w2))
    layer = device_layer(wl)
    want = np.where(np.arange(d) % 3 == 0, -np.inf, np.inf)
    assert np.array_equal(_run_block(layer, wl.x, 1)[0][0].astype(np.float64), want)
    y = torch.empty((1, d), dtype=torch.float32, device="cuda")
    mm.moe_expert_ffn_mixed(layer, 0, dev(wl.x), y, mm.alloc_workspace(layer, 1))
    assert np.array_equal(y.cpu().numpy()[0].astype(np.float64), want)
    assert np.array_equal(_run_block(layer, np.repeat(wl.x, 2, axis=0), 1)[0][0].astype(np.float64), want)   # two tokens


@pytest.mark.parametrize("d,f", [(192, 320), (1024, 2816), (2880, 960)])
@pytest.mark.parametrize("bits", [4, 8])
def test_one_token_infinite_scale_or_zero(orc, d, f, bits):
    """A group whose scale or zero is not finite: one token gives infinities and NaN where the multi-token kernels give
    them, and leaves the other outputs' bits alone."""
    every = dict(int4_experts=(0,)) if bits == 4 else dict(int4_experts=(), int8_experts=(0,))
    wl = build_workload(common.Config("inf_group", d, f, 1, 1, 1, **every), orc)
    layer = device_layer(wl)
    clean = _run_block(layer, wl.x, 1)[0]
    for mat, what, row, value in [("w2", "scale", 7, np.inf), ("w2", "zero", 7, np.nan), ("w2", "zero", 7, -np.inf),
                                  ("w1", "scale", f - 1, np.inf), ("w3", "scale", 0, np.inf)]:
        t = getattr(getattr(layer.experts[0], mat), what)
        kept, t[row, -1] = t[row, -1].clone(), float(value)
        one, two = _run_block(layer, wl.x, 1)[0][0], _run_block(layer, np.repeat(wl.x, 2, axis=0), 1)[0][0]
        t[row, -1] = kept
        for kind in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(kind(one), kind(two)), (mat, what, value)
        assert not np.isfinite(one[7]) and np.array_equal(one[np.isfinite(one)], clean[0][np.isfinite(one)])


def test_one_token_any_width_non_resident_and_chain(orc):
    cfg = common.Config("one_token_chain", 1088, 1472, 6, 2, 1, (0, 3), int8_experts=(1,))
    wl = build_workload(cfg, orc)
    layer = device_layer(wl)
    gain = synth.uniform_f16((cfg.d,), 1.0, 3, 90)
    h = synth.normal_f16((1, cfg.d), 1.0, 3, 91)
    got = dev(h).clone()
    idx = torch.empty((2, 1, 2), dtype=torch.int32, device="cuda")
    ws = mm.alloc_workspace(layer, 1)
    mm.moe_chain_forward(mm.Chain([layer, layer], [dev(gain), dev(gain)]), 1e-5, got, ws, idx)
    ref = h
    for l in range(2):
        ref, ref_idx = orc.chain_layer(ref, gain, 1e-5, wl.wg, wl.experts, cfg.k)[:2]
        assert np.array_equal(idx[l].cpu().numpy(), ref_idx)
        ref = ref.astype(np.float16)
    assert_ffn_close(got.cpu().numpy(), ref, "chain")
    assert mm.moe_read_status(ws) == 0
    first = int(idx[0, 0, 0])
    x = wl.x
    _, ref_idx, ref_gate = orc.layer_forward(x, wl.wg, wl.experts, cfg.k)
    gone, kept = int(ref_idx[0, 0]), int(ref_idx[0, 1])
    experts = list(layer.experts)
    experts[gone] = mm.Expert(experts[gone].prec, None, None, None, resident=False)
    part = mm.Layer(cfg.d, cfg.f, cfg.k, layer.w_gate, experts)
    out = torch.empty((1, cfg.d), dtype=torch.float16, device="cuda")
    mm.moe_layer_forward(part, dev(x), out, ws)
    assert mm.moe_read_status(ws) == mm.STATUS_NOT_RESIDENT
    assert_ffn_close(out.cpu().numpy(), ref_gate[0, 1] * orc.expert_ffn(wl.experts[kept], x), "non-resident")


# Few pairs: the grouping worked out inside the launches against the grouping launch (which runs when its kernel is to be
# measured): one, two and four registers of pairs, all full or ragged, one and two tiles per chunk, several chunks per
# expert, experts without tokens.
@pytest.mark.parametrize("T,E,k,zipf,d,f", [(2, 8, 2, None, 256, 384), (32, 8, 2, None, 512, 1408), (33, 8, 2, 2.0, 512, 1408),
                                            (64, 16, 4, 1.2, 256, 512), (128, 8, 2, 1.2, 384, 640), (33, 9, 7, None, 320, 448),
                                            (29, 32, 8, 1.2, 256, 2816), (5, 8, 2, None, 1024, 14336)])
def test_grouping_inside_the_launches(orc, T, E, k, zipf, d, f):
    cfg = common.Config(f"inline_T{T}_E{E}_k{k}", d, f, E, k, T, tuple(range(0, E, 2)), zipf=zipf, int8_experts=(1,))
    wl = build_workload(cfg, orc)
    layer = device_layer(wl)
    ws = mm.alloc_workspace(layer, T)
    routing = 256 + 2 * ((4 * T * k + 255) // 256 * 256)         # status word, experts, weights; then what the launch groups into
    grouped = ws[routing:routing + 2 * 256 + (4 * T * k + 255) // 256 * 256]
    inside = _run_block(layer, wl.x, k, ws)
    assert bool((grouped == 0xFF).all())                          # no grouping launch has run
    start, stop = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    start.record(), stop.record()
    mm.moe_trace_kernel(mm.KERNEL_PERMUTE, start.cuda_event, stop.cuda_event)
    apart = _run_block(layer, wl.x, k, ws)
    torch.cuda.synchronize()
    assert start.elapsed_time(stop) > 0 and not bool((grouped == 0xFF).all())
    for a, b in zip(inside, apart):
        assert np.array_equal(a, b)
    ref, ref_idx, _ = orc.layer_forward(wl.x, wl.wg, wl.experts, k, bias=wl.bias)
    assert np.array_equal(inside[1], ref_idx)
    assert_ffn_close(inside[0], ref, cfg.name)


# Launches with 128-row chunks hand out the longest workgroups first: experts with no, few, equal and most rows in an
# order of sizes and precisions that is not the order of their indices, every chunk found exactly once.
@pytest.mark.parametrize("E,k,T,bias", [(8, 2, 600, [0, 3, -9, 1, 3, 0, -9, 2]), (32, 8, 300, list(range(32))), (3, 3, 200, [0, 0, 0]),
                                        (5, 1, 700, [-9, 4, -9, 4, 0])])
@pytest.mark.parametrize("d,f", [(1024, 2048), (384, 640)])
def test_chunks_handed_out_by_length(orc, E, k, T, bias, d, f):
    cfg = common.Config(f"lpt_E{E}_T{T}_d{d}", d, f, E, k, T, tuple(range(0, E, 3)), int8_experts=tuple(range(2, E, 3)))
    wg = common.gate_matrix(cfg)
    gate_bias = np.array(bias, np.float32)
    x = common.tokens_with_margin(cfg, wg, gate_bias)
    wl = build_workload(cfg, orc)
    wl.x, wl.bias = x, gate_bias
    out, idx, _ = _run_block(device_layer(wl), x, k)
    ref, ref_idx, _ = orc.layer_forward(x, wg, wl.experts, k, bias=gate_bias)
    assert np.array_equal(idx, ref_idx)
    assert_ffn_close(out, ref, cfg.name)


# 33 to 64 rows per expert, launches of up to one and a half rounds of workgroups: blocks without 16-bit experts run what blocks
# with some run (workgroups of 4 wavefronts), and give the same bits as beside a 16-bit expert that no token reaches.
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("d,f,T", [(640, 896, 140), (1024, 2048, 200), (384, 1536, 256), (1408, 1536, 140), (1408, 5632, 140)])
def test_block_64_row_chunks_without_16bit_experts(orc, bits, d, f, T):
    every = tuple(range(8))
    prec = mm.PREC_INT4G64 if bits == 4 else mm.PREC_INT8G64
    for last in (prec, mm.PREC_FP16):
        assert [(m.waves, m.ct) for m in launch_forms([prec] * 7 + [last], d, f, 2, T)] == [(4, 4)] * 2
    cfg = common.Config(f"rows64_{bits}_{d}_{T}", d, f, 8, 2, T, every if bits == 4 else (), int8_experts=every if bits == 8 else ())
    wl = build_workload(cfg, orc)
    wl.bias = np.array([0, 0, 0, 0, 0, 0, 0, -50.0], np.float32)
    wl.x = common.tokens_with_margin(cfg, wl.wg, wl.bias)
    layer = device_layer(wl)
    out, idx, _ = _run_block(layer, wl.x, 2)
    ref, ref_idx, _ = orc.layer_forward(wl.x, wl.wg, wl.experts, 2, bias=wl.bias)
    assert np.array_equal(idx, ref_idx) and not (idx == 7).any()
    assert_ffn_close(out, ref, cfg.name)
    w1, w3, w2 = (mm.Mat(dev(w)) for w in common.expert_weights_f16(cfg, 7))
    beside = mm.Layer(d, f, 2, layer.w_gate, [*layer.experts[:7], mm.Expert(mm.PREC_FP16, w1, w3, w2)], layer.gate_bias)
    assert np.array_equal(out, _run_block(beside, wl.x, 2)[0])


# ---------------------------------------------------------------- prefill launches

# Workgroups of 4 wavefronts: chunks of 5 to 8 tiles with their ragged last one, rests of 1 to 8, tiles of weight rows that end
# past the matrix, contractions from two steps (shorter than the LDS rings are deep) to eleven, several splits; every token
# reaches an expert of each precision.  (8 wavefronts: test_gpu_prefill.py.)
@pytest.mark.parametrize("T", [65, 80, 81, 97, 113, 127, 128, 129, 145, 161, 177, 193, 209, 225, 241, 256, 257])
@pytest.mark.parametrize("d,f", [(256, 384), (640, 256), (384, 1408)])
def test_prefill_tiles_and_steps(orc, d, f, T):
    assert [m.waves for m in launch_forms([mm.PREC_INT4G64, mm.PREC_INT8G64, mm.PREC_FP16], d, f, 3, T)] == [4, 4]
    _check_block(orc, common.Config(f"prefill_{d}_{f}_{T}", d, f, 3, 3, T, (0,), int8_experts=(1,)))


@pytest.mark.parametrize("shift", [1, 4])
def test_prefill_tokens_off_16_byte_boundaries(orc, shift):
    """Tokens may lie anywhere: those that no 16-byte transfer can fetch give the same result."""
    cfg = common.Config(f"prefill_shift{shift}", 512, 896, 3, 2, 150, (0,), int8_experts=(1,))
    wl = build_workload(cfg, orc)
    layer, n = device_layer(wl), cfg.T * cfg.d
    x = torch.empty(n + 8, dtype=torch.float16, device="cuda")[shift:shift + n].view(cfg.T, cfg.d)
    x.copy_(dev(wl.x))
    out = torch.empty((cfg.T, cfg.d), dtype=torch.float16, device="cuda")
    idx = torch.empty((cfg.T, 2), dtype=torch.int32, device="cuda")
    gate = torch.empty((cfg.T, 2), dtype=torch.float32, device="cuda")
    ws = mm.alloc_workspace(layer, cfg.T)
    mm.moe_layer_forward(layer, x, out, ws, idx, gate)
    assert mm.moe_read_status(ws) == 0
    ref, ref_idx, _ = orc.layer_forward(wl.x, wl.wg, wl.experts, 2)
    assert np.array_equal(idx.cpu().numpy(), ref_idx)
    assert_ffn_close(out.cpu().numpy(), ref, cfg.name)


# Where tokens lie decides neither the launch nor the order of its sums: blocks, the expert-miss path and one expert alone of
# 33 to 64 rows, of more, and of few (which are read from where they are), tokens of eight steps (walked from different places).
@pytest.mark.parametrize("T", [20, 60, 150, 400])
@pytest.mark.parametrize("shift", [1, 2, 4, 7])
def test_same_bits_wherever_tokens_lie(T, shift):
    d, f, E = 1024, 4352, 3
    gen = torch.Generator(device="cuda").manual_seed(T)
    draw = lambda shape, sigma: torch.empty(shape, dtype=torch.float16, device="cuda").normal_(0.0, sigma, generator=gen)
    experts, hosts = [], []
    for bits in (16, 4, 8):
        mats = []
        for o, i in ((f, d), (f, d), (d, f)):
            w = draw((o, i), 0.02)
            if bits < 16:
                codes = torch.empty((o, i * bits // 8), dtype=torch.uint8, device="cuda")
                scale, zero = (torch.empty((o, i // 64), dtype=torch.float16, device="cuda") for _ in range(2))
                (mm.moe_quantize_int4 if bits == 4 else mm.moe_quantize_int8)(w, codes, scale, zero)
            mats.append(mm.Mat(w) if bits == 16 else mm.Mat(codes, scale, zero))
        experts.append(mm.Expert({16: mm.PREC_FP16, 4: mm.PREC_INT4G64, 8: mm.PREC_INT8G64}[bits], *mats))
    wg, x = draw((E, d), 0.02), draw((T, d), 1.0)
    layer = mm.Layer(d, f, 2, wg, experts)
    off = torch.empty(T * d + 8, dtype=torch.float16, device="cuda")[shift:shift + T * d].view(T, d)
    off.copy_(x)
    assert off.data_ptr() % 16 and not x.data_ptr() % 16

    def block(tokens):
        out, ws = torch.full((T, d), float("nan"), dtype=torch.float16, device="cuda"), mm.alloc_workspace(layer, T)
        mm.moe_layer_forward(layer, tokens, out, ws)
        return out

    assert torch.equal(block(x), block(off)) and bool(torch.isfinite(block(off)).all())
    for e in range(E):
        ws = mm.alloc_workspace(layer, (T + 1) // 2).fill_(0xFF)
        a, b = (torch.full((T, d), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
        mm.moe_expert_ffn_mixed(layer, e, x, a, ws)
        mm.moe_expert_ffn_mixed(layer, e, off, b, ws)
        assert torch.equal(a, b) and bool(torch.isfinite(b).all()), e
    pinned = [mm.Mat(*(None if t is None else t.cpu().pin_memory() for t in (m.data, m.scale, m.zero)))
              for m in (experts[1].w1, experts[1].w3, experts[1].w2)]
    part = mm.Layer(d, f, 2, wg, [experts[0], mm.Expert(mm.PREC_INT4G64, None, None, None, resident=False), experts[2]])
    swap = mm.Swap(part, [None, mm.Expert(mm.PREC_INT4G64, *pinned, resident=False), None], 1, T)
    out = torch.full((T, d), float("nan"), dtype=torch.float16, device="cuda")
    assert mm.moe_layer_forward_swap(part, swap, off, out, mm.alloc_workspace(part, T)) == 1
    assert torch.equal(out, block(x))


# Rows per expert on either side of the lines between launches (13, 16, 27, 32, 50, 68, 80 on average): chunks of one and two
# tiles, workgroups of 4 and of 8 wavefronts; loads spread about their mean, a skewed one; two steps up, 33 down.
@pytest.mark.parametrize("T,zipf", [(52, None), (64, None), (108, None), (128, None), (200, None), (272, None), (320, None), (320, 1.2)])
def test_block_at_the_lines_between_launches(orc, T, zipf):
    _check_block(orc, common.Config(f"lines_{T}", 256, 4224, 8, 2, T, (0, 3, 6), zipf=zipf, int8_experts=(1, 4)))
