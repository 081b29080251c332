"""Launches of grouped products in which the wavefronts of a workgroup share its contraction range in teams, each asked from
the library before it is run, against the oracle."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from paper_2407_14417_amd import binding as mm
from tests import common
from tests.common import assert_ffn_close, build_workload
from tests.gpu_common import dev, device_layer, device_layer_with_offloaded

PREC = {"h": mm.PREC_FP16, "q": mm.PREC_INT4G64, "e": mm.PREC_INT8G64}


def launch_teams(bits, d, f, k, n, expert=-1, ws_bytes=1 << 40):
    """Teams per workgroup in the up- and the down-projection, as the library itself says (host only)."""
    experts = (mm.CExpert * len(bits))()
    for e, b in zip(experts, bits):
        e.prec, e.resident = PREC[b], 1
        for m in (e.w1, e.w3, e.w2):
            m.data = m.scale = m.zero = 4096
    layer = mm.CLayer(d, f, len(bits), k, 4096, None, experts)
    teams = (ctypes.c_int * 2)()
    fn = mm.lib().moemix_launch_teams
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_size_t, ctypes.c_void_p]
    assert fn(ctypes.byref(layer), expert, n, ws_bytes, teams) == 0, mm.lib().moe_last_error()
    return tuple(teams)


def _config(bits, d, f, k, T):
    pick = lambda c: tuple(i for i, b in enumerate(bits) if b == c)
    return common.Config(f"teams_{bits}_{d}_{f}_{k}_{T}", d, f, len(bits), k, T, pick("q"), int8_experts=pick("e"))


# Contractions whose parts are whole fours of steps, pairs with a shorter or an odd last one, and end with half a step; tiles of
# weight rows that end past the matrix; chunks of one and two tiles, full and ragged; the three precisions, alone and mixed.
CASES = [
    ("qqq", 2048, 256, 2, 6, (4, 1)), ("hqe", 1792, 384, 2, 5, (4, 1)), ("eee", 2944, 320, 1, 9, (4, 1)),
    ("hhh", 2624, 512, 2, 7, (4, 1)), ("hhh", 1344, 512, 2, 7, (2, 1)), ("qqe", 1088, 704, 3, 4, (2, 1)),
    ("qhqe", 256, 2944, 2, 13, (1, 4)), ("qqqq", 320, 2880, 1, 17, (1, 4)), ("qqqq", 256, 3968, 1, 34, (1, 4)),
    ("eeh", 576, 2944, 3, 15, (1, 4)), ("hh", 512, 6016, 1, 9, (2, 4)), ("qqqq", 512, 512, 2, 2, (2, 1)),
    ("hhhh", 640, 1408, 2, 8, (1, 2)), ("hhh", 256, 2176, 2, 20, (1, 2)), ("qqq", 256, 2944, 3, 24, (1, 4)),
    ("hhe", 320, 2368, 3, 22, (1, 2)), ("qqq", 1152, 640, 2, 40, (2, 1)), ("heq", 960, 832, 2, 47, (2, 2)),
    ("qqqqqqqq", 1024, 1408, 2, 24, (2, 2)), ("qqq", 2048, 256, 3, 25, (4, 1)), ("ee", 1856, 384, 2, 31, (4, 1)),
    ("eqe", 1920, 256, 1, 60, (4, 1)), ("qq", 256, 3968, 2, 20, (1, 4)), ("qqqqq", 2048, 1280, 4, 28, (2, 1)),
    ("qqqqq", 1920, 1664, 4, 28, (1, 2)),
    # odd multiples of 64 take as many teams as the whole steps they round up to; the last team's part is a step and a half
    ("qqq", 704, 256, 2, 4, (2, 1)), ("qqq", 768, 256, 2, 4, (2, 1)), ("heq", 960, 256, 2, 4, (4, 1)), ("heq", 1024, 256, 2, 4, (4, 1)),
    ("hhe", 704, 256, 2, 20, (2, 1)), ("qqe", 960, 256, 2, 22, (4, 1)),
]


@pytest.mark.parametrize("bits,d,f,k,T,teams", CASES)
def test_rule(bits, d, f, k, T, teams):
    assert launch_teams(bits, d, f, k, T) == teams


# Teams of the up-projection on either side of the rule's lines, which count chunks as an even load makes them: of two tiles, where the
# mean is near a chunk and many experts have two (8 experts, mean of 31 rows: 11 chunks); of one tile, where few rows
# reach nearly every expert (36 pairs over 10 experts: 10 chunks).  And one workgroup per compute unit.
@pytest.mark.parametrize("bits,d,f,k,T,up", [
    ("q" * 8, 2048, 896, 1, 248, 1), ("q" * 8, 2048, 640, 1, 248, 2), ("q" * 8, 2048, 896, 1, 152, 2), ("q" * 16, 2048, 448, 2, 240, 1),
    ("h" * 8, 2048, 768, 1, 248, 1), ("q" * 10, 896, 2688, 4, 9, 1), ("q" * 10, 896, 2176, 4, 9, 2), ("h" * 10, 896, 1600, 4, 9, 1),
    ("h" * 10, 896, 1536, 4, 9, 2), ("q" * 8, 2048, 512, 2, 32, 4), ("q" * 8, 2048, 576, 2, 32, 2),
    ("q" * 5, 4160, 832, 2, 8, 2),   # (13 columns of 4.9 chunks: 65 workgroups)
])
def test_rule_counts_chunks(bits, d, f, k, T, up):
    assert launch_teams(bits, d, f, k, T)[0] == up


@pytest.mark.gpu
@pytest.mark.parametrize("bits,d,f,k,T,teams", CASES)
def test_block(orc, bits, d, f, k, T, teams):
    assert launch_teams(bits, d, f, k, T) == teams
    cfg = _config(bits, d, f, k, T)
    wl = build_workload(cfg, orc)
    layer = device_layer(wl)
    x, idx = dev(wl.x), torch.empty((T, k), dtype=torch.int32, device="cuda")
    out, gate = torch.empty_like(x), torch.empty((T, k), dtype=torch.float32, device="cuda")
    ws = mm.alloc_workspace(layer, T)
    for _ in range(2):
        out.fill_(float("nan"))
        mm.moe_layer_forward(layer, x, out, ws, idx, gate)
        ref, ref_idx, _ = orc.layer_forward(wl.x, wl.wg, wl.experts, k)
        assert np.array_equal(idx.cpu().numpy(), ref_idx)
        assert_ffn_close(out.cpu().numpy(), ref, cfg.name)
    assert mm.moe_read_status(ws) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("bits,d,f,n,teams", [("qqq", 2048, 256, 6, (4, 1)), ("hhh", 2048, 2944, 12, (4, 4)), ("eee", 1856, 1408, 20, (4, 2)), ("hhh", 1856, 1408, 20, (2, 2))])
def test_one_expert_alone(orc, bits, d, f, n, teams):
    assert launch_teams(bits, d, f, 2, n, expert=1) == teams
    wl = build_workload(_config(bits, d, f, 2, n), orc)
    layer, y = device_layer(wl), torch.full((n, d), float("nan"), device="cuda")
    mm.moe_expert_ffn_mixed(layer, 1, dev(wl.x), y, mm.alloc_workspace(layer, n))
    assert_ffn_close(y.cpu().numpy(), orc.expert_ffn(wl.experts[1], wl.x), f"{bits} n={n}")


def _forward(layer, x, k, ws=None):
    out = torch.full_like(x, float("nan"))
    idx = torch.empty((x.shape[0], k), dtype=torch.int32, device="cuda")
    ws = mm.alloc_workspace(layer, x.shape[0]) if ws is None else ws
    ws.fill_(0xFF)                                                # NaN wherever it is floats
    mm.moe_layer_forward(layer, x, out, ws, idx)
    return out.cpu().numpy(), idx.cpu().numpy(), mm.moe_read_status(ws)


@pytest.mark.gpu
@pytest.mark.parametrize("bits,d,f,k,T,teams", [("qheq", 1024, 2944, 2, 6, (2, 4)), ("qqqq", 2048, 256, 2, 6, (4, 1)), ("qeqe", 2048, 1408, 1, 70, (2, 2)),
                                                ("qqee", 1024, 3968, 2, 34, (1, 4))])
def test_missing_expert_is_left_out(orc, bits, d, f, k, T, teams):
    """Every tile of a missing expert's rows is zero, whatever the workspace held, in tiles of a half and a quarter of the rows."""
    assert launch_teams(bits, d, f, k, T) == teams
    cfg = _config(bits, d, f, k, T)
    wl = build_workload(cfg, orc)
    ref_idx, ref_gate = orc.route(wl.x, wl.wg, k)
    victim = int(np.bincount(ref_idx.reshape(-1)).argmax())
    layer = device_layer(wl)
    layer.experts[victim].resident = False
    layer = mm.Layer(d, f, k, layer.w_gate, layer.experts)
    out, idx, status = _forward(layer, dev(wl.x), k)
    assert status == mm.STATUS_NOT_RESIDENT and np.array_equal(idx, ref_idx)
    ref = np.zeros((T, d))
    for e in set(range(len(bits))) - {victim}:
        t, s = np.nonzero(ref_idx == e)
        if t.size:
            ref[t] += ref_gate[t, s][:, None].astype(np.float64) * orc.expert_ffn(wl.experts[e], wl.x[t])
    assert_ffn_close(out, ref, cfg.name)
    assert not out[(ref_idx == victim).all(axis=1)].any()


@pytest.mark.gpu
@pytest.mark.parametrize("bits,d,f,k,T,teams", [("qheq", 1024, 2944, 2, 6, (2, 4)), ("heqh", 1024, 1024, 2, 6, (4, 1)), ("qeqe", 1856, 2944, 2, 10, (2, 4)),
                                                ("qeqe", 2048, 576, 1, 70, (4, 1))])
@pytest.mark.parametrize("offloaded,n_slots", [((0, 3), 1), ((0, 1, 2, 3), 2)])
def test_swapped_experts_sum_in_the_same_order(orc, bits, d, f, k, T, teams, offloaded, n_slots):
    """Bit for bit the block with every expert resident, also where all experts of a precision come later."""
    assert launch_teams(bits, d, f, k, T) == teams
    wl = build_workload(_config(bits, d, f, k, T), orc)
    x = dev(wl.x)
    want, want_idx, status = _forward(device_layer(wl), x, k)
    assert status == 0
    layer, hosts = device_layer_with_offloaded(wl, set(offloaded))
    ws, out = mm.alloc_workspace(layer, T), torch.full_like(x, float("nan"))
    ws.fill_(0xFF)
    missed = mm.moe_layer_forward_swap(layer, mm.Swap(layer, hosts, n_slots, T), x, out, ws)
    assert mm.moe_read_status(ws) == 0 and missed == len({int(e) for e in want_idx.reshape(-1)} & set(offloaded))
    assert np.array_equal(out.cpu().numpy().view(np.uint16), want.view(np.uint16))


@pytest.mark.gpu
@pytest.mark.parametrize("bits,d,f,T,teams", [("q", 1984, 448, 6, (4, 1)), ("e", 1984, 448, 6, (4, 1)), ("h", 1984, 448, 6, (4, 1)),
                                              ("q", 320, 3904, 20, (1, 4)), ("e", 320, 3904, 20, (1, 4)), ("h", 320, 3904, 20, (1, 2))])
def test_half_step_of_the_last_team_keeps_neighbours_apart(orc, bits, d, f, T, teams):
    """A row's end is the next row's start in memory: infinities at the start of a token, of a hidden row and of a weight row stay
    with their token and their output column."""
    assert launch_teams(bits, d, f, 1, T) == teams
    wl = build_workload(_config(bits, d, f, 1, T), orc)
    layer = device_layer(wl)
    clean, _, _ = _forward(layer, dev(wl.x), 1)
    x = wl.x.copy()
    x[3, 0] = np.inf
    got, _, _ = _forward(layer, dev(x), 1)
    keep = np.arange(T) != 3
    assert np.array_equal(got[keep], clean[keep]) and not np.isfinite(got[3]).all()
    w2 = layer.experts[0].w2
    (w2.data if bits == "h" else w2.scale)[7, 0] = float("inf")
    got, _, _ = _forward(layer, dev(wl.x), 1)
    cols = np.arange(d) != 7
    assert np.array_equal(got[:, cols], clean[:, cols]) and not np.isfinite(got[:, 7]).any()
