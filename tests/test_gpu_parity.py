"""HIP path against the CPU oracle, element by element, on the same seeded inputs.  Every call goes
through the C-ABI (ctypes binding).  Bars: integers, indices and dequantized weights bit-exact; FFN and
block outputs max|err| <= 1e-2*max|ref| and relative L2 <= 2e-3 against the double-precision oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2407_14417_amd import binding as mm
from paper_2407_14417_amd import synth
from tests import common
from tests.common import (TINY, MEDIUM, MEDIUM_ZIPF, ODD_STEPS, GENERIC, STEPS4, STEPS4_ZIPF, STEPS4_ZIPF_Q, STEPS4_ZIPF_MID,
                          build_workload, assert_ffn_close, launch_forms)
from tests.gpu_common import dev, device_layer, device_mat, prec_of

pytestmark = pytest.mark.gpu

GATE_ATOL = 2e-6          # gates are fp32 on both sides; logits differ by fp32 vs fp64 accumulation


def _say(msg):
    print(msg, flush=True)


# ---------------------------------------------------------------- generator and format

@pytest.mark.parametrize("kind,scale,stream", [(0, float(synth.normal_scale(0.02)), synth.expert_stream(2, 3, 1)),
                                               (0, float(synth.normal_scale(1.0)), synth.x_stream(0)),
                                               (1, float(synth.uniform_scale(0.0346)), synth.STREAM_WG)])
def test_device_fill_equals_host_generator(kind, scale, stream):
    n, first = 1_000_003, 12345
    dst = torch.empty(n, dtype=torch.float16, device="cuda")
    mm.moe_synth_fill_f16(dst, first, 7, stream, scale, kind)
    if kind == 0:
        ref = synth._fill("normal", (n,), 7, stream, np.float32(scale), first, False)
    else:
        ref = synth._fill("uniform", (n,), 7, stream, np.float32(scale), first, False)
    assert np.array_equal(dst.cpu().numpy().view(np.uint16), ref.view(np.uint16))


def test_dequant_bit_exact_all_scales_all_codes(orc):
    """Every fp16 scale pattern (finite) x all 16 codes, for several zeros, plus random (scale, zero) pairs."""
    s_bits = np.arange(0x7C00, dtype=np.uint16)                       # all non-negative finite scales
    rng = np.random.default_rng(5)
    zs = np.array([0.0, -0.0547, 0.031, -1.5, 6.1e-5, -3.0e-6, 100.0], dtype=np.float16)
    rows = []
    for z in zs:
        rows.append((s_bits.view(np.float16), np.full(s_bits.size, z, dtype=np.float16)))
    rs = rng.integers(0, 0x7C00, 40000).astype(np.uint16).view(np.float16)
    rz = (rng.integers(0, 0x7C00, 40000).astype(np.uint16) | (rng.integers(0, 2, 40000).astype(np.uint16) << 15)).view(np.float16)
    rows.append((rs, rz))
    scale = np.concatenate([r[0] for r in rows])[:, None].copy()
    zero = np.concatenate([r[1] for r in rows])[:, None].copy()
    n = scale.shape[0]
    packed = np.zeros((n, 32), dtype=np.uint8)
    for j in range(32):
        packed[:, j] = ((2 * j) % 16) | (((2 * j + 1) % 16) << 4)
    m = orc.Mat(packed, scale, zero)
    ref = orc.dequant_int4(m)
    out = torch.empty((n, 64), dtype=torch.float16, device="cuda")
    mm.moe_dequant_int4(device_mat(m), n, 64, out)
    got = out.cpu().numpy()
    same = got.view(np.uint16) == ref.view(np.uint16)
    both_zero = (got == 0) & (ref == 0)                                  # sign of an exact zero sum is not pinned
    assert (same | both_zero).all(), np.argwhere(~(same | both_zero))[:5]


def test_dequant_bit_exact_on_quantized_weights(orc):
    w = synth.normal_f16((300, 1088), 0.02, 3, 50)
    m = orc.quantize_int4(w)
    out = torch.empty((300, 1088), dtype=torch.float16, device="cuda")
    mm.moe_dequant_int4(device_mat(m), 300, 1088, out)
    assert np.array_equal(out.cpu().numpy().view(np.uint16), orc.dequant_int4(m).view(np.uint16))


@pytest.mark.parametrize("shape,sigma", [((64, 256), 0.02), ((301, 1088), 0.02), ((17, 64), 1.0), ((4, 4096), 3e-4)])
def test_device_quantizer_bit_exact(orc, shape, sigma):
    w = synth.normal_f16(shape, sigma, 4, 60)
    w[0, :64] = w[0, 0]                                                 # a constant group: scale 0, codes 0
    ref = orc.quantize_int4(w)
    got = mm.quantize_mat(dev(w))
    assert np.array_equal(got.data.cpu().numpy(), ref.data)
    assert np.array_equal(got.scale.cpu().numpy().view(np.uint16), ref.scale.view(np.uint16))
    assert np.array_equal(got.zero.cpu().numpy().view(np.uint16), ref.zero.view(np.uint16))


# ---------------------------------------------------------------- gating and grouping

@pytest.mark.parametrize("cfg", [TINY, MEDIUM, MEDIUM_ZIPF], ids=lambda c: c.name)
def test_route_indices_bit_exact_gates_close(orc, cfg):
    wl = build_workload(cfg, orc, experts_needed=())
    layer = device_layer(wl)
    x = dev(wl.x)
    idx = torch.empty((cfg.T, cfg.k), dtype=torch.int32, device="cuda")
    gate = torch.empty((cfg.T, cfg.k), dtype=torch.float32, device="cuda")
    mm.moe_route(layer, x, idx, gate)
    ref_idx, ref_gate = orc.route(wl.x, wl.wg, cfg.k, bias=wl.bias)
    assert np.array_equal(idx.cpu().numpy(), ref_idx)
    assert np.allclose(gate.cpu().numpy(), ref_gate, rtol=0, atol=GATE_ATOL)


@pytest.mark.parametrize("E,k,T", [(8, 2, 1), (8, 2, 16), (4, 2, 16), (8, 1, 33), (8, 3, 70), (32, 8, 40), (8, 8, 5),
                                   (8, 2, 2500)])
def test_route_other_expert_counts_and_topk(orc, E, k, T):
    d = 512
    wg = synth.normal_f16((E, d), 0.02, 21, synth.STREAM_WG)
    cfg = common.Config("r", d, 64, E, k, T, ())
    x = common.tokens_with_margin(cfg, wg, None)
    ex = [mm.Expert(mm.PREC_FP16, None, None, None, resident=False) for _ in range(E)]
    layer = mm.Layer(d, 64, k, dev(wg), ex)
    idx = torch.empty((T, k), dtype=torch.int32, device="cuda")
    gate = torch.empty((T, k), dtype=torch.float32, device="cuda")
    mm.moe_route(layer, dev(x), idx, gate)
    ref_idx, ref_gate = orc.route(x, wg, k)
    assert np.array_equal(idx.cpu().numpy(), ref_idx)
    assert np.allclose(gate.cpu().numpy(), ref_gate, rtol=0, atol=GATE_ATOL)


def test_route_equal_logits_take_lower_index(orc):
    d, E, k = 64, 8, 3
    wg = np.zeros((E, d), dtype=np.float16)
    wg[[1, 4, 6], 0] = 2.0
    wg[3, 0] = 1.0
    x = np.zeros((2, d), dtype=np.float16)
    x[0, 0] = 1.0
    x[1, 0] = -1.0                     # all logits <= 0: zeros tie, lower indices win
    ex = [mm.Expert(mm.PREC_FP16, None, None, None, resident=False) for _ in range(E)]
    layer = mm.Layer(d, 64, k, dev(wg), ex)
    idx = torch.empty((2, k), dtype=torch.int32, device="cuda")
    gate = torch.empty((2, k), dtype=torch.float32, device="cuda")
    mm.moe_route(layer, dev(x), idx, gate)
    ref_idx, ref_gate = orc.route(x, wg, k)
    assert np.array_equal(idx.cpu().numpy(), ref_idx) and list(ref_idx[0]) == [1, 4, 6] and list(ref_idx[1]) == [0, 2, 5]
    assert np.allclose(gate.cpu().numpy(), ref_gate, atol=GATE_ATOL)


@pytest.mark.parametrize("E,k,T", [(8, 2, 1), (4, 2, 16), (8, 2, 512), (8, 3, 100), (32, 8, 77), (8, 2, 3000)])
def test_permute_bit_exact(orc, E, k, T):
    rng = np.random.default_rng(E * 1000 + T)
    idx = np.stack([rng.permutation(E)[:k] for _ in range(T)]).astype(np.int32)
    if T > 100:
        idx[:, 0] = np.minimum(idx[:, 0], rng.integers(0, E, T))      # skew; duplicates inside a token are legal here
    ex = [mm.Expert(mm.PREC_FP16, None, None, None, resident=False) for _ in range(E)]
    layer = mm.Layer(64, 64, k, torch.zeros((E, 64), dtype=torch.float16, device="cuda"), ex)
    ws = mm.alloc_workspace(layer, T)
    counts = torch.empty(E, dtype=torch.int32, device="cuda")
    offsets = torch.empty(E + 1, dtype=torch.int32, device="cuda")
    perm = torch.empty(T * k, dtype=torch.int32, device="cuda")
    mm.moe_permute(layer, dev(idx), counts, offsets, perm, ws)
    rc, ro, rp = orc.permute(idx, E)
    assert np.array_equal(counts.cpu().numpy(), rc)
    assert np.array_equal(offsets.cpu().numpy(), ro)
    assert np.array_equal(perm.cpu().numpy(), rp)
    assert mm.moe_read_status(ws) == 0


def test_permute_flags_bad_index():
    E, k, T = 4, 2, 8
    idx = np.zeros((T, k), dtype=np.int32)
    idx[:, 1] = 1
    idx[3, 1] = 9
    ex = [mm.Expert(mm.PREC_FP16, None, None, None, resident=False) for _ in range(E)]
    layer = mm.Layer(64, 64, k, torch.zeros((E, 64), dtype=torch.float16, device="cuda"), ex)
    ws = mm.alloc_workspace(layer, T)
    counts = torch.empty(E, dtype=torch.int32, device="cuda")
    offsets = torch.empty(E + 1, dtype=torch.int32, device="cuda")
    perm = torch.full((T * k,), -7, dtype=torch.int32, device="cuda")
    mm.moe_permute(layer, dev(idx), counts, offsets, perm, ws)
    assert mm.moe_read_status(ws) == mm.STATUS_BAD_INDEX
    assert list(counts.cpu().numpy()) == [8, 7, 0, 0] and int(offsets[-1]) == 15


# ---------------------------------------------------------------- experts

@pytest.mark.parametrize("cfg", [TINY, MEDIUM], ids=lambda c: c.name)
@pytest.mark.parametrize("n", [1, 2, 3, 5, 17, 40])
def test_expert_ffn_both_precisions(orc, cfg, n):
    wl = build_workload(cfg, orc, experts_needed=(0, 1))
    assert not wl.experts[0].int4 and wl.experts[1].int4
    layer = device_layer(wl)
    x = synth.normal_f16((n, cfg.d), 1.0, 31, synth.x_stream(0))
    ws = mm.alloc_workspace(layer, (n + cfg.k - 1) // cfg.k)
    for e in (0, 1):
        _say(f"expert_ffn cfg={cfg.name} n={n} expert={e}")
        y = torch.empty((n, cfg.d), dtype=torch.float32, device="cuda")
        mm.moe_expert_ffn_mixed(layer, e, dev(x), y, ws)
        assert_ffn_close(y.cpu().numpy(), orc.expert_ffn(wl.experts[e], x), f"{cfg.name} n={n} e={e}")


@pytest.mark.parametrize("n", [2, 16, 17, 33, 40, 72, 90, 105, 130, 300])
def test_expert_ffn_odd_steps_ragged_tiles_many_chunks(orc, n):
    """Matrix-core path: odd step counts (the last pair of 4-bit steps is fetched one step back), a ragged tile of
    weight rows, row counts from one partial 16-row tile to three 128-row chunks; 40, 72, 90 and 105 rows run the
    bodies for exactly 3, 5, 6 and 7 activation tiles."""
    cfg = ODD_STEPS
    wl = build_workload(cfg, orc, experts_needed=(0, 1))
    assert wl.experts[0].int4 and not wl.experts[1].int4
    layer = device_layer(wl)
    x = synth.normal_f16((n, cfg.d), 1.0, 37, synth.x_stream(0))
    ws = mm.alloc_workspace(layer, (n + cfg.k - 1) // cfg.k)
    for e in (0, 1):
        _say(f"expert_ffn cfg={cfg.name} n={n} expert={e}")
        y = torch.full((n, cfg.d), float("nan"), dtype=torch.float32, device="cuda")
        mm.moe_expert_ffn_mixed(layer, e, dev(x), y, ws)
        assert_ffn_close(y.cpu().numpy(), orc.expert_ffn(wl.experts[e], x), f"{cfg.name} n={n} e={e}")


@pytest.mark.parametrize("n", [70, 90, 100, 128, 129, 148, 188, 200, 256, 257, 300, 400, 520])
def test_expert_ffn_pipelined_bodies(orc, n):
    """Matrix-core path, one 16-bit or 4-bit expert alone with more than 64 rows: chunks of up to 128 rows on workgroups of 4
    wavefronts (launches this small), with full, ragged and one-tile last ones (148 = 128 + 20 rows, 188 = 128 + 60,
    129 = 128 + 1, ...)."""
    cfg = STEPS4
    wl = build_workload(cfg, orc, experts_needed=(0, 1))
    assert not wl.experts[0].int4 and wl.experts[1].int4
    layer = device_layer(wl)
    x = synth.normal_f16((n, cfg.d), 1.0, 41, synth.x_stream(0))
    ws = mm.alloc_workspace(layer, (n + cfg.k - 1) // cfg.k)
    for e in (0, 1):
        assert [m.waves for m in launch_forms([prec_of(x) for x in wl.experts[:2]], cfg.d, cfg.f, cfg.k, n, e)] == [4, 4]
        _say(f"expert_ffn cfg={cfg.name} n={n} expert={e}")
        y = torch.full((n, cfg.d), float("nan"), dtype=torch.float32, device="cuda")
        mm.moe_expert_ffn_mixed(layer, e, dev(x), y, ws)
        assert_ffn_close(y.cpu().numpy(), orc.expert_ffn(wl.experts[e], x), f"{cfg.name} n={n} e={e}")


@pytest.mark.parametrize("n", [1, 4, 9])
def test_expert_ffn_shape_agnostic_kernels(orc, n):
    cfg = GENERIC
    wl = build_workload(cfg, orc, experts_needed=(0, 1))
    layer = device_layer(wl)
    x = synth.normal_f16((n, cfg.d), 1.0, 41, synth.x_stream(0))
    ws = mm.alloc_workspace(layer, (n + cfg.k - 1) // cfg.k)
    for e in (0, 1):
        _say(f"expert_ffn cfg={cfg.name} n={n} expert={e}")
        y = torch.empty((n, cfg.d), dtype=torch.float32, device="cuda")
        mm.moe_expert_ffn_mixed(layer, e, dev(x), y, ws)
        assert_ffn_close(y.cpu().numpy(), orc.expert_ffn(wl.experts[e], x), f"{cfg.name} n={n} e={e}")


def test_expert_ffn_single_row_runs_the_one_token_kernels(orc):
    """n = 1 at a shape the batch-1 kernels take (d and f multiples of 2048): the expert alone, before gating and
    weighted average, for a 16-bit and a 4-bit expert; the workspace status stays clear."""
    cfg = common.DECODE_SMALL
    wl = build_workload(cfg, orc, experts_needed=(0, 1))
    assert not wl.experts[0].int4 and wl.experts[1].int4
    layer = device_layer(wl)
    ws = mm.alloc_workspace(layer, 1)
    for seed in (43, 44):
        x = synth.normal_f16((1, cfg.d), 1.0, seed, synth.x_stream(0))
        for e in (0, 1):
            _say(f"expert_ffn one-token kernels cfg={cfg.name} seed={seed} expert={e}")
            y = torch.full((1, cfg.d), float("nan"), dtype=torch.float32, device="cuda")
            mm.moe_expert_ffn_mixed(layer, e, dev(x), y, ws)
            assert mm.moe_read_status(ws) == 0
            assert_ffn_close(y.cpu().numpy(), orc.expert_ffn(wl.experts[e], x), f"{cfg.name} n=1 e={e}")


def test_expert_ffn_identity_weights_exact_structure(orc):
    """One-entry matrices: catches a transposed operand or swapped w1/w3 in the kernels."""
    d, f = 128, 192
    w1 = np.zeros((f, d), dtype=np.float16); w1[70, 5] = 1.5
    w3 = np.zeros((f, d), dtype=np.float16); w3[70, 5] = 0.25
    w2 = np.zeros((d, f), dtype=np.float16); w2[100, 70] = 4.0
    x = np.zeros((2, d), dtype=np.float16); x[0, 5] = 2.0; x[1, 5] = -1.0
    e16 = orc.Expert(orc.Mat(w1), orc.Mat(w3), orc.Mat(w2))
    e4 = orc.Expert(orc.quantize_int4(w1), orc.quantize_int4(w3), orc.quantize_int4(w2))
    wl = common.Workload(common.Config("s", d, f, 2, 1, 2, (1,)), x, np.zeros((2, d), dtype=np.float16), None, [e16, e4])
    layer = device_layer(wl)
    ws = mm.alloc_workspace(layer, 2)
    for e in (0, 1):
        y = torch.empty((2, d), dtype=torch.float32, device="cuda")
        mm.moe_expert_ffn_mixed(layer, e, dev(x), y, ws)
        ref = orc.expert_ffn(wl.experts[e], x)
        got = y.cpu().numpy()
        assert np.count_nonzero(got) == 2 and np.allclose(got, ref, rtol=2e-3, atol=1e-6)


# ---------------------------------------------------------------- whole block

def _run_layer(layer, x_np, cfg):
    x = dev(x_np)
    out = torch.empty_like(x)
    idx = torch.empty((x_np.shape[0], cfg.k), dtype=torch.int32, device="cuda")
    gate = torch.empty((x_np.shape[0], cfg.k), dtype=torch.float32, device="cuda")
    ws = mm.alloc_workspace(layer, x_np.shape[0])
    mm.moe_layer_forward(layer, x, out, ws, idx, gate)
    return out.cpu().numpy(), idx.cpu().numpy(), gate.cpu().numpy(), mm.moe_read_status(ws)


@pytest.mark.parametrize("cfg", [TINY, MEDIUM, MEDIUM_ZIPF, ODD_STEPS, GENERIC, STEPS4, STEPS4_ZIPF, STEPS4_ZIPF_Q,
                                 STEPS4_ZIPF_MID], ids=lambda c: c.name)
def test_layer_forward(orc, cfg):
    wl = build_workload(cfg, orc)
    _say(f"layer_forward cfg={cfg.name}")
    out, idx, gate, status = _run_layer(device_layer(wl), wl.x, cfg)
    ref, ref_idx, ref_gate = orc.layer_forward(wl.x, wl.wg, wl.experts, cfg.k, bias=wl.bias)
    assert status == 0
    assert np.array_equal(idx, ref_idx)
    assert np.allclose(gate, ref_gate, rtol=0, atol=GATE_ATOL)
    assert_ffn_close(out, ref, cfg.name)


@pytest.mark.parametrize("T,tiles", [(288, (8, 8, 1, 8, 3)), (320, (10, 9, 12)), (360, (11, 10, 14))])
def test_layer_forward_4bit_chunks_of_more_than_8_tiles(orc, T, tiles):
    """The busiest 4-bit experts get between 129 and 384 rows: chunks of up to 256 rows, split evenly, on workgroups of 8
    wavefronts (``tiles``: 16-row tiles of the chunks of experts 0 and 1, as the row counts asserted below imply); the
    fewest tokens have 72 rows per expert, which run on workgroups of 4 in chunks of 128 rows and a rest."""
    cfg = common.Config(f"steps4_zipf_4bit_heavy_T{T}", 1024, 5120, 8, 2, T, STEPS4_ZIPF_Q.int4_experts, zipf=1.2)
    wl = build_workload(cfg, orc)
    _say(f"layer_forward cfg={cfg.name}")
    out, idx, gate, status = _run_layer(device_layer(wl), wl.x, cfg)
    ref, ref_idx, ref_gate = orc.layer_forward(wl.x, wl.wg, wl.experts, cfg.k, bias=wl.bias)
    counts = np.bincount(ref_idx.reshape(-1), minlength=cfg.E)
    _say(f"rows per expert: {counts.tolist()}")

    forms = launch_forms([prec_of(e) for e in wl.experts], cfg.d, cfg.f, cfg.k, T)
    assert [(m.waves, m.quant_rows) for m in forms] == [(4, 0) if T == 288 else (8, 256)] * 2

    def chunk_tiles(n):          # the library's rule for a 4-bit expert with more than 128 rows
        nch = -(-n // 256)
        per = (-(-n // nch) + 15) // 16 * 16 if T > 288 else 128
        nch = -(-n // per)
        return tuple((min(per, n - i * per) + 15) // 16 for i in range(nch))
    assert chunk_tiles(int(counts[0])) + chunk_tiles(int(counts[1])) == tiles
    assert status == 0
    assert np.array_equal(idx, ref_idx)
    assert np.allclose(gate, ref_gate, rtol=0, atol=GATE_ATOL)
    assert_ffn_close(out, ref, cfg.name)


def test_layer_forward_many_tokens_several_chunks_per_expert(orc):
    """600 tokens with skewed routing: the busiest experts span several 128-row chunks of the matrix-core path,
    the rarest fit in one partial tile; grouped rows come through the permutation."""
    cfg = common.Config("medium_many", 1024, 2816, 8, 2, 600, (1, 2, 5, 7), zipf=1.2)
    wl = build_workload(cfg, orc)
    _say(f"layer_forward cfg={cfg.name}")
    out, idx, gate, status = _run_layer(device_layer(wl), wl.x, cfg)
    ref, ref_idx, ref_gate = orc.layer_forward(wl.x, wl.wg, wl.experts, cfg.k, bias=wl.bias)
    counts = np.bincount(ref_idx.reshape(-1), minlength=cfg.E)
    _say(f"rows per expert: {counts.tolist()}")
    assert counts.max() > 256 and counts.min() < 64
    assert status == 0
    assert np.array_equal(idx, ref_idx)
    assert np.allclose(gate, ref_gate, rtol=0, atol=GATE_ATOL)
    assert_ffn_close(out, ref, cfg.name)


@pytest.mark.parametrize("E,k,T,zipf", [(32, 8, 500, None), (32, 4, 1500, 1.5), (8, 8, 64, None), (5, 2, 33, 2.0)])
def test_layer_forward_many_experts_and_slots(orc, E, k, T, zipf):
    """The limits of the descriptor (32 experts, top-8), experts that receive no row at all (steep Zipf offsets),
    thousands of grouped rows on a small matrix shape."""
    cfg = common.Config(f"E{E}k{k}T{T}", 256, 512, E, k, T, tuple(range(0, E, 2)), zipf=zipf)
    wl = build_workload(cfg, orc)
    _say(f"layer_forward cfg={cfg.name}")
    out, idx, gate, status = _run_layer(device_layer(wl), wl.x, cfg)
    ref, ref_idx, ref_gate = orc.layer_forward(wl.x, wl.wg, wl.experts, cfg.k, bias=wl.bias)
    counts = np.bincount(ref_idx.reshape(-1), minlength=E)
    _say(f"rows per expert: min {counts.min()} max {counts.max()} empty {int((counts == 0).sum())}")
    assert status == 0
    assert np.array_equal(idx, ref_idx)
    assert np.allclose(gate, ref_gate, rtol=0, atol=GATE_ATOL)
    assert_ffn_close(out, ref, cfg.name)


def _random_configs(n, seed=20240719):
    """Seeded draw of block shapes inside the library's limits: d_model and d_ff multiples of 64 (some multiples
    of 128: matrix-core path, the others: shape-agnostic kernels), 1-12 experts, top-1..4, 1-70 tokens, a random
    precision mask, optional Zipf offsets."""
    rng = np.random.default_rng(seed)
    cfgs = []
    for i in range(n):
        d = int(rng.choice([64, 128, 192, 256, 384, 512, 640, 768, 1024]))
        f = int(rng.choice([64, 128, 320, 384, 512, 896, 1024, 1536]))
        E = int(rng.integers(1, 13))
        k = int(rng.integers(1, min(E, 4) + 1))
        T = int(rng.choice([1, 2, 3, 7, 16, 17, 31, 33, 48, 70]))
        mask = tuple(int(e) for e in range(E) if rng.random() < 0.5)
        zipf = float(rng.choice([0.0, 1.2, 2.0]))
        cfgs.append(common.Config(f"rand{i}_d{d}_f{f}_E{E}_k{k}_T{T}", d, f, E, k, T, mask, seed=100 + i,
                                  zipf=zipf or None))
    return cfgs


@pytest.mark.parametrize("cfg", _random_configs(20), ids=lambda c: c.name)
def test_layer_forward_random_shapes(orc, cfg):
    wl = build_workload(cfg, orc)
    _say(f"layer_forward cfg={cfg.name} int4={cfg.int4_experts} zipf={cfg.zipf}")
    out, idx, gate, status = _run_layer(device_layer(wl), wl.x, cfg)
    ref, ref_idx, ref_gate = orc.layer_forward(wl.x, wl.wg, wl.experts, cfg.k, bias=wl.bias)
    assert status == 0
    assert np.array_equal(idx, ref_idx)
    assert np.allclose(gate, ref_gate, rtol=0, atol=GATE_ATOL)
    assert_ffn_close(out, ref, cfg.name)


def test_layer_forward_single_token_and_odd_token_counts(orc):
    wl = build_workload(MEDIUM, orc)
    layer = device_layer(wl)
    for T in (1, 2, 7):
        _say(f"layer_forward medium T={T}")
        out, idx, gate, status = _run_layer(layer, wl.x[:T], MEDIUM)
        ref, ref_idx, _ = orc.layer_forward(wl.x[:T], wl.wg, wl.experts, MEDIUM.k)
        assert status == 0 and np.array_equal(idx, ref_idx)
        assert_ffn_close(out, ref, f"T={T}")


def test_layer_forward_top1_and_top3(orc):
    for k in (1, 3):
        cfg = common.Config(f"k{k}", 256, 512, 4, k, 16, (1, 3))
        wl = build_workload(cfg, orc)
        out, idx, gate, status = _run_layer(device_layer(wl), wl.x, cfg)
        ref, ref_idx, ref_gate = orc.layer_forward(wl.x, wl.wg, wl.experts, k)
        assert status == 0 and np.array_equal(idx, ref_idx)
        assert np.allclose(gate, ref_gate, rtol=0, atol=GATE_ATOL)
        assert_ffn_close(out, ref, f"k={k}")


def test_non_resident_routed_expert_sets_status_and_is_left_out(orc):
    wl = build_workload(TINY, orc)
    ref_idx, ref_gate = orc.route(wl.x, wl.wg, TINY.k)
    victim = int(ref_idx[0, 0])
    e = wl.experts[victim]
    layer = device_layer(wl)
    layer.experts[victim].resident = False
    layer = mm.Layer(TINY.d, TINY.f, TINY.k, layer.w_gate, layer.experts)
    out, idx, gate, status = _run_layer(layer, wl.x, TINY)
    assert status == mm.STATUS_NOT_RESIDENT
    assert np.array_equal(idx, ref_idx)
    # what remains is the gate-weighted sum over the resident experts only
    ref = np.zeros((TINY.T, TINY.d))
    for t in range(TINY.T):
        for s in range(TINY.k):
            if ref_idx[t, s] != victim:
                ref[t] += float(ref_gate[t, s]) * orc.expert_ffn(wl.experts[ref_idx[t, s]], wl.x[t:t + 1])[0]
    assert_ffn_close(out, ref, "resident part")
    # an unused non-resident expert raises nothing
    unused = [i for i in range(TINY.E) if i not in set(ref_idx[:1].reshape(-1))]
    layer2 = device_layer(wl)
    layer2.experts[unused[0]].resident = False
    layer2 = mm.Layer(TINY.d, TINY.f, TINY.k, layer2.w_gate, layer2.experts)
    _, _, _, status2 = _run_layer(layer2, wl.x[:1], TINY)
    assert status2 == 0


# ---------------------------------------------------------------- chain

def _chain_workloads(cfg, orc, n_layers):
    wls = []
    for l in range(n_layers):
        c = common.Config(f"{cfg.name}_l{l}", cfg.d, cfg.f, cfg.E, cfg.k, cfg.T, cfg.int4_experts, seed=cfg.seed, layer=l)
        wg = common.gate_matrix(c)
        experts = []
        mask = synth.precision_mask(cfg.E * n_layers, cfg.E * n_layers // 2, cfg.seed)
        for e in range(cfg.E):
            w1, w3, w2 = common.expert_weights_f16(c, e)
            if mask[l * cfg.E + e]:
                experts.append(orc.Expert(orc.quantize_int4(w1), orc.quantize_int4(w3), orc.quantize_int4(w2)))
            else:
                experts.append(orc.Expert(orc.Mat(w1), orc.Mat(w3), orc.Mat(w2)))
        wls.append(common.Workload(c, None, wg, None, experts))
    return wls


def _oracle_trajectory(orc, wls, h0, g, eps, k):
    """Oracle hidden states, normed block inputs, block outputs (double), indices and, per token, the smallest
    top-(k+1) adjacent logit gap over all layers."""
    hs, normeds, outs, idxs = [h0], [], [], []
    gap = np.full(h0.shape[0], np.inf)
    for wl in wls:
        h1, idx, gate, normed = orc.chain_layer(hs[-1], g, eps, wl.wg, wl.experts, k)
        out, idx2, _ = orc.layer_forward(normed, wl.wg, wl.experts, k)
        assert np.array_equal(idx, idx2)
        lg = np.sort(common.logits_f64(normed, wl.wg, None), axis=1)[:, ::-1]
        gap = np.minimum(gap, (lg[:, :k] - lg[:, 1:k + 1]).min(axis=1))
        hs.append(h1)
        normeds.append(normed)
        outs.append(out)
        idxs.append(idx)
    return hs, normeds, outs, idxs, gap


@pytest.mark.parametrize("cfg,n_layers", [(TINY, 5), (common.Config("medium1", 1024, 2816, 8, 2, 1, ()), 3)],
                         ids=["tiny5", "medium3_T1"])
def test_chain_teacher_forced_and_free_running(orc, cfg, n_layers):
    eps = 1e-5
    g = np.ones(cfg.d, dtype=np.float16)
    # free-running parity needs tokens whose routing is decided with a margin that the drift between fp32 and
    # fp64 hidden states cannot cross: take the first seed in which at least half of the tokens have it
    for seed in range(8):
        c = common.Config(cfg.name, cfg.d, cfg.f, cfg.E, cfg.k, cfg.T, (), seed=seed)
        wls = _chain_workloads(c, orc, n_layers)
        h0 = synth.normal_f16((c.T, c.d), 1.0, seed, synth.x_stream(0))
        hs, normeds, outs, idxs, gap = _oracle_trajectory(orc, wls, h0, g, eps, c.k)
        safe_tok = gap > 1e-2
        if safe_tok.sum() * 2 >= c.T:
            break
    else:
        pytest.fail("no seed with enough well-separated tokens")
    _say(f"chain cfg={cfg.name} seed={seed} safe tokens {int(safe_tok.sum())}/{c.T}")
    layers = [device_layer(w) for w in wls]
    gains = [dev(g) for _ in range(n_layers)]
    ws = mm.alloc_workspace(layers[0], c.T)
    # teacher forced: every layer gets the oracle's input of that layer
    for l in range(n_layers):
        _say(f"chain teacher-forced layer={l}")
        h = dev(hs[l])
        idx_out = torch.empty((1, c.T, c.k), dtype=torch.int32, device="cuda")
        mm.moe_chain_forward(mm.Chain([layers[l]], [gains[l]]), eps, h, ws, idx_out)
        lg = np.sort(common.logits_f64(orc.rmsnorm(hs[l], g, eps), wls[l].wg, None), axis=1)[:, ::-1]
        ok = (lg[:, :c.k] - lg[:, 1:c.k + 1]).min(axis=1) > 1e-3
        assert ok.any()
        assert np.array_equal(idx_out.cpu().numpy()[0][ok], idxs[l][ok])
        # the block alone on the oracle's normed input: both criteria of the block tolerance
        blk = torch.empty((c.T, c.d), dtype=torch.float16, device="cuda")
        idx_blk = torch.empty((c.T, c.k), dtype=torch.int32, device="cuda")
        mm.moe_layer_forward(layers[l], dev(normeds[l]), blk, ws, idx_blk, None)
        assert np.array_equal(idx_blk.cpu().numpy()[ok], idxs[l][ok])
        assert_ffn_close(blk.cpu().numpy()[ok], outs[l][ok], f"teacher-forced block {l}")
        # extra: the fused RMSNorm + block + residual step.  The stored h is rounded to fp16 on both sides, which
        # can move an element by one unit in its last place on top of the block's own deviation
        upd = h.cpu().numpy().astype(np.float64)[ok] - hs[l].astype(np.float64)[ok]
        ref = hs[l + 1].astype(np.float64)[ok] - hs[l].astype(np.float64)[ok]
        ulp = 2.0 ** -10 * np.abs(hs[l + 1].astype(np.float64)).max()
        assert np.abs(upd - ref).max() <= 1e-2 * np.abs(ref).max() + ulp
    # free running over all layers
    _say("chain free-running")
    h = dev(h0)
    idx_out = torch.empty((n_layers, c.T, c.k), dtype=torch.int32, device="cuda")
    mm.moe_chain_forward(mm.Chain(layers, gains), eps, h, ws, idx_out)
    assert mm.moe_read_status(ws) == 0
    assert np.array_equal(idx_out.cpu().numpy()[:, safe_tok], np.stack(idxs)[:, safe_tok])
    assert_ffn_close(h.cpu().numpy()[safe_tok], hs[-1][safe_tok], "free-running h")


# ---------------------------------------------------------------- batch-1 decode kernels at a small shape

@pytest.mark.parametrize("k", [1, 2, 3])
def test_decode_path_small_shape_all_precision_mixes(orc, k):
    """T=1 goes through the decode kernels (token in registers, factored 4-bit dot products, fused weighted
    average).  Twelve tokens: with 4 of 8 experts 4-bit the routed sets cover 16-bit only, mixed and 4-bit only."""
    base = common.DECODE_SMALL
    cfg = common.Config(base.name, base.d, base.f, base.E, k, 1, base.int4_experts)
    wl = build_workload(cfg, orc)
    layer = device_layer(wl)
    ws = mm.alloc_workspace(layer, 1)
    kinds = set()
    for retry in range(12):
        x = synth.normal_f16((1, cfg.d), 1.0, cfg.seed, synth.x_stream(retry))
        lg = np.sort(common.logits_f64(x, wl.wg, None)[0])[::-1]
        if (lg[:k] - lg[1:k + 1]).min() < 1e-3:
            continue
        _say(f"decode small k={k} token stream {retry}")
        out = torch.empty((1, cfg.d), dtype=torch.float16, device="cuda")
        idx = torch.empty((1, k), dtype=torch.int32, device="cuda")
        gate = torch.empty((1, k), dtype=torch.float32, device="cuda")
        mm.moe_layer_forward(layer, dev(x), out, ws, idx, gate)
        assert mm.moe_read_status(ws) == 0
        ref, ref_idx, ref_gate = orc.layer_forward(x, wl.wg, wl.experts, k)
        assert np.array_equal(idx.cpu().numpy(), ref_idx)
        assert np.allclose(gate.cpu().numpy(), ref_gate, rtol=0, atol=GATE_ATOL)
        assert_ffn_close(out.cpu().numpy(), ref, f"decode small k={k} retry={retry}")
        kinds.add(tuple(sorted(int(e) in cfg.int4_experts for e in ref_idx[0])))
    assert len(kinds) >= (3 if k == 2 else 2)


@pytest.mark.parametrize("d,f,E,k,mask", [(2048, 2048, 3, 1, (0,)), (2048, 6144, 5, 3, (1, 2, 4)), (4096, 2048, 2, 2, (1,)),
                                          (2048, 4096, 4, 4, ()), (2048, 2048, 6, 2, (0, 1, 2, 3, 4, 5)),
                                          (6144, 2048, 2, 2, (0,)), (8192, 2048, 2, 1, (1,)), (8192, 4096, 2, 2, (0, 1)),
                                          (2048, 16384, 2, 2, (1,)), (2048, 4096, 8, 8, (0, 2, 3, 5)),
                                          (2048, 2048, 8, 5, (1, 2, 3, 6)), (2048, 2048, 32, 7, tuple(range(0, 32, 3)))])
def test_decode_path_other_shapes(orc, d, f, E, k, mask):
    """Other shapes the batch-1 kernels take (d_model and d_ff multiples of 2048, d_model up to the limit of 8192):
    two to 32 experts, top-1..8 (slots are taken two at a time: odd counts leave the last pair half empty),
    all-16-bit, all-4-bit and mixed tables, three tokens each."""
    cfg = common.Config(f"dec_d{d}_f{f}_E{E}_k{k}", d, f, E, k, 1, mask, seed=7)
    wl = build_workload(cfg, orc)
    layer = device_layer(wl)
    ws = mm.alloc_workspace(layer, 1)
    done = 0
    for retry in range(12):
        x = synth.normal_f16((1, d), 1.0, cfg.seed, synth.x_stream(retry))
        lg = np.sort(common.logits_f64(x, wl.wg, None)[0])[::-1]
        if k < E and (lg[:k] - lg[1:k + 1]).min() < 1e-3 or k == E and k > 1 and (lg[:-1] - lg[1:]).min() < 1e-3:
            continue
        _say(f"decode {cfg.name} token stream {retry}")
        out = torch.empty((1, d), dtype=torch.float16, device="cuda")
        idx = torch.empty((1, k), dtype=torch.int32, device="cuda")
        gate = torch.empty((1, k), dtype=torch.float32, device="cuda")
        mm.moe_layer_forward(layer, dev(x), out, ws, idx, gate)
        assert mm.moe_read_status(ws) == 0
        ref, ref_idx, ref_gate = orc.layer_forward(x, wl.wg, wl.experts, k)
        assert np.array_equal(idx.cpu().numpy(), ref_idx)
        assert np.allclose(gate.cpu().numpy(), ref_gate, rtol=0, atol=GATE_ATOL)
        assert_ffn_close(out.cpu().numpy(), ref, f"{cfg.name} retry={retry}")
        done += 1
        if done == 3:
            break
    assert done == 3


def test_decode_path_non_resident_and_chain(orc):
    cfg = common.DECODE_SMALL
    wl = build_workload(cfg, orc)
    x = synth.normal_f16((1, cfg.d), 1.0, cfg.seed, synth.x_stream(0))
    ref_idx, ref_gate = orc.route(x, wl.wg, cfg.k)
    layer = device_layer(wl)
    layer.experts[int(ref_idx[0, 1])].resident = False
    layer = mm.Layer(cfg.d, cfg.f, cfg.k, layer.w_gate, layer.experts)
    out, idx, gate, status = _run_layer(layer, x, cfg)
    assert status == mm.STATUS_NOT_RESIDENT and np.array_equal(idx, ref_idx)
    ref = float(ref_gate[0, 0]) * orc.expert_ffn(wl.experts[int(ref_idx[0, 0])], x)
    assert_ffn_close(out, ref, "decode, one expert left out")
    # three chained blocks at this shape: RMSNorm -> decode kernels with the residual fused into the down-projection
    eps, g = 1e-5, np.ones(cfg.d, dtype=np.float16)
    wls = _chain_workloads(cfg, orc, 3)
    hs, _, _, idxs, gap = _oracle_trajectory(orc, wls, x, g, eps, cfg.k)
    assert gap[0] > 1e-2, "pick another token stream"
    layers = [device_layer(w) for w in wls]
    h = dev(x)
    idx_out = torch.empty((3, 1, cfg.k), dtype=torch.int32, device="cuda")
    ws = mm.alloc_workspace(layers[0], 1)
    mm.moe_chain_forward(mm.Chain(layers, [dev(g)] * 3), eps, h, ws, idx_out)
    assert mm.moe_read_status(ws) == 0
    assert np.array_equal(idx_out.cpu().numpy(), np.stack(idxs))
    assert_ffn_close(h.cpu().numpy(), hs[-1], "decode chain")
    # the same chain captured in a HIP graph (the benchmark's launch configuration), replayed: every replay
    # starts from a fresh copy of the input and must end in the eager result, bit for bit
    h_eager = h.clone()
    chain = mm.Chain(layers, [dev(g)] * 3)
    x_dev = dev(x)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        h.copy_(x_dev)
        mm.moe_chain_forward(chain, eps, h, ws, idx_out)                # warm-up outside the capture
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            mm.moe_chain_forward(chain, eps, h, ws, idx_out)
        for rep in range(3):
            h.copy_(x_dev)
            idx_out.fill_(-1)
            stream.synchronize()
            graph.replay()
            stream.synchronize()
            _say(f"chain graph replay {rep}")
            assert torch.equal(h, h_eager) and np.array_equal(idx_out.cpu().numpy(), np.stack(idxs))
    torch.cuda.synchronize()
