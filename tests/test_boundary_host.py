"""The C-ABI library loads, exports what include/moemix.h declares, and its host-side argument checks
answer with the documented codes.  No kernel is launched here (runs without a GPU)."""
import ctypes
import re
from pathlib import Path

import pytest

from paper_2407_14417_amd import binding as mm
from tests.common import launch_forms, unsplit_workspace_bytes

ROOT = Path(__file__).resolve().parent.parent


@pytest.fixture(scope="module")
def L():
    if not (ROOT / "paper_2407_14417_amd" / "libmoemix.so").exists():
        from paper_2407_14417_amd import buildlib
        buildlib.build()
    return mm.lib()


def test_every_declared_symbol_is_exported(L):
    header = (ROOT / "include" / "moemix.h").read_text()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(moe_[a-z0-9_]+)\s*\(", header))
    assert declared == set(mm.EXPORTS), declared ^ set(mm.EXPORTS)
    for name in declared:
        assert hasattr(L, name), name
    assert L.moe_version() >= 1000


def _layer(d=256, f=512, E=4, k=2, gate=1, experts=None):
    ex = experts if experts is not None else (mm.CExpert * E)()
    return mm.CLayer(d, f, E, k, gate, None, ex), ex


def test_workspace_bytes_is_monotone_and_rejects_nonsense(L):
    lay, _ = _layer()
    a = L.moe_workspace_bytes(ctypes.byref(lay), 1)
    b = L.moe_workspace_bytes(ctypes.byref(lay), 16)
    assert 0 < a < b and a % 256 == 0 and b % 256 == 0
    # at least the hidden rows and the expert outputs must fit
    assert b >= 16 * 2 * 512 * 2 + 16 * 2 * 256 * 4
    assert L.moe_workspace_bytes(ctypes.byref(lay), 0) == 0
    assert L.moe_workspace_bytes(None, 4) == 0


def test_workspace_of_odd_multiples_of_64(L):
    """Never less than the unsplit call needs, exactly that at one token, and partial results of split contractions
    only within the library's own scratch: what fits there unsplit still does."""
    own = L.moe_static_scratch_bytes()
    for d, f, E, k in [(1088, 3008, 8, 2), (832, 2752, 8, 2), (320, 512, 32, 8), (512, 320, 5, 1), (64, 64, 4, 2)]:
        lay, _ = _layer(d=d, f=f, E=E, k=k)
        for T in [*range(1, 130), 500, 2000]:
            need, unsplit = L.moe_workspace_bytes(ctypes.byref(lay), T), unsplit_workspace_bytes(d, f, E, k, T)
            assert unsplit <= need and (need == unsplit or (T > 1 and need <= own)), (d, f, T)


@pytest.mark.parametrize("d,f", [(832, 2816), (1472, 1152), (320, 2304), (64 * 5, 1408), (1088, 3008), (2880, 2048), (2944, 2880), (448, 16384)])
@pytest.mark.parametrize("E,k", [(4, 2), (32, 8), (1, 1), (7, 3)])
def test_smaller_workspaces_leave_equal_ranges(L, d, f, E, k):
    """Ranges of a split contraction may differ in length only in the launches that look at each range's end: 16-row chunks
    and the variant for odd multiples of 64.  Every workspace from the unsplit call's up, block and one expert alone."""
    steps = (f + 127) // 128
    for T in [2, 3, 5, 8, 9, 16, 17, 20, 33, 40, 64, 65, 95, 130, 257, 300, 700]:
        lay, _ = _layer(d=d, f=f, E=E, k=k)
        least, full = unsplit_workspace_bytes(d, f, E, k, T), L.moe_workspace_bytes(ctypes.byref(lay), T)
        seen = set()
        for ws in sorted({least, full, *(least + s * 4 * T * k * d for s in range(1, 17)), *(least + (full - least) * i // 9 for i in range(9))}):
            for prec in (mm.PREC_FP16, mm.PREC_INT4G64):
                for expert, n in ((-1, T), (0, T), (0, T * k), (0, T * k - k + 1)):
                    if (n if expert == 0 else T * k) < 2 or n == 1:
                        continue
                    _, down = launch_forms([prec] * E, d, f, k, n, expert, ws)
                    seen.add(down.splits)
                    last = steps - (down.splits - 1) * down.steps_per_split
                    assert last >= min(2, steps)
                    if not (down.half or (down.ct == 1 and not down.waves)):
                        assert down.splits * down.steps_per_split == steps, (T, ws, expert, n, down.splits)
        assert 1 in seen


@pytest.mark.parametrize("bits,d,f,k,T,ct", [
    ("h" * 16, 5760, 2688, 8, 26, 1),      # 13 rows per expert on average, half of the experts per token: few have more than 16
    ("q" * 8, 4096, 14336, 2, 52, 2),      # the same mean, a quarter of them
    ("q" * 8, 4096, 14336, 2, 48, 1), ("h" * 4, 1024, 512, 4, 16, 1), ("q" * 4, 1024, 8192, 4, 16, 1),
    ("q" * 2, 2560, 1408, 1, 30, 1),       # twice the chunks would run side by side as well
    ("qe" * 4, 2304, 4480, 1, 256, 2),     # 32 rows: the workgroups of the down-projection do not fill the chip
    ("q" * 8, 4096, 14336, 2, 126, 4), ("h" * 8, 3072, 10752, 2, 126, 4), ("h" * 8, 3072, 10752, 4, 56, 2),
])
def test_chunk_length_follows_the_spread_of_loads(L, bits, d, f, k, T, ct):
    precs = [{"h": mm.PREC_FP16, "q": mm.PREC_INT4G64, "e": mm.PREC_INT8G64}[b] for b in bits]
    assert [m.ct for m in launch_forms(precs, d, f, k, T)] == [ct] * 2


@pytest.mark.parametrize("bits,d,f,k,T,up,down", [
    ("qe" * 4, 1024, 7168, 4, 110, 0, 0),  # 55 rows per expert, half of the experts per token: few have more than 64
    ("qe" * 4, 1024, 7168, 2, 220, 4, 4),  # the same mean, a quarter of them
    ("qe" * 4, 1024, 7168, 2, 200, 0, 0),  # one and a half to two rounds of workgroups in both projections
    ("qe" * 4, 1024, 5120, 2, 200, 4, 4), ("h" + "q" * 7, 1024, 7168, 2, 200, 4, 4),
    ("q" * 2, 5632, 3712, 1, 68, 4, 4),    # long ranges, few workgroups
    ("q" * 8, 4096, 14336, 2, 180, 0, 0),
])
def test_64_rows_per_expert_by_rounds_of_workgroups(L, bits, d, f, k, T, up, down):
    precs = [{"h": mm.PREC_FP16, "q": mm.PREC_INT4G64, "e": mm.PREC_INT8G64}[b] for b in bits]
    assert [(m.ct, m.waves) for m in launch_forms(precs, d, f, k, T)] == [(4, up), (4, down)]


@pytest.mark.parametrize("kwargs,code", [
    (dict(d=250), mm.MOE_ESHAPE), (dict(f=100), mm.MOE_ESHAPE), (dict(E=33), mm.MOE_ESHAPE),
    (dict(k=5), mm.MOE_ESHAPE), (dict(k=0), mm.MOE_ESHAPE), (dict(gate=None), mm.MOE_EINVAL),
])
def test_bad_layers_are_rejected_on_the_host(L, kwargs, code):
    E = kwargs.get("E", 4)
    lay, _ = _layer(**{**kwargs, "experts": (mm.CExpert * max(E, 1))()})
    assert L.moe_route(ctypes.byref(lay), 1, 1, 1, 1, None) == code
    assert L.moe_last_error()
    assert L.moe_layer_forward(ctypes.byref(lay), 1, 1, 1, None, None, 256, 1 << 30, None) == code


def test_misaligned_matrices_are_rejected_on_the_host(L):
    """Weights, scales and zeros are read with 128-bit loads: a resident expert whose pointers are not 16-byte
    aligned is refused before any launch."""
    ex = (mm.CExpert * 4)()
    for e in range(4):
        ex[e].prec, ex[e].resident = mm.PREC_FP16, 1
        for m in (ex[e].w1, ex[e].w3, ex[e].w2):
            m.data = 4096
    lay, _ = _layer(experts=ex)
    assert L.moe_workspace_bytes(ctypes.byref(lay), 4) > 0
    ex[2].w3.data = 4096 + 8
    assert L.moe_route(ctypes.byref(lay), 1, 1, 1, 1, None) == mm.MOE_EINVAL
    assert b"16-byte aligned" in L.moe_last_error()
    ex[2].w3.data = 4096
    ex[1].prec = mm.PREC_INT4G64
    for m in (ex[1].w1, ex[1].w3, ex[1].w2):
        m.scale, m.zero = 8192, 8192 + 2
    assert L.moe_route(ctypes.byref(lay), 1, 1, 1, 1, None) == mm.MOE_EINVAL


def test_null_and_size_arguments(L):
    lay, _ = _layer()
    assert L.moe_route(ctypes.byref(lay), None, 1, 1, 1, None) == mm.MOE_EINVAL
    assert L.moe_route(ctypes.byref(lay), 1, 0, 1, 1, None) == mm.MOE_ESHAPE
    assert L.moe_layer_forward(ctypes.byref(lay), 256, 4, 256, None, None, None, 0, None) == mm.MOE_EWORKSPACE
    assert L.moe_layer_forward(ctypes.byref(lay), 256, 4, 256, None, None, 256, 1024, None) == mm.MOE_EWORKSPACE
    assert L.moe_layer_forward(ctypes.byref(lay), 256, 4, 256, None, None, 257, 1 << 30, None) == mm.MOE_EWORKSPACE
    assert b"needed" in L.moe_last_error() or b"aligned" in L.moe_last_error()
    assert L.moe_dequant_int4(None, 1, 64, 1, None) == mm.MOE_EINVAL
    m = mm.CMat(1, 1, 1)
    assert L.moe_dequant_int4(ctypes.byref(m), 4, 96, 1, None) == mm.MOE_ESHAPE
    assert L.moe_quantize_int4(1, 4, 100, 1, 1, 1, None) == mm.MOE_ESHAPE
    assert L.moe_synth_fill_f16(None, 8, 0, 0, 0, 1.0, 0, None) == mm.MOE_EINVAL
    assert L.moe_synth_fill_f16(1, 8, 0, 0, 0, 1.0, 7, None) == mm.MOE_EINVAL


def test_explicit_non_resident_expert_fails_on_the_host(L):
    ex = (mm.CExpert * 4)()
    for e in ex:
        e.prec, e.resident = mm.PREC_FP16, 1
        e.w1.data = e.w3.data = e.w2.data = 256
    ex[2].resident = 0
    lay, _ = _layer(experts=ex)
    assert L.moe_expert_ffn_mixed(ctypes.byref(lay), 2, 256, 1, 256, 256, 1 << 30, None) == mm.MOE_ENOTRESIDENT
    assert L.moe_expert_ffn_mixed(ctypes.byref(lay), 9, 256, 1, 256, 256, 1 << 30, None) == mm.MOE_EINVAL
    ex[1].prec = mm.PREC_INT4G64          # 4-bit expert without scale/zero
    assert L.moe_route(ctypes.byref(lay), 256, 1, 256, 256, None) == mm.MOE_EINVAL
