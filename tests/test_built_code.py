"""The device code of the built library: what the compiler does not look after inside inline assembly."""
import re
import shutil
import struct
import subprocess
from pathlib import Path

import pytest

LIB = Path(__file__).resolve().parent.parent / "paper_2407_14417_amd" / "libmoemix.so"
OBJDUMP = shutil.which("llvm-objdump", path="/opt/rocm/llvm/bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects():
    """The gfx950 objects in the library's offload bundles: magic, count, then (offset, size, length of target, target)."""
    data = LIB.read_bytes()
    at = data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n]:
                yield data[at + offset:at + offset + size]
            p += 24 + n
        at = data.find(MAGIC, at + 1)


@pytest.mark.skipif(OBJDUMP is None or not LIB.exists(), reason="needs llvm-objdump and the built library")
def test_transfers_into_lds_after_lane_reads(tmp_path):
    """A memory instruction needs five wait states after a lane read that wrote its scalar base; the compiler does not count
    them in front of inline assembly.  And M0, which holds the LDS address, is written by scalar instructions only."""
    transfers = 0
    for i, code in enumerate(_code_objects()):
        if b"prefill_kernel" not in code:
            continue
        obj = tmp_path / f"{i}.co"
        obj.write_bytes(code)
        asm = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], capture_output=True, text=True, check=True).stdout
        recent = []                                        # the last instructions: (scalars a lane read wrote, wait states)
        for line in asm.splitlines():
            ins = re.match(r"\s+([a-z]\w+)\s*(.*?)\s*(//.*)?$", line)
            if not ins:
                continue
            name, args = ins.group(1), ins.group(2)
            if name.startswith("global_load_lds"):
                transfers += 1
                lo, hi = map(int, re.search(r"s\[(\d+):(\d+)\]", args).groups())
                states = 0
                for wrote, wait in reversed(recent):
                    if states >= 5:
                        break
                    assert not wrote & {lo, hi}, line
                    states += wait
            dst = re.match(r"s(\d+)", args)
            lane = {int(dst.group(1))} if name in ("v_readlane_b32", "v_readfirstlane_b32") and dst else set()
            assert name.startswith("s_") or not args.startswith("m0,"), line
            recent = recent[-8:] + [(lane, 1 + int(args, 0) if name == "s_nop" else 1)]
    assert transfers > 1000
