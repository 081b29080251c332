"""Compile the HIP library ``libmoemix.so`` for gfx950 with hipcc (in-tree, next to this file)."""
from __future__ import annotations

import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

HERE = Path(__file__).resolve().parent
CSRC = HERE / "csrc"
LIB = HERE / "libmoemix.so"

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]
# the matrix-core kernels of the two projections are compiled side by side
PARTS = {s: (["-DMOEMIX_MFMA_UP"], ["-DMOEMIX_MFMA_DOWN"]) for s in ("ffn_mfma.hip", "ffn_prefill.hip")}


def sources():
    return sorted(CSRC.glob("*.hip"))


def _run(cmd) -> str:
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "packed-fp32-ops"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{err}")
    return err


def build(verbose: bool = False) -> Path:
    """Always recompiles every ``csrc/*.hip`` into ``libmoemix.so``."""
    with tempfile.TemporaryDirectory() as tmp:
        jobs = [(s, part, str(Path(tmp) / f"{s.stem}{i}.o"))
                for s in sources() for i, part in enumerate(PARTS.get(s.name, ([],)))]
        with ThreadPoolExecutor(max_workers=8) as pool:
            errs = list(pool.map(lambda j: _run(["hipcc", *HIPCC_FLAGS, *j[1], "-c", str(j[0]), "-o", j[2]]), jobs))
        errs.append(_run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", str(LIB), *[j[2] for j in jobs]]))
    if verbose and any(e.strip() for e in errs):
        print("\n".join(e for e in errs if e.strip()))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
