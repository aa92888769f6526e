"""Builds the C-ABI library `libhet_cache.so` for gfx950 with hipcc, in-tree.

    python -m paper_2112_07221_amd.build
"""
import hashlib
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
# (source, parts it is compiled in): the parts run side by side; the sources check that they are as many as they have
SOURCES = [("het_cache.hip", 1), ("apply_variants.hip", 8), ("fill_variants.hip", 2)]
OUT = os.path.join(HERE, "libhet_cache.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    # packed-fp32 instructions stay off: plain float code must not be fused into them
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def source_id() -> str:
    """Short hash of the sources the library is built from (the header and everything in csrc/):
    what `het_build_id()` returns, so that a measurement can name the build it was taken on."""
    h = hashlib.sha256()
    files = [os.path.join(HERE, "..", "include", "het_cache.h")]
    files += sorted(os.path.join(HERE, "csrc", f) for f in os.listdir(os.path.join(HERE, "csrc")))
    for f in files:
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:12]


def build(verbose: bool = False, flags=()) -> str:
    with tempfile.TemporaryDirectory() as tmp:
        jobs, objects = [], []
        for name, parts in SOURCES:
            for part in range(parts):
                objects.append(os.path.join(tmp, f"{name}.{part}.o"))
                jobs.append([HIPCC, *FLAGS, *flags, "-c", f'-DHET_BUILD_ID="{source_id()}"', f"-DHET_PART={part}", f"-DHET_PARTS={parts}", os.path.join(CSRC, name), "-o", objects[-1]])
        if verbose:
            print("\n".join(" ".join(j) for j in jobs))
        with ThreadPoolExecutor(max(1, min(len(jobs), os.cpu_count() or 1))) as pool:
            for done in [pool.submit(subprocess.run, j, check=True) for j in jobs]:
                done.result()
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", *objects, "-o", OUT], check=True)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
