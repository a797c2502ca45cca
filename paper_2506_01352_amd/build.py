"""Compile csrc/*.hip into libtahq.so (gfx950) next to this file."""
import glob
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = [os.path.join(HERE, "csrc", name) for name in ("tahq.hip", "tahq_rank_quant.hip")]
LIB = os.path.join(HERE, "libtahq.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -ffp-contract=off: the numerics contract allows fused multiply-adds only where the source writes them.
# packed-fp32-ops is switched off for the device pass (the host pass warns that it does not know the feature).
# amdgpu-kernarg-preload-count: the first words of a kernel's arguments are in scalar registers when its wavefronts start.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wextra",
    "-I" + os.path.join(ROOT, "include"),
]


def _newest_input():
    """When the sources, or the headers that nearly all of the code is in, were last changed."""
    headers = glob.glob(os.path.join(HERE, "csrc", "*.hpp")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    return max(os.path.getmtime(path) for path in SOURCES + headers)


def build(force=True):
    if not force and os.path.exists(LIB) and os.path.getmtime(LIB) >= _newest_input():
        return LIB
    # a compiler for each source, side by side
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, os.path.basename(src) + ".o") for src in SOURCES]
        running = [subprocess.Popen([HIPCC] + FLAGS + ["-c", src, "-o", obj]) for src, obj in zip(SOURCES, objects)]
        codes = [p.wait() for p in running]
        if any(codes):
            raise subprocess.CalledProcessError(next(c for c in codes if c), HIPCC)
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared"] + objects + ["-o", LIB], check=True)
    return LIB


if __name__ == "__main__":
    print(build())
