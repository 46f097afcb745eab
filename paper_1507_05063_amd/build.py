"""Build the gfx950 HIP library libexcmg.so in-tree with hipcc."""
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libexcmg.so")
SOURCES = ["excmg.hip", "kernels_cg.hip", "kernels_transfer.hip", "kernels_grad.hip", "kernels_probe.hip"]
ARCH = "gfx950"

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # no packed FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False) -> str:
    # one compiler per source, side by side, then one link
    with tempfile.TemporaryDirectory() as tmp:
        cmds = [["hipcc", *FLAGS, "-c", "-o", os.path.join(tmp, s + ".o"), os.path.join(CSRC, s)] for s in SOURCES]
        if verbose:
            for c in cmds:
                print(" ".join(c), flush=True)
        procs = [subprocess.Popen(c) for c in cmds]
        codes = [p.wait() for p in procs]
        for c, code in zip(cmds, codes):
            if code:
                raise subprocess.CalledProcessError(code, c)
        out = LIB + ".tmp"
        subprocess.run(["hipcc", "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", out, *[c[-2] for c in cmds]],
                       check=True)
    os.replace(out, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
