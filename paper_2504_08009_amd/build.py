"""Compile liboz2.so (HIP kernels + C ABI) for gfx950, in-tree."""
import glob
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liboz2.so")

HIP_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result",
]


# Per-file additions.  The CRT kernels use the matrix cores for a few instructions among vector arithmetic on their
# results, and the small-tile and thin GEMMs need fewer than 256 registers in all: there the MFMA results belong in ordinary
# vector registers (otherwise every result is copied out of the accumulation registers, and the accumulator start copied
# in, one instruction per register).
EXTRA_FLAGS = {
    "oz2_stage3.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "oz2_stage2_tiles.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "oz2_thin.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def build(verbose=False):
    objs = []
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    procs = []
    for src in sources():
        obj = os.path.join(bdir, os.path.basename(src) + ".o")
        cmd = ["hipcc"] + HIP_FLAGS + EXTRA_FLAGS.get(os.path.basename(src), []) + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd))
        procs.append((subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT), cmd))
        objs.append(obj)
    for proc, cmd in procs:
        out, _ = proc.communicate()
        text = "\n".join(l for l in out.decode().splitlines() if "packed-fp32-ops" not in l)
        if proc.returncode:
            raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), text))
        if verbose and text.strip():
            print(text)
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
