"""Compile liboz2.so (HIP kernels + C ABI) for gfx950, in-tree."""
import glob
import os
import re
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
    "oz2_calibrate.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "oz2_stage3.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "oz2_stage2_tiles.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "oz2_thin.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


# The large GEMM keeps its accumulators in registers that its inline assembly names (oz2_stage2.hip): v112..v239 and
# a128..a255.  That is sound only while the compiler keeps everything of its own out of them, which no language rule says.
GEMM_SOURCE = "oz2_stage2.hip"
GEMM_KERNEL = "gemm_i8_kernel"
NAMED_VGPR, NAMED_AGPR = 112, 128


def named_register_faults(assembly):
    """Lines of the GEMM kernels' assembly in which the compiler has put a value of its own into an accumulator register or
    into scratch memory, as (kernel, line) pairs; an empty list when all is well."""
    faults, kernel, inside, kernels = [], None, False, 0
    for line in assembly.splitlines():
        label = re.match(r"(\w+):", line)
        if label and GEMM_KERNEL in label.group(1):
            kernel, kernels = label.group(1), kernels + 1
        if kernel is None:
            continue
        if line.startswith(".Lfunc_end"):
            kernel = None
            continue
        if "#ASMSTART" in line or "#ASMEND" in line:
            inside = "#ASMSTART" in line
            continue
        code = line.split(";")[0].split("//")[0].strip()
        if not code or code.startswith("."):
            continue
        # M0 holds the target of the copies into LDS between statements of the source
        if code.startswith(("scratch_", "buffer_load", "buffer_store")) or (not inside and re.search(r"\bm0\b", code)):
            faults.append((kernel, code))
        for found in re.finditer(r"\b([va])(?:(\d+)\b|\[(0x[0-9a-f]+|\d+)(\+\d+)?(?::(0x[0-9a-f]+|\d+))?\])", code):
            kind, single, low, offset, high = found.groups()
            first = int(single or low, 0)
            last = int(high, 0) if high else first
            if kind == "v" and last < NAMED_VGPR:
                continue
            # a statement of the source: a whole tile of four registers, as the result or the accumulator of a product, or one
            # register counted from a tile's first
            base = NAMED_VGPR if kind == "v" else NAMED_AGPR
            named = code[:found.start()].count(",") in (0, 3) if last == first + 3 else offset and int(offset) < 4
            if inside and first >= base and (first - base) % 4 == 0 and named:
                continue
            faults.append((kernel, code))
    if not kernels:
        faults.append((GEMM_KERNEL, "not found"))
    return faults


def start_gemm_listing():
    cmd = ["hipcc"] + HIP_FLAGS + EXTRA_FLAGS.get(GEMM_SOURCE, []) + ["--offload-device-only", "-S", os.path.join(CSRC, GEMM_SOURCE),
                                                                     "-o", "-"]
    return subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL), cmd


def build(verbose=False):
    objs = []
    listing, listing_cmd = start_gemm_listing()
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
    assembly = listing.communicate()[0].decode()
    if listing.returncode:
        raise RuntimeError("compile failed: %s" % " ".join(listing_cmd))
    faults = named_register_faults(assembly)
    if faults:
        raise RuntimeError("%s: the compiler uses registers that the accumulators live in, or scratch memory:\n%s"
                           % (GEMM_SOURCE, "\n".join("%s: %s" % f for f in faults[:20])))
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
