"""Compile libq4kv.so (hand-written HIP for gfx950 + the C ABI) in-tree with hipcc."""
import hashlib
import os
import re
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libq4kv.so")
SOURCES = ["api.hip", "codec.hip", "decode_attention.hip", "chunk_attention.hip", "mla_decode.hip", "read_probe.hip", "persist.hip", "block_pool.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# No fast-math anywhere: the quantizer needs IEEE binary32 division and rounding.
# packed-fp32 instruction selection is switched off (some of its forms have given wrong results on this hardware).
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-fno-gpu-sanitize"]
# These kernels read most of their matrix results with vector instructions (scales, softmax), so their matrix
# instructions write vector registers directly instead of accumulator registers that must be copied out first.
VGPR_FORM = ["-mllvm", "-amdgpu-mfma-vgpr-form"]
# What a file is compiled for one by one; once, with nothing defined, where it is not named.
PARTS = {"chunk_attention.hip": [f"-DQ4KV_CHUNK_WIDTH={width}" for width in (256, 192, 128, 64)]}
FILE_FLAGS = {"chunk_attention.hip": VGPR_FORM, "mla_decode.hip": VGPR_FORM}
# Files whose kernels must keep everything in vector registers, and the flags that make the compiler say so.  A chunk kernel that
# spilled gave wild addresses: the spill was behind a divergent loop, where some lanes were still switched off.
NO_SPILLS = ["chunk_attention.hip"]
RESOURCES = ["-Rpass-analysis=kernel-resource-usage", "-fno-caret-diagnostics"]


def spills(remarks):
    """What the compiler's resource remarks say of kernels that use scratch memory, spill or hold values in accumulator registers."""
    found, kernel = [], None
    for name, what, count in re.findall(r"remark: +(?:Function Name: (\S+)|(ScratchSize \[bytes/lane\]|VGPRs Spill|AGPRs): (\d+))", remarks):
        kernel = name or kernel
        if what and int(count):
            found.append(f"{kernel}: {what} {count}")
    return found


def sources_hash():
    """Names a state of everything the library is compiled from; the library carries the one it was built from as text."""
    h = hashlib.sha256(repr([SOURCES, FLAGS, PARTS, FILE_FLAGS]).encode())
    for d in (CSRC, os.path.join(HERE, os.pardir, "include")):
        for name in sorted(os.listdir(d)):
            h.update(name.encode() + b"\0")
            with open(os.path.join(d, name), "rb") as f:
                h.update(f.read())
    return h.hexdigest()


def build(verbose=False):
    stamp = f"q4kv sources {sources_hash()}"
    with tempfile.TemporaryDirectory(prefix="q4kv_build_") as tmp:
        def compile_one(job):
            src, part = job
            obj = os.path.join(tmp, src.replace(".hip", (part or "") + ".o"))
            cmd = [HIPCC] + FLAGS + ([part] if part else []) + FILE_FLAGS.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
            if src in NO_SPILLS:
                cmd += RESOURCES
            if verbose:
                print(" ".join(cmd))
            done = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
            sys.stderr.write("".join(line for line in done.stderr.splitlines(True) if RESOURCES[0][1:] not in line))
            done.check_returncode()
            if src in NO_SPILLS and spills(done.stderr):
                raise RuntimeError(f"{src}: kernels that do not keep everything in registers:\n" + "\n".join(spills(done.stderr)))
            return obj
        jobs = sorted(((src, part) for src in SOURCES for part in PARTS.get(src, [None])), key=lambda job: job[1] is None)  # the long ones first
        with ThreadPoolExecutor(max_workers=min(len(jobs), os.cpu_count() or 1, 8)) as pool:
            objs = list(pool.map(compile_one, jobs))
        with open(os.path.join(tmp, "stamp.c"), "w") as f:
            f.write(f'__attribute__((used)) static const char q4kv_sources[] = "{stamp}";\n')
        objs.append(os.path.join(tmp, "stamp.o"))
        subprocess.check_call([HIPCC, "-x", "c", "-fPIC", "-c", os.path.join(tmp, "stamp.c"), "-o", objs[-1]])
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-sanitize", "-o", LIB] + objs
        if verbose:
            print(" ".join(cmd))
        subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    import sys
    print(build(verbose="-v" in sys.argv))
