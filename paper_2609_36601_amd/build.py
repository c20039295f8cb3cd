"""Builds libsaki.so (the gfx950 HIP library behind include/saki.h) in-tree."""
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libsaki.so")
CSRC = os.path.join(HERE, "csrc")
# (source, defines): the units of the library, compiled in parallel
UNITS = [("saki.hip", [])] + [("couple.hip", [f"-DSAKI_PART={p}"]) for p in range(4)] + \
        [("verify.hip", [f"-DSAKI_PART={p}"]) for p in range(2)]

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    # no packed FP32 instructions (v_pk_*_f32) in any kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no machine-level hoisting of loop invariants: in the persistent kernels it
    # lifts the double constants of the per-row serial math (log / exp
    # coefficients) out of the row loop, where they stay live across the
    # sweeps and are spilled to scratch, then reloaded at memory latency in the
    # serial steps of every row
    "-mllvm", "-disable-machine-licm",
]


def hipcc():
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    path = os.path.join(rocm, "bin", "hipcc")
    return path if os.path.exists(path) else "hipcc"


def build(verbose=False):
    """Compile libsaki.so for gfx950 (always recompiles)."""
    with tempfile.TemporaryDirectory(prefix="saki_build_") as tmp:
        jobs = []
        for i, (src, defines) in enumerate(UNITS):
            obj = os.path.join(tmp, f"{i}.o")
            cmd = [hipcc()] + HIPCC_FLAGS + defines + ["-c", os.path.join(CSRC, src), "-o", obj]
            jobs.append((obj, subprocess.Popen(cmd, cwd=HERE, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                                               text=True)))
        logs = [p.communicate()[0] for _, p in jobs]
        ok = all(p.returncode == 0 for _, p in jobs)
        out = LIB + ".tmp"
        if ok:
            res = subprocess.run([hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC"] + [o for o, _ in jobs] +
                                 ["-o", out], cwd=HERE, capture_output=True, text=True)
            logs.append(res.stdout + res.stderr)
            ok = res.returncode == 0
    text = "\n".join(l for l in "\n".join(logs).splitlines() if "packed-fp32-ops" not in l)
    if not ok:
        sys.stderr.write(text)
        raise RuntimeError("hipcc failed building libsaki.so")
    if verbose and text.strip():
        print(text)
    os.replace(out, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
