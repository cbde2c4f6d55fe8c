"""Build the HIP library liblbm.so for gfx950 with hipcc (in-tree, next to this file)."""
import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblbm.so")

SOURCES = ["lbm_api.hip", "host_copy.hip", "bgk.hip", "bgk_multi.hip", "bgk3_multi.hip", "ddf.hip", "ddf_pair.hip", "ddf3.hip", "reduced.hip", "mlp.hip", "copy.hip"]

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # no packed-FP32 instructions (v_pk_*_f32) anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]

# Per-source additions. mlp.hip: matrix-core results in ordinary vector registers (no copy out
# of the accumulation registers after every tile; the surrogate step reads each result once).
SOURCE_FLAGS = {
    "mlp.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=true"],
}


def hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    return "hipcc"


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed (exit %d): %s" % (res.returncode, cmd[-3]))


def build(verbose=False):
    """Compile each source to an object in parallel (no device code crosses files), then link.
    LBM_EXTRA_HIPCC_FLAGS (environment) adds flags, e.g. -DLBM_TUNING_ENV for launch-shape
    sweeps through environment variables."""
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    inc += os.environ.get("LBM_EXTRA_HIPCC_FLAGS", "").split()
    tmpdir = tempfile.mkdtemp(prefix="lbm_build_")
    try:
        objs = [os.path.join(tmpdir, os.path.splitext(s)[0] + ".o") for s in SOURCES]
        cmds = [[hipcc()] + FLAGS + SOURCE_FLAGS.get(s, []) + inc
                + ["-c", os.path.join(CSRC, s), "-o", o]
                for s, o in zip(SOURCES, objs)]
        workers = max(1, min(len(cmds), os.cpu_count() or 1, 8))
        with ThreadPoolExecutor(workers) as ex:
            list(ex.map(lambda c: _run(c, verbose), cmds))
        tmp = LIB + ".tmp"
        _run([hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950"] + objs + ["-o", tmp], verbose)
        os.replace(tmp, LIB)
    finally:
        shutil.rmtree(tmpdir, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
