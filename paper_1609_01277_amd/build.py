"""Build libsbli.so (HIP, gfx950) in-tree with hipcc."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libsbli.so")
SOURCES = ["sbli.hip", "closure.hip", "scalar.hip", "staged.hip"] + ["stage_%s_r%d.hip" % (t, r) for t in ("f64", "f32") for r in (1, 2, 3, 4)]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # a*b + c is fused only within one source expression (the hot arithmetic
    # spells its fused multiply-adds out), so rounding never depends on how the
    # compiler schedules a particular kernel variant
    "-ffp-contract=on",
    # packed FP32 instructions stay disabled for every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]

# Per-source additions.  The FP32 order-4 stage kernels issue faster under the
# ILP-first machine scheduler: 10,430 against 9,962 Mpoint-steps/s for the
# autotuned variant at 512^3 (the FP64 kernels gain nothing measurable from it).
# Scheduling never changes results: the arithmetic's fused multiply-adds are
# spelled out in the source (-ffp-contract=on).
# The FP64 order-4 and the staged kernels fill the register file; with the target's own
# register-pressure trackers in the scheduler the plane wavefronts spill nothing (4 to 12
# registers without), and a stage at 256^3, FP64, order 8 takes 1,160 instead of 1,185 us,
# order 12 1,634 instead of 1,653.
SOURCE_FLAGS = {
    "stage_f32_r2.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"],
    "stage_f64_r2.hip": ["-mllvm", "-amdgpu-use-amdgpu-trackers=1"],
    "staged.hip": ["-mllvm", "-amdgpu-use-amdgpu-trackers=1"],
}


STAMP = LIB + ".sources"   # digest of the sources and flags the library was built from


def sources_digest():
    """sha256 over every file under csrc/ and include/, the compiler flags and the
    source list: what a build of libsbli.so depends on."""
    import hashlib
    h = hashlib.sha256()
    h.update(repr((HIPCC_FLAGS, SOURCE_FLAGS, SOURCES)).encode())
    for d in (CSRC, INCLUDE):
        for name in sorted(os.listdir(d)):
            path = os.path.join(d, name)
            if os.path.isfile(path) and not name.startswith("."):
                h.update(name.encode())
                with open(path, "rb") as f:
                    h.update(f.read())
    return h.hexdigest()


def is_current():
    """True when libsbli.so exists and was built from the sources as they are now."""
    try:
        with open(STAMP) as f:
            return os.path.exists(LIB) and f.read().strip() == sources_digest()
    except OSError:
        return False


def hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _clean(text):
    return "\n".join(l for l in text.splitlines() if "packed-fp32-ops" not in l)


def build(verbose=False):
    """Compile every HIP source of the library (in parallel) and link
    paper_1609_01277_amd/libsbli.so."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        objs.append(obj)
        cmd = [hipcc()] + compile_flags + SOURCE_FLAGS.get(src, []) + ["-c", "-I", INCLUDE, "-I", CSRC, "-o", obj, os.path.join(CSRC, src)]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    errors = []
    for src, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0:
            errors.append("%s:\n%s" % (src, _clean(out)))
    if errors:
        raise RuntimeError("hipcc failed:\n" + "\n".join(errors))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + _clean(res.stdout))
    digest = sources_digest()
    os.replace(tmp, LIB)
    with open(STAMP + ".tmp", "w") as f:
        f.write(digest + "\n")
    os.replace(STAMP + ".tmp", STAMP)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    print("built", LIB)
    sys.exit(0)
