"""Build step of the HIP library (hipcc, gfx950).  Used by __graft_entry__.build()."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
# (object, source, defines): the fixed-length pencil passes compile in groups
# of lengths side by side
JOBS = [("rpm_solver", "rpm_solver.hip", ["-DRPM_PENCIL_SEPARATE"]), ("rpm_fno", "rpm_fno.hip", [])] + [
    (f"rpm_pencil{k}", "rpm_pencil.hip", [f"-DRPM_PENCIL_GROUP={k}"]) for k in range(6)]
OUT = os.path.join(HERE, "librpmfft.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed FP32 instructions stay off: plain scalar/float2 code only
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result", "-Wno-unused-value",
]


def build(verbose=False):
    inc = ["-I", os.path.join(ROOT, "include")]
    objs = [os.path.join(CSRC, name + ".o") for name, _, _ in JOBS]
    procs = []
    for (_, src, defs), obj in zip(JOBS, objs):
        cmd = ["hipcc"] + HIPCC_FLAGS + defs + inc + ["-c", "-o", obj, os.path.join(CSRC, src)]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append(subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True))
    for p in procs:
        _, err = p.communicate()
        if p.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + err[-8000:])
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT + ".tmp"] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    for obj in objs:  # intermediate objects do not travel with the tree
        if os.path.exists(obj):
            os.remove(obj)
    if r.returncode != 0:
        raise RuntimeError("hipcc link failed:\n" + r.stderr[-8000:])
    os.replace(OUT + ".tmp", OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
