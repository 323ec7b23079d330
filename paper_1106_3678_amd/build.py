"""Builds the HIP library libmlbicgstab.so for gfx950 in-tree with hipcc."""
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
# (object, source, flags): the whole-solve kernels compile once per value type
UNITS = [("engine", "mlb_engine.hip", [])] + [
    (f"grid{k}", "mlb_grid.hip", [f"-DMLB_GRID_TYPE={t}"])
    for k, t in enumerate(("double", "float", "cplx<double>", "cplx<float>"))
]
OUT = os.path.join(HERE, "libmlbicgstab.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # no packed-fp32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result",
]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as d:
        # the units compile side by side, then link
        objs = [os.path.join(d, name + ".o") for name, _, _ in UNITS]
        cmds = [[hipcc, *HIPCC_FLAGS, *flags, "-c", "-o", obj, os.path.join(CSRC, src)]
                for (_, src, flags), obj in zip(UNITS, objs)]
        if verbose:
            print("\n".join(" ".join(c) for c in cmds), flush=True)
        procs = [subprocess.Popen(c) for c in cmds]
        if any([p.wait() for p in procs]):
            raise RuntimeError("hipcc failed")
        tmp = OUT + ".tmp"
        subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
