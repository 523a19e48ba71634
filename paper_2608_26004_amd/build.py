"""Build libasymspec.so (gfx950) in-tree with hipcc."""

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "build")
INC = os.path.join(ROOT, "include")
OUT = os.path.join(HERE, "libasymspec.so")
# per-kernel register and scratch use reported by the compiler for the last
# build (a kernel that spills to scratch loses most of its read rate)
RESOURCES = os.path.join(HERE, "libasymspec.resources.txt")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from emitting packed-FP32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=off",
    "-Wall", "-Wno-unused-function",
]


def units():
    """(object name, source, defines) of every object of the library: the host
    side, the cross-family kernels per storage type, and one object per
    instance of the decision kernel (storage type x source of delta x variant),
    compiled in parallel."""
    out = [("asymspec", "asymspec.hip", [])]
    for dt in (0, 1):
        out.append((f"xv_{dt}", "xvocab.hip", [f"-DASYMSPEC_PART_DT={dt}"]))
        for dm in (0, 1, 2):
            for var in (0, 1, 2, 3):
                out.append((f"fv_{dt}{dm}{var}", "kernels.hip",
                            [f"-DASYMSPEC_PART_DT={dt}", f"-DASYMSPEC_PART_DM={dm}", f"-DASYMSPEC_PART_VAR={var}"]))
    return out


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    lines = (r.stdout + r.stderr).splitlines()
    usage = [l for l in lines if "kernel-resource-usage" in l]
    msg = "\n".join(l for l in lines if "packed-fp32-ops" not in l and "unknown target feature" not in l
                    and "kernel-resource-usage" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed ({r.returncode}): {' '.join(cmd)}\n{msg}")
    return usage, msg


def build(verbose: bool = False, extra=()) -> str:
    os.makedirs(OBJ, exist_ok=True)

    def compile_one(unit):
        name, src, defs = unit
        obj = os.path.join(OBJ, name + ".o")
        return obj, *_run([HIPCC, *FLAGS, "-c", "-Rpass-analysis=kernel-resource-usage",
                           "-fno-caret-diagnostics", *defs, *extra, "-I", INC, os.path.join(CSRC, src), "-o", obj])

    jobs = int(os.environ.get("MAX_JOBS", 0)) or len(os.sched_getaffinity(0))
    with ThreadPoolExecutor(max(1, min(jobs, 16))) as pool:
        done = list(pool.map(compile_one, units()))
    tmp = OUT + ".tmp"
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *(d[0] for d in done), "-o", tmp])
    if verbose:
        print("\n".join(d[2] for d in done if d[2].strip()))
    os.replace(tmp, OUT)
    with open(RESOURCES, "w") as f:
        f.write(resource_report([l for d in done for l in d[1]]))
    return OUT


def resource_report(lines) -> str:
    """One line per kernel: name, VGPRs, scratch bytes per lane, occupancy."""
    rows, cur = [], {}
    for l in lines:
        txt = l.split("remark:", 1)[-1].split("[-Rpass", 1)[0].strip()
        key, _, val = txt.partition(":")
        key, val = key.strip(), val.strip()
        if key == "Function Name":
            if cur:
                rows.append(cur)
            cur = {"name": val}
        elif key in ("VGPRs", "ScratchSize [bytes/lane]", "Occupancy [waves/SIMD]"):
            cur[key.split()[0]] = val
    if cur:
        rows.append(cur)
    return "".join(f"{r['name']} vgprs={r.get('VGPRs', '?')} scratch={r.get('ScratchSize', '?')} "
                   f"occupancy={r.get('Occupancy', '?')}\n" for r in rows)


EXAMPLE_SRC = os.path.join(HERE, "examples", "fuse_verify_c.cpp")
EXAMPLE = os.path.join(HERE, "examples", "fuse_verify_c")


def build_example(verbose: bool = False) -> str:
    """The C-ABI example, a host program linked against libasymspec.so."""
    cmd = [HIPCC, "--offload-arch=gfx950", "-O2", "-std=c++17", "-I", INC, EXAMPLE_SRC,
           "-L", HERE, "-lasymspec", f"-Wl,-rpath,{HERE}", "-o", EXAMPLE]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"example build failed ({r.returncode}):\n{r.stdout}{r.stderr}")
    if verbose:
        print(f"built {EXAMPLE}")
    return EXAMPLE


PROBE_SRC = os.path.join(HERE, "csrc", "probe.hip")
PROBE = os.path.join(HERE, "libasymspec_probe.so")


def build_probe(verbose: bool = False) -> str:
    """libasymspec_probe.so: the read-ceiling probe (not the decision step)."""
    tmp = PROBE + ".tmp"
    cmd = [HIPCC, *FLAGS, "-shared", "-I", INC, PROBE_SRC, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"probe build failed ({r.returncode}):\n{r.stdout}{r.stderr}")
    os.replace(tmp, PROBE)
    if verbose:
        print(f"built {PROBE}")
    return PROBE


if __name__ == "__main__":
    print(build(verbose=True))
    build_example(verbose=True)
    build_probe(verbose=True)
    sys.exit(0)
