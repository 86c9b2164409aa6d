"""Build paper_2506_05632_amd/libllc_hip.so for gfx950 with hipcc (cross-compiles without a GPU)."""
import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

from .binding import OUTPUTS_PATH

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libllc_hip.so")
PROBE_LIB = os.path.join(HERE, "libllc_probe.so")   # machine probes for bench.py --workload peaks
SOURCES = ["api.hip", "static_scratch.hip", "finalize.hip", "topm.hip", "lml.hip", "scan_f32_shared.hip", "scan_f32_perk.hip",
           "scan_bf16_shared.hip", "scan_bf16_perk.hip", "scan_f32_shared_minf.hip", "scan_f32_perk_minf.hip",
           "scan_bf16_shared_minf.hip", "scan_bf16_perk_minf.hip"]
HEADERS = ["common.hpp", "scan.hpp", "finalize_row.hpp", "lml_search.hpp", os.path.join("..", "..", "include", "llc.h")]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _newest_header():
    return max(os.path.getmtime(os.path.join(CSRC, h)) for h in HEADERS)


def _build_outputs(run):
    """The one piece that knows torch's C++ side; host code only."""
    import torch
    from torch.utils import cpp_extension
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    include = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"]]
    for other in glob.glob(os.path.join(HERE, "_outputs*.so")):  # (of another torch or Python)
        os.remove(other)
    run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
         *("-isystem" + i for i in include), os.path.join(CSRC, "outputs.cpp"), "-o", OUTPUTS_PATH,
         "-L" + lib, "-lc10", "-ltorch_cpu", "-ltorch", "-ltorch_python"])


def build(force: bool = False, verbose: bool = False, extra_flags=()) -> str:
    os.makedirs(OBJ, exist_ok=True)
    hipcc = _hipcc()
    hdr = _newest_header()
    jobs = []
    for src in SOURCES:
        s = os.path.join(CSRC, src)
        o = os.path.join(OBJ, src.replace(".hip", ".o"))
        stale = force or not os.path.exists(o) or os.path.getmtime(o) < max(os.path.getmtime(s), hdr)
        if stale:
            jobs.append([hipcc, *FLAGS, *extra_flags, "-c", s, "-o", o])

    def run(cmd):
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed: " + " ".join(cmd) + "\n" + r.stdout + err)
        if verbose and err.strip():
            print(err, file=sys.stderr)

    with ThreadPoolExecutor(max_workers=min(6, max(1, len(jobs)))) as ex:
        list(ex.map(run, jobs))
    objs = [os.path.join(OBJ, s.replace(".hip", ".o")) for s in SOURCES]
    if jobs or not os.path.exists(LIB):
        run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB])
    probe_src = os.path.join(CSRC, "probe.hip")
    if force or not os.path.exists(PROBE_LIB) or os.path.getmtime(PROBE_LIB) < os.path.getmtime(probe_src):
        run([hipcc, *FLAGS, *extra_flags, "-shared", probe_src, "-o", PROBE_LIB])
    outputs_src = os.path.join(CSRC, "outputs.cpp")
    if force or not os.path.exists(OUTPUTS_PATH) or os.path.getmtime(OUTPUTS_PATH) < os.path.getmtime(outputs_src):
        _build_outputs(run)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
