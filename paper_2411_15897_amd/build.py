"""Build the native library libehelm.so in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libehelm.so")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(HERE, "csrc"),
]


# translation units: (source, extra flags); the multigrid kernels are compiled
# per precision (the fused legs per leg too), side by side with the host driver
UNITS = [("ehelm.hip", [])]
UNITS += [("eh_fused.hip", ["-DEH_T=" + t, "-DEH_UP=%d" % up]) for t in ("float", "double") for up in (0, 1)]
UNITS += [("eh_sweep.hip", ["-DEH_T=" + t]) for t in ("float", "double")]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        objs, procs = [], []
        try:
            for i, (src, extra) in enumerate(UNITS):
                obj = os.path.join(tmp, "%d.o" % i)
                cmd = [hipcc, "-c"] + FLAGS + extra + [os.path.join(CSRC, src), "-o", obj]
                objs.append(obj)
                procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
            outs = [p.communicate()[0] for _, p in procs]
        finally:
            for _, p in procs:
                if p.poll() is None:
                    p.kill()
                    p.wait()
        so = OUT + ".tmp"
        if all(p.returncode == 0 for _, p in procs):
            res = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", so],
                                 capture_output=True, text=True)
            outs.append(res.stdout + res.stderr)
            failed = res.returncode != 0
        else:
            failed = True
        if failed:
            sys.stderr.write("".join(outs))
            raise RuntimeError("hipcc failed to build libehelm.so")
        if verbose:
            sys.stderr.write("".join(outs))
        os.replace(so, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
