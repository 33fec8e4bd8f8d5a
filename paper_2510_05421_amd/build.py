"""Build libdvi.so (the HIP engine) for gfx950 with hipcc, in-tree."""
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SO = os.path.join(HERE, "libdvi.so")
SOURCES = [os.path.join(HERE, "csrc", f) for f in ("kernels.hip", "prefill.hip", "engine.hip")]
ARCH = os.environ.get("DVI_OFFLOAD_ARCH", "gfx950")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC",
    "--offload-arch=" + ARCH,
    # never emit packed-fp32 VALU ops (v_pk_*_f32) in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


def build(verbose: bool = False) -> str:
    """Compile the sources side by side, then link them into libdvi.so."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = SO + ".tmp%d" % os.getpid()
    with tempfile.TemporaryDirectory() as d:
        objs = [os.path.join(d, os.path.basename(s) + ".o") for s in SOURCES]
        jobs = [[hipcc] + HIPCC_FLAGS + ["-c", s, "-o", o] for s, o in zip(SOURCES, objs)]
        procs = [subprocess.Popen(c, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True) for c in jobs]
        outs = [p.communicate()[0] for p in procs]
        link = [hipcc] + HIPCC_FLAGS + ["-shared"] + objs + ["-o", tmp]
        if all(p.returncode == 0 for p in procs):
            r = subprocess.run(link, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            procs.append(r)
            outs.append(r.stdout)
    if verbose:
        print("\n".join(" ".join(c) for c in jobs + [link]), flush=True)
    errs = "\n".join(l for o in outs for l in o.splitlines()
                     if "packed-fp32-ops' is not a recognized feature" not in l)
    if any(p.returncode != 0 for p in procs):
        raise RuntimeError("hipcc failed:\n" + errs)
    if verbose and errs.strip():
        print(errs, file=sys.stderr)
    os.replace(tmp, SO)
    return SO


if __name__ == "__main__":
    print(build(verbose=True))
