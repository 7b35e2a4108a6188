"""Build the HIP library in-tree: python -m paper_2302_02407_amd.build [--incremental]"""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libhe_mi355x.so")
SOURCES = ["ctx.hip", "ntt.hip", "ntt2p.hip", "colconv.hip", "ksrows.hip", "rescale.hip", "elementwise.hip", "keyswitch.hip", "conv2d.hip", "noalloc.hip", "smallring.hip"]
HEADERS = ["he_internal.h", "modarith.h", "ntt_blocks.h", os.path.join("..", "..", "include", "he_mi355x.h")]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
         "-Rpass-analysis=kernel-resource-usage"]
REPORT = re.compile(r"remark: .*\[-Rpass-analysis=kernel-resource-usage\]")
FIELD = re.compile(r"remark: (?:\S+:\d+:\d+: )?\s*([A-Za-z][\w /\[\]]*): (\S+) \[-Rpass-analysis")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    lines, out = [l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l and l.strip()], []
    for l in lines:                                      # without the resource report and the source lines quoted under it
        if REPORT.search(l):
            out.append(None)
        elif not (out and out[-1] is None and re.match(r" *\d* \|", l)):
            out.append(l)
    text = "\n".join(l for l in out if l is not None)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + text)
    if verbose and text:
        print(text)
    return lines


def scratch_kernels(lines):
    """(kernel, bytes a lane) of the kernels that a resource report shows to use scratch memory; None: an amount that is only known
    when they run."""
    found, name = [], None
    for l in lines:
        m = FIELD.search(l)
        if not m:
            continue
        if m.group(1) == "Function Name":
            name = m.group(2)
        elif m.group(1).startswith("ScratchSize") and m.group(2) != "0":
            found.append((name, int(m.group(2))))
        elif m.group(1) == "Dynamic Stack" and m.group(2) != "False":
            found.append((name, None))
    return found


def compile_object(hipcc, src, obj, extra=(), verbose=False):
    """One source to one object.  A kernel that uses scratch memory (registers spilled, an array indexed at run time) is an error, and its
    object is not kept: one that spilled has given wrong results on this GPU, for a reason that is not known (ksrows.hip)."""
    lines = _run([hipcc] + FLAGS + list(extra) + ["-c", src, "-o", obj], verbose)
    bad = scratch_kernels(lines)
    if bad:
        os.remove(obj)
        raise RuntimeError("%s: kernels that use scratch memory: %s" % (os.path.basename(src), ", ".join(
            "%s (%s)" % (n, "dynamic" if b is None else "%d bytes a lane" % b) for n, b in bad)))


def source_hash() -> str:
    """sha256 over the library's sources and headers (the build identifier compiled into the library)."""
    import hashlib
    h = hashlib.sha256()
    for name in sorted(SOURCES) + sorted(HEADERS):
        with open(os.path.join(CSRC, name), "rb") as f:
            h.update(name.encode() + b"\0" + f.read())
    return h.hexdigest()[:16]


def build_library(verbose: bool = True, incremental: bool = False) -> str:
    """Compile every HIP source for gfx950 (one object per source, in parallel) and link them into one
    shared library next to this file.  incremental=True skips objects newer than their source and the
    headers."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    newest_header = max(os.path.getmtime(os.path.join(CSRC, h)) for h in HEADERS)
    jobs = []
    build_id = source_hash()
    for s in SOURCES:
        src, obj = os.path.join(CSRC, s), os.path.join(OBJ, s + ".o")
        if incremental and s != "ctx.hip" and os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(src), newest_header):
            continue
        extra = ['-DHE_BUILD_ID="%s"' % build_id] if s == "ctx.hip" else []
        jobs.append((src, obj, extra))
    with ThreadPoolExecutor(max_workers=8) as ex:
        list(ex.map(lambda j: compile_object(hipcc, *j, verbose=verbose), jobs))
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc"] + [os.path.join(OBJ, s + ".o") for s in SOURCES]
         + ["-o", LIB], verbose)
    return LIB


if __name__ == "__main__":
    build_library(incremental="--incremental" in sys.argv[1:])
    sys.exit(0)
