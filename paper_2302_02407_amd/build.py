"""Build the HIP library in-tree: python -m paper_2302_02407_amd.build [--incremental]"""
import os
import re
import shutil
import subprocess
import sys
import tempfile
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


def device_listing(hipcc, obj):
    """The assembly of an object's kernels, line by line; empty where it has none."""
    tools = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(shutil.which(hipcc) or hipcc))), "llvm", "bin")
    if not os.path.isdir(tools):
        tools = "/opt/rocm/llvm/bin"
    with tempfile.TemporaryDirectory() as tmp:
        fat, dev = os.path.join(tmp, "fat"), os.path.join(tmp, "dev")
        headers = _run([os.path.join(tools, "llvm-objdump"), "-h", obj], False)
        if not any(".hip_fatbin " in l for l in headers):
            return []
        _run([os.path.join(tools, "llvm-objcopy"), "--dump-section", ".hip_fatbin=" + fat, obj, os.devnull], False)
        _run([os.path.join(tools, "clang-offload-bundler"), "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--input=" + fat, "--output=" + dev], False)
        return _run([os.path.join(tools, "llvm-objdump"), "-d", "--no-show-raw-insn", dev], False)


def ieee_kernels(listing):
    """Kernels of a listing that take a minimum of doubles without having switched the wavefront's IEEE mode off before their first branch
    (csub_min and ieee_off, modarith.h)."""
    found, name, entry, off = [], None, True, False
    for l in listing:
        m = re.match(r"[0-9a-f]+ <(.*)>:$", l)
        if m:
            name, entry, off = m.group(1), True, False
        elif "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 9, 1), 0" in l:
            off = off or entry
        elif re.match(r"\s+s_c?branch", l):
            entry = False
        elif "v_min_f64" in l and not off and name not in found:
            found.append(name)
    return found


def compile_object(hipcc, src, obj, extra=(), verbose=False):
    """One source to one object; where a kernel is refused that is an error and the object is not kept.  Refused are kernels that use scratch
    memory (registers spilled, an array indexed at run time): one that spilled has given wrong results on this GPU, for a reason that
    is not known (ksrows.hip).  And kernels with conditional subtractions by csub_min in a mode in which its minimum of a number and a
    signalling pattern is not the number."""
    lines = _run([hipcc] + FLAGS + list(extra) + ["-c", src, "-o", obj], verbose)
    bad = scratch_kernels(lines)
    if bad:
        os.remove(obj)
        raise RuntimeError("%s: kernels that use scratch memory: %s" % (os.path.basename(src), ", ".join(
            "%s (%s)" % (n, "dynamic" if b is None else "%d bytes a lane" % b) for n, b in bad)))
    bad = ieee_kernels(device_listing(hipcc, obj))
    if bad:
        os.remove(obj)
        raise RuntimeError("%s: kernels that use csub_min and do not start with ieee_off(): %s" % (os.path.basename(src), ", ".join(bad)))


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
