"""Build the gfx950 shared library in-tree with hipcc.

    python -m paper_2506_15174_amd.build

Output: paper_2506_15174_amd/lib/libspmm_cdna4.so (C ABI of include/spmm.h).
"""
import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_DIR = os.path.join(HERE, "lib")
LIB_PATH = os.path.join(LIB_DIR, "libspmm_cdna4.so")
# the tensor-level entry (spmm_torch.cpp): a Python extension module beside the library
TORCH_EXT_SOURCE = "spmm_torch.cpp"
TORCH_EXT_PATH = os.path.join(LIB_DIR, "_spmm_torch.so")

SOURCES = ["spmm_kernels.hip", "spmm_tiles.hip", "spmm_strips.hip", "spmm_plan.cpp", "spmm_api.cpp"]
HEADERS = ["spmm_format.h", "spmm_kernels.h", "spmm_plan.h", "spmm_tiles.h", "spmm_strips.h", "spmm_strips_build.h", "spmm_upload.h", "spmm_launch.h", "spmm_places.h"]


ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def _hipcc():
    exe = shutil.which("hipcc") or os.path.join(ROCM, "bin", "hipcc")
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; the library targets gfx950 only")
    return exe


def is_stale():
    if not os.path.exists(LIB_PATH) or not os.path.exists(TORCH_EXT_PATH):
        return True
    t = min(os.path.getmtime(LIB_PATH), os.path.getmtime(TORCH_EXT_PATH))
    deps = [os.path.join(CSRC, f) for f in SOURCES + HEADERS + [TORCH_EXT_SOURCE]]
    deps.append(os.path.join(os.path.dirname(HERE), "include", "spmm.h"))
    return any(os.path.getmtime(d) > t for d in deps)


def _run(cmd, verbose):
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = ("is not a recognized feature for this target", "-Rpass-analysis=kernel-resource-usage")
    import re
    err = "\n".join(ln for ln in res.stderr.splitlines()
                    if not any(n in ln for n in noise) and not re.match(r"^\s*(\d+)?\s*\|", ln))
    if verbose and err:
        print(err)
    if res.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (cmd[0], err))
    return res.stderr


def check_no_spills(remarks):
    """The kernels issue their loads of B rows from inline assembly and await them later
    (an explicit s_waitcnt): a register the compiler spills or copies in between would
    carry stale data.  No instance may therefore use scratch memory at all: the compiler's
    resource remarks (-Rpass-analysis=kernel-resource-usage) must report zero spilled
    VGPRs and SGPRs and a zero scratch size for every kernel.  Returns the number of
    kernels checked; raises with the offenders otherwise."""
    import re
    name, bad, seen = None, [], 0
    for ln in remarks.splitlines():
        m = re.search(r"Function Name: (\S+)", ln)
        if m:
            name = m.group(1)
            seen += 1
            continue
        m = re.search(r"(VGPRs Spill|SGPRs Spill|ScratchSize \[bytes/lane\]): (\d+)", ln)
        if m and name and int(m.group(2)) != 0:
            bad.append("%s: %s = %s" % (name, m.group(1), m.group(2)))
    if seen == 0:
        raise RuntimeError("the compiler printed no resource remarks: the spill check did not run")
    if bad:
        raise RuntimeError("kernel instances use scratch memory (give them a larger register budget "
                           "or a shallower pipeline):\n  " + "\n  ".join(bad))
    return seen


def check_waits_at_barriers(assembly):
    """A kernel that waits for all loads but the youngest n before a barrier (`s_waitcnt vmcnt(n) lgkmcnt(0)`, `s_barrier`) has
    loads to LDS in flight that other waves read behind it: on every way to the wait at least n plain loads must come after the last of those, or
    the barrier lets a stale row through.  Walks the compiler's assembly back from every such wait; returns how many there are, raises where an order is another."""
    import re
    label = re.compile(r"^(\S+):")
    lines = [ln.split(";")[0].strip() for ln in assembly.splitlines()]
    lines = [ln for ln in lines if ln and (not ln.startswith(".") or label.match(ln))]
    at = {label.match(ln).group(1): i for i, ln in enumerate(lines) if label.match(ln)}
    to = {}
    for i, ln in enumerate(lines):
        m = re.match(r"s_c?branch\S*\s+(\S+)", ln)
        if m and m.group(1) in at:
            to.setdefault(at[m.group(1)], []).append(i)
    checked = 0
    for i, ln in enumerate(lines[:-1]):
        m = re.match(r"s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)$", ln)
        if not m or m.group(1) == "0" or lines[i + 1] != "s_barrier":
            continue
        checked += 1
        todo, seen = [(i, int(m.group(1)))], set()
        while todo:
            j, left = todo.pop()
            if left == 0 or (j, left) in seen:
                continue
            seen.add((j, left))
            before = list(to.get(j, []))
            if j > 0 and not re.match(r"s_branch|s_endpgm|s_setpc", lines[j - 1]):
                before.append(j - 1)
            for k in before:
                op = lines[k]
                if re.match(r"s_waitcnt.*vmcnt\(0\)", op):
                    continue  # nothing older is in flight
                if re.match(r"(buffer|global|flat|scratch)_", op):
                    if not re.match(r"(buffer|global)_load", op) or op.endswith(" lds") or "_load_lds" in op:
                        raise RuntimeError("a barrier waits for all but %s loads, and %d before it is `%s`" % (m.group(1), int(m.group(1)) - left + 1, op))
                    todo.append((k, left - 1))
                else:
                    todo.append((k, left))
    return checked


def build(verbose=False):
    """Compile every source for gfx950 and link the shared library.

    The device translation unit goes through hipcc on its own (its fat binary
    is embedded in its object file); host-only units are plain C++; the link is
    an ordinary shared-library link against the HIP runtime."""
    os.makedirs(LIB_DIR, exist_ok=True)
    obj_dir = os.path.join(LIB_DIR, "obj")
    os.makedirs(obj_dir, exist_ok=True)
    hipcc = _hipcc()
    common = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wextra", "-Wno-unused-parameter",
              "-I", CSRC, "-I", os.path.join(ROCM, "include"), "-D__HIP_PLATFORM_AMD__=1"]
    objects = []
    for s in SOURCES:
        obj = os.path.join(obj_dir, os.path.splitext(s)[0] + ".o")
        if s.endswith(".hip"):
            cmd = [hipcc, "--offload-arch=gfx950",
                   # packed-fp32 forms are kept out of the generated code on purpose
                   "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                   "-Rpass-analysis=kernel-resource-usage"]
        else:
            cmd = [hipcc, "-x", "c++"]
        remarks = _run(cmd + common + ["-c", os.path.join(CSRC, s), "-o", obj], verbose)
        if s.endswith(".hip"):
            n = check_no_spills(remarks)
            if verbose:
                print("%s: %d kernel instances, none uses scratch memory" % (s, n))
        if s == "spmm_strips.hip":
            listing = obj[:-2] + ".s"
            _run(cmd + common + ["-S", "--cuda-device-only", os.path.join(CSRC, s), "-o", listing], False)
            with open(listing) as f:
                n = check_waits_at_barriers(f.read())
            os.remove(listing)
            if n < 4:
                raise RuntimeError("%s: of the barriers behind a strip's copy, one in each kernel, %d were found" % (s, n))
            if verbose:
                print("%s: %d barriers that loads may cross, none of them to LDS" % (s, n))
        objects.append(obj)
    _run([hipcc, "-shared", "-fPIC"] + objects +
         ["-L", os.path.join(ROCM, "lib"), "-lamdhip64", "-pthread", "-o", LIB_PATH], verbose)
    build_torch_extension(verbose)
    return LIB_PATH


def build_torch_extension(verbose=False):
    """Compile the tensor-level entry (host code: plain C++ against torch's headers), linked
    to the library beside it.  torch's own copy of the HIP runtime is the one in the process
    (see binding.load), so no runtime is named here."""
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    _run([shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
          "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
          "-I", sysconfig.get_paths()["include"], "-isystem", os.path.join(root, "include"),
          "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"), "-isystem", os.path.join(ROCM, "include"),
          os.path.join(CSRC, TORCH_EXT_SOURCE), "-o", TORCH_EXT_PATH,
          "-L", LIB_DIR, "-lspmm_cdna4", "-Wl,-rpath,$ORIGIN",
          "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip", "-Wl,-rpath," + os.path.join(root, "lib")],
         verbose)
    return TORCH_EXT_PATH


if __name__ == "__main__":
    print(build(verbose=True))
