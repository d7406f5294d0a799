"""Compile the HIP kernels and the C ABI into paper_2601_12212_amd/libdt.so (gfx950 only), the argument marshalling of
the Python binding into paper_2601_12212_amd/_dtcall.so (gcc; finds libdt.so beside itself), and what reads a tensor's
properties for it without the interpreter into _dttensor-<torch's version>.so (g++; against the torch that is installed).
For the tests, both once more with waits that end early (SHORT_WAITS in csrc/hands.hpp), in _build."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdt.so")
PYCALL = os.path.join(HERE, "_dtcall.so")
SOURCES = ["api.cpp", "profile.cpp", "rows.hip", "tree.hip", "attention.hip", "accept.hip", "commit.hip", "policy.hip"]
WAITING = ["rows.hip", "attention.hip"]   # kernels whose workgroups wait for each other
BUILD = os.path.join(HERE, "_build")
LIB_SHORT, PYCALL_SHORT = os.path.join(BUILD, "libdt_short_waits.so"), os.path.join(BUILD, "_dtcall.so")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         # packed-FP32 code generation is switched off: some of its instruction forms have given wrong
         # results on this hardware now and then, without any error
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def build(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    procs = []
    os.makedirs(BUILD, exist_ok=True)
    obj = lambda src, kind="": os.path.join(BUILD, src + kind + ".o")
    for src, kind, more in [(src, "", []) for src in SOURCES] + [(src, ".short_waits", ["-DSHORT_WAITS"]) for src in WAITING]:
        cmd = [hipcc] + FLAGS + more + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj(src, kind)]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
        if verbose and out.strip():
            print(out)
    include = "-I" + sysconfig.get_paths()["include"]
    for lib, pycall, kind in ((LIB, PYCALL, ""), (LIB_SHORT, PYCALL_SHORT, ".short_waits")):
        tmp = lib + ".tmp%d" % os.getpid()
        subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] +
                              [obj(src, kind if src in WAITING else "") for src in SOURCES])
        os.replace(tmp, lib)
        tmp = pycall + ".tmp%d" % os.getpid()
        subprocess.check_call(["gcc", "-O2", "-shared", "-fPIC", "-Wall", include, os.path.join(CSRC, "pycall.c"), "-o", tmp,
                               "-L" + os.path.dirname(lib), "-l:" + os.path.basename(lib), "-Wl,-rpath,$ORIGIN"])
        os.replace(tmp, pycall)
    build_reader(include)
    return LIB


def reader_path(torch_version):
    """Where the tensor reader built against that torch is."""
    return os.path.join(HERE, "_dttensor-%s.so" % torch_version)


def build_reader(include):
    try:
        import torch
    except ImportError:
        print("no torch here: tensors will be read through their methods")
        return
    tdir = os.path.dirname(torch.__file__)
    path = reader_path(torch.__version__)
    tmp = path + ".tmp%d" % os.getpid()
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", include,
                           "-isystem", os.path.join(tdir, "include"),
                           "-isystem", os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
                           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch.compiled_with_cxx11_abi(),
                           os.path.join(CSRC, "tensor_reader.cpp"), "-o", tmp,
                           "-L" + os.path.join(tdir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"])
    os.replace(tmp, path)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
