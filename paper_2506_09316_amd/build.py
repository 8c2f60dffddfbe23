"""Builds libdsla.so (the C-ABI library) from csrc/ with hipcc for gfx950, and _marshal.so (its hot calls for
binding.py) with g++ against the headers of PyTorch and Python, in-tree.  The library needs neither of the two and
the binding does without _marshal.so where it is not built.

The translation units are compiled in parallel and linked into
paper_2506_09316_amd/libdsla.so.  hipcc cross-compiles without a GPU.
"""
import hashlib
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdsla.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
SOURCES = ["api.hip", "decode.hip", "attention.hip", "attention_prefill.hip", "controller.hip", "project.hip", "prefill_short.hip", "prefill.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    # hipcc must not form packed fp32 instructions on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def marshal_stamp():
    """What _marshal.so was built for has to be what it is loaded in: its calls rely on the header and on these versions."""
    import torch
    with open(os.path.join(ROOT, "include", "dsla.h"), "rb") as f:
        header = hashlib.sha256(f.read()).hexdigest()[:16]
    return f"python {sys.version_info[0]}.{sys.version_info[1]}, torch {torch.__version__}, dsla.h {header}"


def _marshal_command():
    import torch
    root = os.path.dirname(torch.__file__)
    include = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
               sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    return ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-w",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DDSLA_BUILT_FOR="{marshal_stamp()}"', *[x for i in include for x in ("-isystem", i)],
            os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL, "-L" + os.path.join(root, "lib"), "-lc10", "-ltorch_cpu", "-ltorch_python"]


def build(verbose: bool = False, extra_flags=()) -> str:
    objs, procs = [], []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = [HIPCC, *FLAGS, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    if os.path.exists(MARSHAL):   # (one that is left is that of this build)
        os.remove(MARSHAL)
    try:
        procs.append(("marshal.cpp", subprocess.Popen(_marshal_command(), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    except (ImportError, OSError) as e:
        sys.stderr.write(f"--- marshal.cpp ---\n{e}\n")
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            failed = failed or src != "marshal.cpp"
            sys.stderr.write(f"--- {src} failed ---\n{out}\n")
        elif verbose and out.strip():
            sys.stderr.write(f"--- {src} ---\n{out}\n")
    if failed:
        raise RuntimeError("compilation failed")
    link = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(link, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
