"""Build the gfx950 shared library in-tree (hipcc for the kernels, g++ for the host-only
selector).  Usage: python -m paper_2512_04226_amd.build [-f]
With --out LIB [-DNAME=VALUE ...] it builds a second library with extra kernel defines
somewhere else, e.g. the builds `calibrate.py --loop-forms` compares:
  python -m paper_2512_04226_amd.build --out /tmp/lf0.so -DG355_FORCE_LOOP_FORM=0"""
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libgemm355.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
             "-packed-fp32-ops", "-Wno-unused-command-line-argument"]
HOST_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-Wall", "-Wextra"]
EXT_SRC = os.path.join(PKG, "pyext", "fastcall.cpp")
EXT = os.path.join(PKG, "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX"))   # (another Python does not take it for its own)


def _sources():
    hip = sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))
    host = sorted(f for f in os.listdir(CSRC) if f.endswith(".cpp"))
    return hip, host


def _deps_mtime():
    return max(os.path.getmtime(os.path.join(CSRC, f)) for f in os.listdir(CSRC)
               if f.endswith((".hpp", ".inc", ".h"))) if os.path.isdir(CSRC) else 0


def _compile(src, force, obj_dir=None, defines=()):
    obj = os.path.join(obj_dir or OBJ, src + ".o")
    path = os.path.join(CSRC, src)
    newest = max(os.path.getmtime(path), _deps_mtime(),
                 os.path.getmtime(os.path.join(PKG, "..", "include", "gemm.h")))
    if not force and os.path.exists(obj) and os.path.getmtime(obj) >= newest:
        return obj, False
    if src.endswith(".hip"):
        cmd = [HIPCC] + HIP_FLAGS + list(defines) + ["-c", path, "-o", obj]
    else:
        cmd = ["g++"] + HOST_FLAGS + ["-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), r.stderr))
    return obj, True


def _hip_include():
    """The headers beside the compiler, which HIPCC may name by a path, a link or a name on PATH."""
    found = shutil.which(HIPCC) or HIPCC
    for path in (found, os.path.realpath(found)):
        include = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(path))), "include")
        if os.path.exists(os.path.join(include, "hip", "hip_runtime.h")):
            return include
    return "/opt/rocm/include"


def build_extension(force=False):
    """The Python extension of api.matmul's short way, against the installed torch, whose version it carries.  Built again when
    its source, the header or the command (torch, Python, paths) is another."""
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = EXT + ".%d.tmp" % os.getpid()
    cmd = (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", '-DFASTCALL_TORCH="%s"' % torch.__version__,
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch.compiled_with_cxx11_abi(), "-isystem", os.path.join(root, "include"), "-isystem",
            os.path.join(root, "include", "torch", "csrc", "api", "include"), "-isystem", sysconfig.get_paths()["include"], "-isystem",
            _hip_include(), EXT_SRC, "-o", tmp, "-L" + os.path.join(root, "lib")] +
           ["-l" + x for x in ("c10", "c10_hip", "torch_cpu", "torch_hip", "torch", "torch_python")])
    header = os.path.join(PKG, "..", "include", "gemm.h")
    stamp, same = os.path.join(OBJ, "fastcall.cmd"), " ".join(cmd).replace(tmp, EXT)
    if (not force and os.path.exists(EXT) and os.path.exists(stamp) and open(stamp).read() == same and
            os.path.getmtime(EXT) >= max(os.path.getmtime(EXT_SRC), os.path.getmtime(header))):
        return EXT
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("extension build failed: %s\n%s" % (" ".join(cmd), r.stderr))
    os.replace(tmp, EXT)
    os.makedirs(OBJ, exist_ok=True)
    with open(stamp, "w") as f:
        f.write(same)
    return EXT


def build(force=False, jobs=8, out=None, defines=(), strict=False):
    """out / defines: build another library (always from scratch, objects beside it) with extra
    -D options for the kernels; the in-tree library is the default.  strict: an extension that cannot be
    built is an error too (it needs torch's headers, which the library does not), else it is reported."""
    lib = os.path.abspath(out) if out else LIB
    obj_dir = lib + ".obj" if out else OBJ
    force = force or bool(out)
    os.makedirs(obj_dir, exist_ok=True)
    hip, host = _sources()
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        extension = None if out else ex.submit(build_extension, force)
        res = list(ex.map(lambda s: _compile(s, force, obj_dir, defines), hip + host))
    objs = [o for o, _ in res]
    if force or any(changed for _, changed in res) or not os.path.exists(lib):
        tmp = lib + ".%d.tmp" % os.getpid()
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed: %s\n%s" % (" ".join(cmd), r.stderr))
        os.replace(tmp, lib)
    if extension is not None:
        try:
            extension.result()
        except Exception as e:
            if strict:
                raise
            print("the library is built, api.matmul's compiled short way is not (its calls go the general way): %s" % e, file=sys.stderr)
    return lib


if __name__ == "__main__":
    argv = sys.argv[1:]
    print(build(force="-f" in argv, out=argv[argv.index("--out") + 1] if "--out" in argv else None,
                defines=[a for a in argv if a.startswith("-D")]))
