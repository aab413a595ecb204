"""Builds libgemm_mi355x.so from the HIP sources in csrc/ with hipcc for gfx950."""
import concurrent.futures
import glob
import os
import subprocess
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
OBJDIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libgemm_mi355x.so")
BINDING_SRC = os.path.join(CSRC, "binding.cpp")
BINDING = os.path.join(HERE, "_binding" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I" + INCLUDE, "-I" + CSRC,
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _stale(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _compile(src, force):
    obj = os.path.join(OBJDIR, os.path.basename(src)[:-4] + ".o")
    deps = [src] + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(INCLUDE, "*.h"))
    if force or _stale(obj, deps):
        subprocess.run([HIPCC] + FLAGS + ["-c", src, "-o", obj], check=True,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return obj


def build_binding(force=False):
    """Compile the Python extension that calls the library (host code only). Returns its path."""
    if force or _stale(BINDING, [BINDING_SRC]):
        tmp = BINDING + ".tmp%d" % os.getpid()
        subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
                        "-I" + sysconfig.get_paths()["include"], BINDING_SRC, "-o", tmp], check=True,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
        os.replace(tmp, BINDING)
    return BINDING


def build(force=False, jobs=None):
    """Compile every .hip file and link the shared library, and the Python extension. Returns the library's path.
    The extension is optional (calls go through ctypes without it): that it cannot be built is a warning."""
    os.makedirs(OBJDIR, exist_ok=True)
    srcs = sources()
    jobs = jobs or min(8, len(srcs), os.cpu_count() or 1)
    try:
        with concurrent.futures.ThreadPoolExecutor(jobs) as ex:
            objs = list(ex.map(lambda s: _compile(s, force), srcs))
    except subprocess.CalledProcessError as e:
        raise RuntimeError("hipcc failed:\n" + (e.stdout or b"").decode(errors="replace")) from e
    if force or _stale(LIB, objs):
        tmp = LIB + ".tmp%d" % os.getpid()
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs, check=True)
        os.replace(tmp, LIB)
    try:
        build_binding(force)
    except (OSError, subprocess.CalledProcessError) as e:
        warnings.warn("the Python extension was not built (%s)\n%s" % (e, (getattr(e, "stdout", None) or b"").decode(errors="replace")))
    return LIB


if __name__ == "__main__":
    print(build(force=True))
