"""The host side of libcamera_hip under AddressSanitizer and UndefinedBehaviorSanitizer (no GPU needed): the library is
rebuilt with its host code instrumented (device code as usual) and a small C++ driver walks the argument-validation
paths of every entry point, with tables at their limits.  Any report from a sanitizer fails the run."""
import concurrent.futures
import os
import shutil
import subprocess

import pytest

from paper_2508_02322_amd import build as libbuild

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OUT = os.path.join(ROOT, "_build", "sanitize")
SAN = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fno-omit-frame-pointer",
       "-Xarch_host", "-fno-sanitize-recover=undefined"]


def _run(cmd, **kw):
    res = subprocess.run(cmd, capture_output=True, text=True, **kw)
    assert res.returncode == 0, f"{' '.join(cmd)}\n{res.stdout[-3000:]}\n{res.stderr[-3000:]}"
    return res


def test_host_code_is_clean_under_asan_and_ubsan():
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not available")
    hipcc = libbuild.hipcc()
    os.makedirs(OUT, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(OUT, os.path.splitext(src)[0] + ".o")
        _run([hipcc, *libbuild.FLAGS, *SAN, "-c", os.path.join(libbuild.CSRC, src), "-o", obj])
        return obj

    with concurrent.futures.ThreadPoolExecutor(max_workers=8) as pool:
        objs = list(pool.map(compile_one, libbuild.SOURCES))
    lib = os.path.join(OUT, "libcamera_hip_san.so")
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-fsanitize=address", "-fsanitize=undefined", "-o", lib, *objs])
    exe = os.path.join(OUT, "abi_host_checks")
    # the driver is plain C++: built with the same compiler family, so that both halves share one sanitizer runtime
    clang = os.path.join(os.path.dirname(os.path.realpath(hipcc)), "..", "lib", "llvm", "bin", "clang++")
    if not os.path.exists(clang):
        clang = "/opt/rocm/lib/llvm/bin/clang++"
    _run([clang, "-O1", "-g", "-std=c++17", "-fsanitize=address", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
          os.path.join(ROOT, "tests", "native", "abi_host_checks.cpp"), "-o", exe, lib, f"-Wl,-rpath,{OUT}"])
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1:abort_on_error=0", UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    res = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=120)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    assert "all passed" in res.stdout
    assert "ERROR: AddressSanitizer" not in res.stderr and "runtime error" not in res.stderr


def test_launch_helpers_under_tsan(tmp_path):
    """Kernel attributes are set per device, from any host thread, and grids stay inside a launch's limits: the helpers of
    the launchers, host code only."""
    clang = "/opt/rocm/lib/llvm/bin/clang++"
    if not os.path.exists(clang):
        pytest.skip("clang++ not available")
    exe = str(tmp_path / "host_launch_checks")
    _run([clang, "-O1", "-g", "-std=c++17", "-pthread", "-fsanitize=thread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
          os.path.join(ROOT, "tests", "native", "host_launch_checks.cpp"), "-o", exe])
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-4000:]
    assert "all passed" in res.stdout and "WARNING: ThreadSanitizer" not in res.stderr
