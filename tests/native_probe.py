"""Compile a small host program against the library's internal headers and run it (CPU only)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1811_12378_amd")
LIB = os.path.join(PKG, "libhfci.so")
HIPCC = "/opt/rocm/bin/hipcc"
available = os.path.exists(LIB) and os.path.exists(HIPCC)


def run_native(source: str, tmp_path) -> str:
    """The standard output of `source` (C++, host code only) linked with the built library."""
    src, obj, exe = (str(tmp_path / n) for n in ("probe.cpp", "probe.o", "probe"))
    with open(src, "w") as f:
        f.write(source)
    for cmd in ([HIPCC, "-x", "c++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                 "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"), "-c", src, "-o", obj],
                [HIPCC, obj, "-o", exe, LIB, "-Wl,-rpath," + PKG]):
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
