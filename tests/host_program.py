"""Builds a host check of the device code's headers (tests/native/) and runs it."""
import os
import subprocess

from paper_1510_06897_amd import build

NATIVE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native")


def run(name, tmp_path, *args):
    """Compiles tests/native/<name> (a .hip file as the library is, a .cpp file against the stand-in
    runtime of tests/native/stub) and returns the finished process; its output is printed."""
    prog, src = str(tmp_path / os.path.splitext(name)[0]), os.path.join(NATIVE, name)
    if name.endswith(".hip"):
        flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared", "-O3")]
        cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "-O1", "-Xarch_host", "-mfma"]
    else:
        cmd = ["g++", "-std=c++17", "-O1", "-g", "-Wall", "-pthread", "-I" + os.path.join(NATIVE, "stub")]
    made = subprocess.run([*cmd, "-o", prog, src], capture_output=True, text=True)
    assert made.returncode == 0, made.stderr
    done = subprocess.run([prog, *args], capture_output=True, text=True, timeout=300)
    print(done.stdout)
    return done
