"""Builds a host check of the device code's headers (tests/native/) and runs it."""
import os
import subprocess

from paper_1510_06897_amd import build

NATIVE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native")


def run(name, tmp_path, *flags):
    """Compiles tests/native/<name> and returns the finished process (its output is printed)."""
    prog = str(tmp_path / os.path.splitext(name)[0])
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    base = [f for f in build.FLAGS if f not in ("-fPIC", "-shared", "-O3")]
    made = subprocess.run([hipcc, *base, "-O1", *flags, "-o", prog, os.path.join(NATIVE, name)],
                          capture_output=True, text=True)
    assert made.returncode == 0, made.stderr
    done = subprocess.run([prog], capture_output=True, text=True, timeout=300)
    print(done.stdout)
    return done
