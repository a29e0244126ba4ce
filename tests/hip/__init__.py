"""Device checks of pieces of the kernels: tests/hip/*.hip built into tests/hip/libchecks.so."""
import ctypes
import glob
import os
import subprocess

from paper_2406_06488_amd import build as hip_build

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "libchecks.so")


def build():
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hip_build.HIPCC] + hip_build.COMMON + hip_build.DEVICE + ["-shared", "-o", tmp] + \
        sorted(glob.glob(os.path.join(HERE, "*.hip")))
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + r.stderr)
    os.replace(tmp, LIB)
    return LIB


def load():
    return ctypes.CDLL(LIB if os.path.exists(LIB) else build())
