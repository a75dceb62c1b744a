"""Builds the GPU code that only the tests run: ``_build/libtanh_sweep.so``."""
import os
import subprocess

from paper_2605_07083_amd import build as hipbuild

HERE = os.path.dirname(os.path.abspath(__file__))
TANH_SWEEP = os.path.join(os.path.dirname(HERE), "_build", "libtanh_sweep.so")


def build():
    os.makedirs(os.path.dirname(TANH_SWEEP), exist_ok=True)
    out = TANH_SWEEP + ".tmp"
    subprocess.check_call([hipbuild.hipcc()] + hipbuild.flags() +
                          ["-shared", "-o", out, os.path.join(HERE, "tanh_sweep.hip")])
    os.replace(out, TANH_SWEEP)
    return TANH_SWEEP
