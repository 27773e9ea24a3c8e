"""Numbers that waves claim from one counter (csrc/wave_claim.h), compiled for the CPU with two waves of 64 lanes whose atomic
operations come one by one, in any order: each number goes to one wave, whose lanes all get it, and none is left out."""
import ctypes
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WAVES, TIMES = 2, 300


def test_each_number_once(tmp_path):
    out = str(tmp_path / "claims.so")
    subprocess.check_call(["g++", "-O1", "-std=c++20", "-shared", "-fPIC", "-o", out,
                           "-I", os.path.join(ROOT, "paper_2507_11941_amd", "csrc"),
                           os.path.join(ROOT, "tests", "wave_claim_driver.cpp")])
    taken = np.zeros((WAVES, 64, TIMES), np.uint32)
    lib = ctypes.CDLL(out)
    lib.claims.restype = ctypes.c_uint32
    counter = lib.claims(WAVES, TIMES, ctypes.c_void_p(taken.ctypes.data))
    assert (taken == taken[:, :1]).all()
    assert sorted(taken[:, 0].ravel()) == list(range(WAVES * TIMES)) and counter == WAVES * TIMES
