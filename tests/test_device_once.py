"""The bookkeeping of settings that are made once per device (csrc/device_once.h), compiled for the CPU."""
import ctypes
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_17307_amd", "csrc")
WRAP = """
#include "device_once.h"
static rs::DeviceOnce once;
extern "C" int done(int device) { return once.done(device); }
extern "C" void mark(int device) { once.mark(device); }
"""


def test_a_setting_of_one_device_does_not_count_for_another(tmp_path):
    src, so = tmp_path / "wrap.cpp", tmp_path / "libdevice_once.so"
    src.write_text(WRAP)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    assert not any(lib.done(d) for d in (-1, 0, 1, 7, 63, 64, 1000))
    lib.mark(0)
    lib.mark(63)
    assert lib.done(0) and lib.done(63) and not lib.done(1) and not lib.done(62)
    for d in (-1, 64, 1000):                              # not remembered: made again each time
        lib.mark(d)
        assert not lib.done(d)
    assert lib.done(0) and not lib.done(1)
