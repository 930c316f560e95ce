"""Questions to a table while another device is current (no GPU needed): the library's host part runs on a
runtime of two devices that launches nothing (fake_hip.c) but keeps HIP's rules of streams, events and devices."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2505_01637_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))

ASK = r"""
import ctypes as C, sys
sys.path.insert(0, sys.argv[2])
sys.modules["torch"] = None                       # (its own runtime would be loaded first)
hip = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
import numpy as np
from paper_2505_01637_amd import binding as B, workloads as W

def buffer(n):
    p = C.c_void_p()
    assert hip.hipMalloc(C.byref(p), C.c_size_t(n)) == 0
    return p

own_stream = sys.argv[3] == "own"
cfg = W.config(4, max_size=4)
lat = cfg["lattices"][0][1]
assert hip.hipSetDevice(1) == 0
stream = C.c_void_p()
if own_stream:
    assert hip.hipStreamCreateWithFlags(C.byref(stream), 1) == 0
target = B.Target(cfg["target"])
sizes = B.table_bytes(target, lat)
h, stats = C.c_void_p(), B.Stats()
B._check(B.lib().mrl_solve(target._h, C.byref(B._lattice_desc(lat)), None, C.c_uint32(0), *(buffer(n) for n in sizes[:3]),
                           C.c_size_t(sizes[2]), stream, C.byref(h), C.byref(stats)))
ext, n_specs = B.geometry(target, lat)
tab = B.Table(h, target, lat, ext, None, stats)
assert hip.fake_launches(1) > 0
assert hip.hipSetDevice(0) == 0
for compressed in (False, True):
    for n in (1, 32768, 32769, 100003):
        tab.query(np.zeros((n, len(ext)), dtype=np.uint32), compressed=compressed)
        now = C.c_int(-1)
        hip.hipGetDevice(C.byref(now))
        assert now.value == 0, "the caller's device is current again"
before = hip.fake_launches(1)
try:
    tab.schedule([0] * len(ext))                  # (no kernel runs: the chain that it reads is empty)
except B.MorelloError as e:
    assert e.code == B.E_HIP
assert hip.fake_launches(1) == before + 1
assert hip.fake_launches(0) == 0, "every launch goes to the table's device"
print("asked")
"""


@pytest.mark.parametrize("stream", ["own", "null"])
def test_questions_with_another_device_current(stream, tmp_path):
    """Of one launch and in stretches, in the table, in its boxes and for a program, of a table that was solved on a
    stream of its device and on its null stream: answered, on the table's device, which is not left current."""
    gcc = shutil.which("gcc")
    if not gcc or not os.path.exists(B.LIB_PATH):
        pytest.skip("needs gcc and the built library")
    versions = tmp_path / "versions"
    versions.write_text("hip_4.2 { global: *; };\n")
    fake = tmp_path / "libfakehip.so"
    subprocess.run([gcc, "-O1", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7", f"-Wl,--version-script={versions}",
                    os.path.join(HERE, "fake_hip.c"), "-o", str(fake)], check=True)
    run = subprocess.run([sys.executable, "-c", ASK, str(fake), os.path.dirname(HERE), stream], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "asked" in run.stdout, run.stdout + run.stderr
