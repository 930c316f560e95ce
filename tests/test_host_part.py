"""The library's host part on the CPU (no GPU needed): it runs on a runtime of two devices that launches nothing
(fake_hip.c) but keeps HIP's rules of streams, events and devices and counts what is launched."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2505_01637_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))

HEAD = r"""
import ctypes as C, re, sys
sys.path.insert(0, sys.argv[2])
sys.modules["torch"] = None                       # (its own runtime would be loaded first)
hip = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
import numpy as np
from paper_2505_01637_amd import binding as B, workloads as W

def buffer(n):
    p = C.c_void_p()
    assert hip.hipMalloc(C.byref(p), C.c_size_t(n)) == 0
    return p

def solve(target, lat, scratch_bytes=None, stream=None):
    cost, arg, most = B.table_bytes(target, lat)
    scratch_bytes = most if scratch_bytes is None else scratch_bytes
    h, stats = C.c_void_p(), B.Stats()
    B._check(B.lib().mrl_solve(target._h, C.byref(B._lattice_desc(lat)), None, C.c_uint32(0), buffer(cost), buffer(arg), buffer(scratch_bytes),
                               C.c_size_t(scratch_bytes), stream, C.byref(h), C.byref(stats)))
    return B.Table(h, target, lat, B.geometry(target, lat)[0], None, stats)
"""

ASK = HEAD + r"""
own_stream = sys.argv[3] == "own"
cfg = W.config(4, max_size=4)
lat = cfg["lattices"][0][1]
assert hip.hipSetDevice(1) == 0
stream = C.c_void_p()
if own_stream:
    assert hip.hipStreamCreateWithFlags(C.byref(stream), 1) == 0
tab = solve(B.Target(cfg["target"]), lat, stream=stream)
ext = tab.extents
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
print("done")
"""


ROWS = HEAD + r"""
# 64 sizes along n and along m (k), eight words a shape: 512 planes of one row, 16 planes of up to 64
r = list(range(1, 65))
sizes, many, few = {"one-row": ([[1], r, [1], r], 512, 512), "rows": ([[1], [1, 2], r, r], 1024, 16)}[sys.argv[3]]
cfg = W.config(4, max_size=4)
lat = dict(cfg["lattices"][0][1], sizes=sizes)
target = B.Target(cfg["target"])

def launched(scratch_bytes=None):
    for part in ("row_total", "row_", "head_flags"):
        hip.fake_launches_of(part.encode())
    solve(target, lat, scratch_bytes)
    return tuple(hip.fake_launches_of(part.encode()) for part in ("row_total", "row_", "head_flags"))

total, rows, boxes = launched()
assert total == 0 and rows > 5 and boxes == 0, "plenty of scratch: by words, nothing asked before"
try:
    solve(target, lat, 256)
    assert False
except B.MorelloError as e:
    assert e.code == B.E_NOMEM
    least = int(re.search(r"at least (\d+)", str(e)).group(1))
hip.fake_row_total(many)
total, rows, boxes = launched(least + 4096)
assert rows == 0 and boxes > 0 and total == (1 if many > few else 0), "the words cannot fit: no kernel of that merge"
if many > few:
    hip.fake_row_total(few)
    total, rows, boxes = launched(least + 4096)
    assert total == 1 and rows > 5 and boxes == 0, "few of the rows are kept: their words fit"
print("done")
"""


def run_on_fake_hip(tmp_path, program, *args):
    gcc = shutil.which("gcc")
    if not gcc or not os.path.exists(B.LIB_PATH):
        pytest.skip("needs gcc and the built library")
    versions = tmp_path / "versions"
    versions.write_text("hip_4.2 { global: *; };\n")
    fake = tmp_path / "libfakehip.so"
    subprocess.run([gcc, "-O1", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7", f"-Wl,--version-script={versions}",
                    os.path.join(HERE, "fake_hip.c"), "-o", str(fake)], check=True)
    run = subprocess.run([sys.executable, "-c", program, str(fake), os.path.dirname(HERE), *args], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "done" in run.stdout, run.stdout + run.stderr


@pytest.mark.parametrize("stream", ["own", "null"])
def test_questions_with_another_device_current(stream, tmp_path):
    """Of one launch and in stretches, in the table, in its boxes and for a program, of a table that was solved on a
    stream of its device and on its null stream: answered, on the table's device, which is not left current."""
    run_on_fake_hip(tmp_path, ASK, stream)


@pytest.mark.parametrize("case", ["one-row", "rows"])
def test_no_merge_by_words_that_cannot_fit(case, tmp_path):
    """Scratch that holds the boxes and not the words: nothing of the merge by words is launched, where the sizes tell
    (one row per plane is kept at least) and where the number of rows, which is asked for then, does."""
    run_on_fake_hip(tmp_path, ROWS, case)
