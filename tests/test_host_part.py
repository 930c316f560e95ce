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


# (tables that read others, and the least scratch of a lattice)
MORE = HEAD + r"""
def solve(target, lat, scratch_bytes=None, deps=()):
    cost, arg, most = B.table_bytes(target, lat)
    scratch_bytes = most if scratch_bytes is None else scratch_bytes
    h, stats = C.c_void_p(), B.Stats()
    handles = (C.c_void_p * max(1, len(deps)))(*[d._h for d in deps])
    B._check(B.lib().mrl_solve(target._h, C.byref(B._lattice_desc(lat)), handles if deps else None, C.c_uint32(len(deps)), buffer(cost), buffer(arg),
                               buffer(scratch_bytes), C.c_size_t(scratch_bytes), None, C.byref(h), C.byref(stats)))
    return B.Table(h, target, lat, B.geometry(target, lat)[0], None, stats, deps)

def least_scratch(target, lat, deps=()):
    try:
        solve(target, lat, 256, deps=deps)
    except B.MorelloError as e:
        assert e.code == B.E_NOMEM
        return int(re.search(r"at least (\d+)", str(e)).group(1))
    assert False
"""

SCRATCH = MORE + r"""
# (configuration, largest size, table): what mrl_table_bytes asked for, and the least that a solve took
enough = {(1, 16, "M"): (5966080, 457216), (2, None, "M"): (3041477888, 29908736), (3, 8, "M"): (1563904, 88832),
          (3, None, "M"): (16899584, 307712), (4, 8, "M"): (24762112, 1164544), (4, None, "M"): (4322228480, 54018304),
          (5, 2, "M"): (823552, 85760), (5, 2, "E"): (219904, 35072), (5, 2, "F"): (12913920, 1114880), (6, 8, "P"): (6072576, 172800),
          (7, 2, "B"): (173770240, 1400832), (9, 8, "V"): (27818240, 1271040), (9, 4, "M"): (6203648, 303872),
          (10, 4, "G"): (254094080, 15173376), (11, 4, "A"): (459776, 44544), (11, 4, "R"): (129792, 24832), (11, 4, "S"): (459776, 44544),
          (12, 4, "M"): (24762112, 1164544)}
for (number, most, want), (asked, least) in enough.items():
    cfg = W.config(number, max_size=most)
    target, tabs = B.Target(cfg["target"]), {}
    for label, lat, deps in cfg["lattices"]:
        deps = [tabs[d] for d in deps]
        if label == want:
            assert B.table_bytes(target, lat)[2] <= asked, (number, most, label, B.table_bytes(target, lat)[2])
            assert least_scratch(target, lat, deps) <= least, (number, most, label, least_scratch(target, lat, deps))
            break
        tabs[label] = solve(target, lat, deps=deps)
print("done")
"""

FORMS = MORE + r"""
# every diagonal of a Matmul whose Moves are Move Specs, without layouts, has 128 or 129 entries; a chain's workgroup of 1024 lanes takes
# eight of them an entry
cfg = W.config(9, max_size=2)
(_, lat_v, _), (_, lat_m, _) = cfg["lattices"]
lat_m["layout_coord"] = [0] * 5
target = B.Target(cfg["target"])
moves = solve(target, lat_v)
for units, chained in ((128, True), (129, False)):
    hip.fake_units(units)
    for part in ("fill_chain", "fill_split"):
        hip.fake_launches_of(part.encode())
    tab = solve(target, lat_m, deps=[moves], scratch_bytes=64 << 20)
    chains, splits = (hip.fake_launches_of(part.encode()) for part in ("fill_chain", "fill_split"))
    assert (chains, splits) == ((1, 0) if chained else (0, 13)), (units, chains, splits)        # 4 dependency levels, 10 ranks
print("done")
"""

LIMIT = MORE + r"""
# diagonals around the most that one launch's threads can take: eight lanes per entry and eight entries per unit, or four and one
# (few memory levels, so that a shape has too few cells for its levels to be filled at once; the places in the list are 32 bits)
layouts, most, levels, diagonals = {"layouts": ([1, 1, 1, 0, 0], (1 << 26) - 4, 2, 4), "no-layouts": ([0] * 5, (1 << 30) - 64, 1, 1)}[sys.argv[3]]
cfg = W.config(6, max_size=1)
cfg["target"].update(n_levels=levels, microkernels=[])
for _, lat, _ in cfg["lattices"]:
    lat["layout_coord"] = layouts
target, (serial, parallel) = B.Target(cfg["target"]), [lat for _, lat, _ in cfg["lattices"]]
table = solve(target, serial)
room = buffer(1 << 20)                            # (nothing is launched: the list's places are never written)
for units, pieces in ((most, 1), (most + 1, 2), (most + 100, 2)):
    hip.fake_units(units)
    for part in (b"fill_split", b"fill_chain", b"fill_quad"):
        hip.fake_launches_of(part)
    h, stats = C.c_void_p(), B.Stats()
    B._check(B.lib().mrl_solve(target._h, C.byref(B._lattice_desc(parallel)), (C.c_void_p * 1)(table._h), C.c_uint32(1), buffer(1 << 20), buffer(1 << 20), room,
                               C.c_size_t(1 << 40), None, C.byref(h), C.byref(stats)))
    launches = sum(hip.fake_launches_of(part) for part in (b"fill_split", b"fill_chain", b"fill_quad"))       # (a chain: a rest of few entries)
    assert launches == diagonals * pieces, (units, pieces, launches)
    assert stats.n_admissible == units * diagonals << (3 if layouts[0] else 0)
print("done")
"""

LEVELS = MORE + r"""
# a Matmul of all sizes to 24 (13 levels, 10 ranks): its levels of shapes are filled at once from a number of level assignments on
cfg = W.config(4, max_size=1)
lat = cfg["lattices"][0][1]
name = sys.argv[3]
r = list(range(1, 25))
lat.update(sizes=[[1], r, r, r], layout_coord={"none": [0] * 5, "layouts": [1, 1, 1, 0, 0]}.get(name, [0] * 5))
if name == "few-levels":
    cfg["target"]["n_levels"] = 2
if name == "sparse":
    lat["sizes"] = [[1], list(range(1, 97)), list(range(1, 97)), list(range(1, 97))]
target = B.Target(cfg["target"])
levels = 19 if name == "sparse" else 13
diagonals = levels + (4 if name == "few-levels" else 10) - 1
# so many for each level, and a part of all places, the larger the more layouts there are
line = {"none": 190000 * 13 + 24 ** 3 * 64 * 16 // 100, "layouts": 150000 * 13 + 24 ** 3 * 64 * 50 // 100, "sparse": 190000 * 19 + 96 ** 3 * 64 * 16 // 100, "few-levels": 1 << 40}[name]
for units, at_once in (((line - 1) // diagonals, False), (-(-line // diagonals) if line < 1 << 32 else 1 << 22, line < 1 << 32)):
    hip.fake_units(units)
    for part in (b"fill_shapes", b"fill_split", b"fill_quad", b"fill_entry"):
        hip.fake_launches_of(part)
    h, stats = C.c_void_p(), B.Stats()
    units < 1 << 26 and B._check(B.lib().mrl_solve(target._h, C.byref(B._lattice_desc(lat)), None, C.c_uint32(0), buffer(1 << 20), buffer(1 << 20), buffer(1 << 28),
                               C.c_size_t(1 << 40), None, C.byref(h), C.byref(stats)))
    others = sum(hip.fake_launches_of(part) for part in (b"fill_split", b"fill_quad", b"fill_entry"))
    assert (hip.fake_launches_of(b"fill_shapes"), others) == ((levels, 0) if at_once else (0, diagonals if units < 1 << 26 else 0)), (units, at_once, others)
print("done")
"""

WINDOWS = MORE + r"""
# all sizes to 40, two memory levels, 8 level assignments a shape: half a million units in 19 diagonals, of which the least scratch holds a part at a time
hip.fake_blocks_of.restype = C.c_uint64
cfg = W.config(1)
cfg["lattices"][0][1]["sizes"][1:] = [list(range(1, 41))] * 3
target, lat = B.Target(cfg["target"]), cfg["lattices"][0][1]
least = least_scratch(target, lat)
hip.fake_units(28000)

def listed(scratch_bytes):
    for part in (b"list_units", b"fill_split"):
        hip.fake_launches_of(part)
    hip.fake_blocks_of(b"list_units")
    solve(target, lat, scratch_bytes)
    return hip.fake_launches_of(b"list_units"), hip.fake_blocks_of(b"list_units"), hip.fake_launches_of(b"fill_split")

once, blocks, pieces = listed(64 << 20)
assert (once, pieces) == (1, 19) and blocks > 500, (once, pieces, blocks)
windows, more, parts = listed(least)
assert windows > 3 and parts >= 19
assert more < windows * blocks / 2, (windows, blocks, more)          # a window's levels and ranks, not all of them again

# four memory levels, of which a shape has cells enough: in two parts, and by levels of shapes where there would be more parts than those are launches
cfg = W.config(2, max_size=40)
target, lat = B.Target(cfg["target"]), cfg["lattices"][0][1]
least = least_scratch(target, lat)
for scratch_bytes, want in ((64 << 20, (1, 0)), (least + 8 * 60000 * 25, (2, 0)), (least, (1, 16))):
    hip.fake_units(100000)
    for part in (b"list_units", b"fill_shapes"):
        hip.fake_launches_of(part)
    solve(target, lat, scratch_bytes)
    lists, levels = (hip.fake_launches_of(part) for part in (b"list_units", b"fill_shapes"))
    assert (lists, levels) == want, (scratch_bytes, lists, levels)
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


def test_scratch_that_sufficed_suffices(tmp_path):
    """A program may keep a buffer of exactly the size that mrl_table_bytes once asked for, or of the least that a solve
    once took, for every kind of lattice: neither has grown."""
    run_on_fake_hip(tmp_path, SCRATCH)


def test_chains_hold_diagonals_of_one_round(tmp_path):
    """A chain takes the diagonals that its workgroup does in one go, by the lanes that its kernel has per entry."""
    run_on_fake_hip(tmp_path, FORMS)


@pytest.mark.parametrize("case", ["layouts", "no-layouts"])
def test_diagonals_of_more_entries_than_a_launch_has_threads_for(case, tmp_path):
    """A launch has fewer than 2^32 threads; a diagonal of the largest tables asks for more, and goes in pieces."""
    run_on_fake_hip(tmp_path, LIMIT, case)


@pytest.mark.parametrize("case", ["none", "layouts", "sparse", "few-levels"])
def test_tables_of_which_much_fits_are_filled_by_levels_of_shapes(case, tmp_path):
    """From as many level assignments as pay for a launch a level and for the places of those that are not there, and if a shape has cells enough."""
    run_on_fake_hip(tmp_path, LEVELS, case)


def test_a_window_of_the_work_list_is_made_from_its_own_levels(tmp_path):
    """Where the scratch holds a part of the list at a time, a part is made from the shapes that have units in it."""
    run_on_fake_hip(tmp_path, WINDOWS)
