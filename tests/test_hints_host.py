"""The pair list's hint kernel on the CPU (tests/wave: a wavefront of 64 fibers), and two
functions of the pair kernels.

A group's pages go into a table of 512 places; a group that names more than 384 pages gets
no hints.  The kernel counts the pages once per chunk of 256 entries, each of which can
name another page, so that a chunk may meet a table without a free place: it has to end
all the same, with the entries untouched and no header.  Where there are hints, each entry's
number has to lead back to the entry."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIMIT = 100_000  # operations across lanes of one wavefront: a table's worth of probes 30 times over


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    so = str(tmp_path_factory.mktemp("wave") / "libhints.so")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-w", f"-I{HERE}/wave",
                        f"-I{ROOT}/paper_1604_03290_amd/csrc", f"-I{ROOT}/include",
                        f"{HERE}/wave/hints.cpp", "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lib = C.CDLL(so)
    lib.hints_run.argtypes = [C.c_int64] + [C.c_void_p] * 3 + [C.c_long]
    return lib


def limits(lib):
    return list((C.c_int32 * 5).in_dll(lib, "hints_limits"))


def entries_of(new, seed, far):
    """Entries (steps, 64) of a group whose chunk c of four steps names new[c] pages that no
    chunk before it names, and otherwise pages already named."""
    rng = np.random.default_rng(seed)
    total = sum(new)
    pages = rng.choice(1 << 27, total, replace=False) if far else np.arange(total) + 7
    rows, known = [], 0
    for k in new:
        known += k
        fresh = np.arange(known - k, known)
        which = np.concatenate([fresh, rng.integers(0, known, 256 - k)])
        rows.append(16 * pages[rng.permutation(which)] + rng.integers(0, 16, 256))
    return np.concatenate(rows).reshape(-1, 64).astype(np.int32)


def run(lib, rows, counts, room):
    """(returned, entries after, words after) for one group with the given rows and counts."""
    steps = rows.shape[0]
    slot = np.full(64 * room + 1, 0x5a5a5a5a, dtype=np.int32)
    at = 1 if slot.ctypes.data & 7 else 0  # (the array is 8-byte aligned)
    s = slot[at:at + 64 * room]
    s[:64 * steps] = rows.ravel()
    start = np.array([0, 64 * room], dtype=np.int64)
    cnt = np.asarray(counts, dtype=np.int32)
    rc = lib.hints_run(64, cnt.ctypes.data, start.ctypes.data, s.ctypes.data, LIMIT)
    return rc, s[:64 * steps].reshape(steps, 64), s


def check(lib, rows, counts, room):
    places, max_pages, max_locals, header, magic = limits(lib)
    steps = rows.shape[0]
    rc, after, s = run(lib, rows, counts, room)
    assert rc == 0, "the wavefront does not end"
    assert np.array_equal(after, rows)
    named = np.concatenate([rows[:c, lane] for lane, c in enumerate(counts)])
    slots, pages = np.unique(named), np.unique(named >> 4)
    head = s[-header:]
    uni_words = 64 * (room // 8)
    if pages.size > max_pages or slots.size > min(max_locals, uni_words):
        assert head[0] == 0
        return False
    assert list(head[:3]) == [magic, slots.size, steps]
    uni = s[64 * room - header - uni_words:64 * room - header]
    assert np.array_equal(np.sort(uni[:slots.size]), slots)
    top = 64 * room - header - uni_words
    local = np.zeros((steps, 64), dtype=np.int64)
    for c in range(steps // 4):
        four = s[top - 128 * (c + 1):top - 128 * c].view(np.uint16).reshape(64, 4)
        local[4 * c:4 * c + 4] = four.T
    valid = np.arange(steps)[:, None] < np.asarray(counts)[None, :]
    assert np.array_equal(uni[local[valid]], rows[valid])
    for r in range((steps + 31) // 32):
        word = int(np.uint32(head[64 + r]))
        assert word & 0xffff == local[32 * r:][valid[32 * r:]].min()
        assert word >> 16 == local[:32 * r + 32][valid[:32 * r + 32]].max() + 1
    return True


@pytest.mark.parametrize("far", [False, True])
@pytest.mark.parametrize("new,hints", [
    ([255], True), ([256], True), ([256, 1], True), ([256, 128], True), ([128, 256], True),
    ([256, 129], False),               # one page too many
    ([256, 256], False),               # the table exactly full
    ([256, 128, 128], False),          # and met so by the last chunk
    ([256, 128, 129], False),          # one page without a place
    ([184, 172, 173], False), ([76, 256, 256], False),
    ([128, 256, 256], False),          # as many as a chunk can bring
    ([256, 128, 0, 256, 256], False),  # later chunks too
])
def test_pages(lib, new, hints, far):
    rows = entries_of(new, sum(new), far)
    assert check(lib, rows, [rows.shape[0]] * 64, 8 * rows.shape[0]) == hints


def test_ragged_counts_and_rounds(lib):
    """Lists of unequal lengths, several rounds of 32 steps."""
    rng = np.random.default_rng(3)
    rows = entries_of([40] + [5] * 24, 9, False)
    counts = rng.integers(0, rows.shape[0] + 1, 64)
    counts[17] = rows.shape[0]
    assert check(lib, rows, counts, 2 * rows.shape[0])


def test_too_many_locals(lib):
    """More slots than may be numbered, in few enough pages."""
    max_locals = limits(lib)[2]
    for extra in (0, 1):
        slots = np.arange(max_locals + extra)
        rows = np.resize(slots, (36, 64)).astype(np.int32)
        assert check(lib, rows, [36] * 64, 400) == (extra == 0)


@pytest.mark.parametrize("width", [576, 640, 704])
def test_places_of_a_window(lib, width):
    """Every number that is given has its place mod the window, any other a place of it."""
    max_locals = limits(lib)[2]
    assert [lib.window_place(width, l) for l in range(max_locals + 1)] == [l % width for l in range(max_locals + 1)]
    assert all(0 <= lib.window_place(width, l) < width for l in range(1 << 16))


@pytest.mark.parametrize("run", [64, 24, 8, 0, -1])
def test_every_workgroup_is_placed_once(lib, run):
    """The order in which workgroups go to the XCDs, at and beside whole rounds of runs."""
    lib.placed.restype = C.c_int64
    for n in (1, 7, 8, 9, 63, 64, 65, 191, 192, 193, 511, 512, 513, 1024, 1562, 4095, 4096, 4097):
        assert sorted(lib.placed(n, i, run) for i in range(n)) == list(range(n))
