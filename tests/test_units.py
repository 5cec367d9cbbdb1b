"""Host-side checks of how the waves divide an image (no GPU needed).

3D: a strip is 6 rows; its slots are its position columns and one more.  The slots of
the strips that lie whole in the image are numbered through and cut into wave tasks
of 2 x 63; the other strips are cut each for itself.  2D: blocks of `depth` rows in
place of strips.  The numbers of strips and tasks come from the library's own host
code (``ecc_internal.h``, compiled here); where a lane of a task stands is written
out below as the kernels compute it.  Every strip (block) and slot must belong to
one lane, whole tasks must touch rows inside the image only, byte offsets must fit 32
bits, and a batch's segment must not cover more voxels than its int32 counters hold.
"""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

from paper_2203_09087_amd import ecc

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2203_09087_amd", "csrc")
UNIT, ROWS = 63, 6          # owned lanes of a half task; rows of a strip
MAX_ROW_BYTES = 1 << 27     # longest row that is accepted
FRESH = 1 << 30             # row offset in a 2D block past which the loads start anew

SHIM = r"""
#include <string.h>
#include "ecc_internal.h"
static void put(const ecc::Units& u, int64_t* o)
{
    o[0] = u.slots; o[1] = u.sa; o[2] = u.sb; o[3] = u.pairs_full; o[4] = u.pairs_edge; o[5] = u.tasks;
}
extern "C" void units3(int64_t n0, int64_t n1, int64_t n2, int cons, int64_t* o)
{
    put(ecc::units_3d(ecc::Geom{n0, n1, n2}, cons), o);
}
extern "C" void units2(int64_t n1, int64_t n2, int cons, int64_t depth, int64_t* o)
{
    put(ecc::units_2d(ecc::Geom{1, n1, n2}, cons, depth), o);
}
extern "C" void work(int ndim, int64_t n0, int64_t n1, int64_t n2, int cons, int d3, int d2, int64_t planes, int64_t* o)
{
    ecc::BatchImage im;
    memset((void*)&im, 0, sizeof im);
    im.ndim = ndim;
    im.g = ecc::Geom{n0, n1, n2};
    const ecc::BatchWork w = ecc::batch_work(im, cons, d3, d2, planes);
    o[0] = w.bricks; o[1] = w.brick_voxels; o[2] = w.steps; o[3] = im.depth;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not os.path.exists(ecc.LIB_PATH):
        pytest.skip("libecc_hip.so not built")
    ecc.load_library()   # torch's HIP runtime first, as in a program
    d = tmp_path_factory.mktemp("units")
    src, so = str(d / "units.cpp"), str(d / "units.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", CSRC, src, ecc.LIB_PATH, "-o", so], check=True)
    shim = ctypes.CDLL(so)
    for name, nargs in (("units3", 3), ("units2", 2)):
        getattr(shim, name).argtypes = [ctypes.c_int64] * nargs + [ctypes.c_int] + \
            ([ctypes.c_int64] if name == "units2" else []) + [ctypes.POINTER(ctypes.c_int64)]
    shim.work.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3 + [ctypes.c_int] * 3 + [ctypes.c_int64,
                                                                                     ctypes.POINTER(ctypes.c_int64)]
    return shim


def call(fn, *args):
    out = (ctypes.c_int64 * 6)()
    fn(*args, out)
    return list(out)


def passed(c, slots):
    """Strips passed by place c, as the kernels divide (16-bit reciprocal)."""
    return (c * (65536 // slots + 1)) >> 16 if slots < 128 else (1 if c >= slots else 0)


def owned(U, strips):
    """(strip, slot, whole) of every owned lane of every task."""
    slots, sa, sb, full, edge, tasks = U
    for task in range(tasks):
        if task < full:
            at = task * 2 * UNIT
            first, c0, left = sa + at // slots, at % slots, (sb - sa) * slots - at
        else:
            i, k = divmod(task - full, edge)
            c0 = k * 2 * UNIT
            first, left = (i if i < sa else sb + i - sa), slots - c0
        for half in (0, UNIT):
            for lane in range(UNIT):
                if half + lane < left:
                    c = c0 + half + lane
                    q = passed(c, slots)
                    assert q == c // slots
                    assert first + q < strips
                    yield first + q, c - q * slots, task < full


def shapes(seed, count):
    rng = np.random.default_rng(seed)
    yield from [(1, 1), (6, 62), (7, 63), (7, 127), (8, 125), (13, 126), (14, 1), (31, 2), (40, 61), (12, 300)]
    for _ in range(count):
        yield int(rng.integers(1, 60)), int(rng.integers(1, 300))


@pytest.mark.parametrize("top", [0, 1])
def test_strips_are_covered_once(lib, top):
    for n1, n2 in shapes(3 + top, 60):
        U = call(lib.units3, 4, n1, n2, top)
        strips = -(-(n1 + top) // ROWS)
        got = list(owned(U, strips))
        assert sorted((s, c) for s, c, _ in got) == [(s, c) for s in range(strips) for c in range(n2 + top + 1)], (n1, n2)
        for s, _, whole in got:
            if whole:
                assert -top + ROWS * s >= 0 and -top + ROWS * s + ROWS < n1, (n1, n2, s)


@pytest.mark.parametrize("top", [0, 1])
@pytest.mark.parametrize("depth", [16, 48])
def test_blocks_are_covered_once(lib, top, depth):
    for n1, n2 in shapes(5 + top, 60):
        U = call(lib.units2, n1, n2, top, depth)
        blocks = -(-n1 // depth)
        got = list(owned(U, blocks))
        assert sorted((b, c) for b, c, _ in got) == [(b, c) for b in range(blocks) for c in range(n2 + top + 1)], (n1, n2)
        for b, _, whole in got:
            assert not whole or depth * (b + 1) <= n1


def test_reciprocal_is_exact():
    for slots in range(2, 300):
        for c in range(slots + 2 * 64):
            if slots >= 128 or c < 256:
                assert passed(c, slots) == c // slots


@pytest.mark.parametrize("top", [0, 1])
def test_byte_offsets_fit_32_bits(lib, top):
    """Rows from 1 byte to 2^27: a lane's column, the strips (blocks) that it is past
    the wave's first one, and the rows of the march from one 64-bit address."""
    for e in range(28):
        for n2 in {1 << e, max(1, (1 << e) - 1), max(1, (1 << e) * 3 // 4)}:
            for size in (1, 2, 4):
                if n2 * size > MAX_ROW_BYTES:
                    continue
                slots = n2 + top + 1
                q = passed(min(slots - 1 + 2 * UNIT, 255) if slots < 128 else slots - 1 + 2 * UNIT, slots)
                assert (n2 + q * ROWS * n2 + ROWS * n2) * size < 2 ** 32
                for depth in (16, 112, 512, 4096):
                    U = call(lib.units2, 4 * depth + 3, n2, top, depth)
                    if U[2] > 0:     # numbered through: offsets reach over all the blocks of a task
                        assert (n2 + q * depth * n2 + (depth + 1) * n2) * size < 2 ** 32, (n2, size, depth)
                    else:            # every block for itself: 8 rows past FRESH at most
                        assert FRESH + (n2 + 8 * n2) * size < 2 ** 32


@pytest.mark.parametrize("top", [0, 1])
@pytest.mark.parametrize("ndim", [2, 3])
def test_a_position_changes_a_prefix_sum_by_two_at_most(ndim, top):
    """The cells at a position (a single or a pair of neighbours per axis) that lie in a
    sublevel set, with their signs: over all 2^(2^ndim) sets of its voxels."""
    sums = set()
    for inside in range(1 << (1 << ndim)):
        total = 0
        for pairs in itertools.product((0, 1), repeat=ndim):
            voxels = itertools.product(*[(0, 1) if p else (top,) for p in pairs])
            got = [inside >> sum(b << k for k, b in enumerate(v)) & 1 for v in voxels]
            if any(got) if top else all(got):
                total += (-1) ** (ndim - sum(pairs) if top else sum(pairs))
        sums.add(total)
    assert max(abs(v) for v in sums) <= 2, sums


@pytest.mark.parametrize("top", [0, 1])
def test_rows_fit_int32(lib, top):
    """A workgroup's row holds prefix sums of its histogram: at most 2 in absolute value
    per position (above).  A batch's segment takes at most 2^27 voxels counted in bricks
    and runs the same share of the volume's steps; a single image has at least one
    workgroup per 2^27 voxels, each taking an equal number of wave tasks.  The most
    positions that a step (a plane of a task, or 16 rows of it) holds bound the row."""
    segment = single = flat = 0.0
    big = [(1 << 14, 127), (7, 1 << 20), (1000, 1000), (255, 129)]
    ragged = [(n1, n2) for n1 in (1, 2, 6, 7, 8, 13, 14) for n2 in range(1, 400)]
    for n1, n2 in list(shapes(7 + top, 200)) + ragged + big:
        _, sa, sb, _, _, tasks = call(lib.units3, 4, n1, n2, top)
        step = max(min(2 * UNIT, n2 + top) * min(ROWS, n1 + top), min(2 * UNIT, (sb - sa) * (n2 + top)) * ROWS)
        for n0, d3, planes in ((17, 8, 16), (100000, 4, 16), (100000, 8, 86), (100000, 16, 10 ** 9)):
            bricks, brick_voxels, steps, _, _, _ = call(lib.work, 3, n0, n1, n2, top, d3, 128, planes)
            segment = max(segment, step * steps / (bricks * brick_voxels))
        if n1 * n2 >= 16:   # more than 2^27 voxels for each of 256 CUs, in at most 2^31 planes
            single = max(single, tasks * step / (n1 * n2))
        for d2 in (32, 64, 128):
            for rows in (n1, 16 * n1, 16 * n1 + 1, 10 ** 6):
                bricks, brick_voxels, steps, _, _, _ = call(lib.work, 2, 1, rows, n2, top, 8, d2, 16)
                flat = max(flat, min(2 * UNIT * 16, rows * (n2 + top)) * steps / (bricks * brick_voxels))
    # and the part of a brick or step that rounding adds
    assert 2 * (max(segment, single, flat) * 2 ** 27 + 16 * 2 * UNIT * ROWS * 4096) < 2 ** 31, (segment, single, flat)
