"""GPU parity of the packed marching kernels at the sizes where their layout can
go wrong, against the oracle, bit for bit.

A wave takes two units of 63 position columns; the columns of consecutive strips
(6 rows each) are numbered through, so a unit may end inside a row and go on in
the next strip.  The sizes put the end of a row, of a strip and of a unit on and
next to each other, with images smaller than a unit or a strip, every dtype,
values that tie, and histograms of one bin, one window and several windows.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def say(*args):
    print(*args, flush=True, file=sys.stderr)


def to_dev(a):
    if a.dtype == np.uint16:
        return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def draw_image(rng, shape, kind):
    if kind == "u8":
        return rng.integers(0, 7, size=shape).astype(np.uint8), 7, (0, 6)
    if kind == "u16":
        return rng.integers(0, 65536, size=shape).astype(np.uint16), 4096, "auto"
    if kind == "u16wide":   # more bins than one window
        return rng.integers(0, 65536, size=shape).astype(np.uint16), 20000, (0, 65535)
    img = rng.standard_normal(shape).astype(np.float32)
    img[rng.random(shape) < 0.02] = np.nan
    img[rng.random(shape) < 0.02] = np.inf
    img[rng.random(shape) < 0.02] = -np.inf
    return img, (1 if kind == "f32one" else 333), (-1.5, 1.25)


SHAPES_3D = [(1, 1, 1), (2, 6, 62), (3, 7, 63), (2, 5, 64), (4, 12, 125), (3, 13, 126), (2, 14, 127), (5, 31, 3),
             (3, 40, 1), (2, 25, 41), (9, 8, 189)]


@pytest.mark.parametrize("cons", ["vertex", "top"])
@pytest.mark.parametrize("kind", ["u8", "u16", "u16wide", "f32", "f32one"])
def test_strips_and_units_3d(oracle_mod, cons, kind):
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(4100)
    ctx = ecc.Context(0, cons)
    try:
        for shape in SHAPES_3D:
            img, nbins, r = draw_image(rng, shape, kind)
            say(f"case: {cons} {kind} {shape} nbins={nbins}")
            dev = to_dev(img)
            want = oracle_mod.ecc(img, nbins, cons, value_range=r, threads=8)
            for depth in (0, 1, 2, 3):
                ctx.set_launch_shape(dev, nbins, depth=depth)
                got = ctx.compute(dev, nbins, value_range=r)
                torch.cuda.synchronize()
                assert np.array_equal(got.cpu().numpy(), want), (cons, kind, shape, depth)
    finally:
        ctx.close()


SHAPES_2D = [(1, 1), (1, 200), (16, 62), (15, 63), (17, 64), (32, 125), (33, 126), (48, 127), (16, 2), (200, 1),
             (160, 3), (97, 41), (256, 189)]


@pytest.mark.parametrize("cons", ["vertex", "top"])
@pytest.mark.parametrize("kind", ["u8", "u16", "u16wide", "f32", "f32one"])
def test_blocks_and_units_2d(oracle_mod, cons, kind):
    """2D: blocks of `depth` rows in place of strips; heights of whole blocks, one
    row more and one row less."""
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(4200)
    ctx = ecc.Context(0, cons)
    try:
        for shape in SHAPES_2D:
            img, nbins, r = draw_image(rng, shape, kind)
            say(f"case: {cons} {kind} {shape} nbins={nbins}")
            dev = to_dev(img)
            want = oracle_mod.ecc(img, nbins, cons, value_range=r, threads=8)
            for depth in (0, 16, 32, 48):
                ctx.set_launch_shape(dev, nbins, depth=depth)
                got = ctx.compute(dev, nbins, value_range=r)
                torch.cuda.synchronize()
                assert np.array_equal(got.cpu().numpy(), want), (cons, kind, shape, depth)
    finally:
        ctx.close()


@pytest.mark.parametrize("cons", ["vertex", "top"])
def test_batch_shares_of_wave_tasks(oracle_mod, cons):
    """A batch's segments are shares of each volume's wave tasks: images of one
    task and less than one task per workgroup, uneven 2D, 3D and 4D ones together,
    one window and several, unplanned and at plan shapes with 1 to 4 workgroups
    per CU."""
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(4300)
    shapes = SHAPES_3D + SHAPES_2D + [(3, 4, 7, 64), (2, 9, 13, 130), (1, 2, 5, 3)]
    ctx = ecc.Context(0, cons)
    try:
        for kind in ("u8", "u16wide", "f32"):
            drawn = [draw_image(rng, s, kind) for s in shapes]
            nbins, r = drawn[0][1], drawn[0][2]
            hosts = [d[0] for d in drawn]
            devs = [to_dev(h) for h in hosts]
            say(f"case: batch {cons} {kind} {len(hosts)} images nbins={nbins}")
            want = [oracle_mod.ecc(h, nbins, cons, value_range=r, threads=8) for h in hosts]
            got = ctx.compute_batch(devs, nbins, value_ranges=[r] * len(devs))
            torch.cuda.synchronize()
            for h, g, w in zip(hosts, got, want):
                assert np.array_equal(g.cpu().numpy(), w), (cons, kind, h.shape)
            plan = ctx.plan_batch(devs, nbins, [r] * len(devs))
            plan.autotune(1)
            for o in plan.outs:
                o.fill_(-1)
            plan.launch()
            torch.cuda.synchronize()
            for h, g, w in zip(hosts, plan.outs, want):
                assert np.array_equal(g.cpu().numpy(), w), (cons, kind, h.shape, "plan")
            plan.close()
    finally:
        ctx.close()


@pytest.mark.parametrize("nbins", [4097, 8192, 8193, 16384, 16385, 40000, 65535])
def test_wide_histograms(oracle_mod, nbins):
    """Histograms wider than 4096 bins: one pass up to 16384 bins (two copies of the
    counters up to 8192, then one), passes of 16384 above; 2D, 3D and 4D, small and
    large enough for several workgroups, also without allocation, with forced copies
    and windows, and in a batch (passes of 4096)."""
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(4400)
    for cons in ("vertex", "top"):
        ctx = ecc.Context(0, cons)
        try:
            for shape in ((3, 2), (130, 257), (9, 30, 141), (2, 3, 14, 65)):
                for dtype in (np.uint16, np.float32):
                    img = (rng.integers(0, 65536, size=shape).astype(np.uint16) if dtype == np.uint16
                           else rng.standard_normal(shape).astype(np.float32))
                    say(f"case: wide {cons} {nbins} {shape} {np.dtype(dtype).name}")
                    dev = to_dev(img)
                    want = oracle_mod.ecc(img, nbins, cons, value_range="auto", threads=8)
                    got = [ctx.compute(dev, nbins, value_range="auto")]
                    out = torch.full((nbins,), -5, dtype=torch.int64, device="cuda")
                    got.append(ctx.compute_noalloc(dev, nbins, out, value_range="auto"))
                    for copies, window in ((8, 0), (2, 4096), (0, 1500)):
                        ctx.set_launch_shape(dev, nbins, copies=copies, window=window)
                        got.append(ctx.compute(dev, nbins, value_range="auto"))
                    got += ctx.compute_batch([dev], nbins, value_ranges=["auto"])
                    torch.cuda.synchronize()
                    for k, g in enumerate(got):
                        assert np.array_equal(g.cpu().numpy(), want), (cons, nbins, shape, dtype, k)
            ctx.autotune(dev, nbins, value_range="auto", reps=1)
            got = ctx.compute(dev, nbins, value_range="auto")
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy(), want), (cons, nbins, "tuned")
        finally:
            ctx.close()


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
def test_integer_levels_as_bins(oracle_mod, dtype):
    """The three binnings of integer data: the level itself (an AUTO range from 0 or
    the type's whole range, one bin per level), the level minus the lowest one with
    levels outside the range clamped, and the general one; data that start at 0 and
    that do not, and explicit ranges narrower than the data on either side.  2D, 3D
    and 4D, alone and in a batch."""
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(4500)
    top = int(np.iinfo(dtype).max)
    cases = []   # (lowest level, highest level, value range, bins)
    for lo, hi in ((0, 199), (17, 90), (top - 199, top), (3, 3), (0, 0)):
        cases += [(lo, hi, "auto", hi - lo + 1), (lo, hi, "auto", hi - lo + 2), (lo, hi, (lo, hi), hi - lo + 1)]
    cases += [(0, 199, (0, 120), 121), (0, 199, (40, 120), 81), (0, 199, (40, 255), 216), (0, 199, (40, 120), 50)]
    most = min(top + 1, 65535)
    cases += [(0, top, (0, top), most), (0, top, "auto", most), (0, top, (1, top), top), (0, top - 1, "auto", top)]
    for cons in ("vertex", "top"):
        ctx = ecc.Context(0, cons)
        try:
            for lo, hi, r, nbins in cases:
                hosts = []
                for shape in ((19, 131), (4, 9, 70), (2, 3, 8, 65)):
                    img = rng.integers(lo, hi + 1, size=shape).astype(dtype)
                    img.flat[0], img.flat[-1] = lo, hi
                    hosts.append(img)
                say(f"case: levels {cons} {np.dtype(dtype).name} [{lo}, {hi}] range={r} nbins={nbins}")
                devs = [to_dev(h) for h in hosts]
                want = [oracle_mod.ecc(h, nbins, cons, value_range=r, threads=8) for h in hosts]
                got = [ctx.compute(d, nbins, value_range=r) for d in devs]
                batch = ctx.compute_batch(devs, nbins, value_ranges=[r] * len(devs))
                torch.cuda.synchronize()
                for h, w, g, b in zip(hosts, want, got, batch):
                    assert np.array_equal(g.cpu().numpy(), w), (cons, lo, hi, r, nbins, h.shape)
                    assert np.array_equal(b.cpu().numpy(), w), (cons, lo, hi, r, nbins, h.shape, "batch")
        finally:
            ctx.close()


@pytest.mark.parametrize("cons", ["vertex", "top"])
def test_batch_parts_of_wave_tasks(oracle_mod, cons):
    """Batches whose waves take several steps each (planes, or groups of 16 rows) and
    start and end inside a wave task: ragged 2D and 3D images, blocks with fewer rows
    than the others, 4D pair volumes, each type, at 1 to 4 workgroups per CU."""
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(4600)
    shapes = [(int(a), int(b)) for a, b in zip(rng.integers(100, 1500, 12), rng.integers(20, 1500, 12))]
    shapes += [(129, 2500), (1700, 65), (17, 9000)]
    shapes += [tuple(int(n) for n in rng.integers(20, 120, 3)) for _ in range(8)] + [(260, 50, 60), (3, 30, 50, 64)]
    ctx = ecc.Context(0, cons)
    try:
        for kind in ("u8", "u16", "u16wide", "f32"):
            drawn = [draw_image(rng, s, kind) for s in shapes]
            nbins, r = drawn[0][1], drawn[0][2]
            hosts = [d[0] for d in drawn]
            devs = [to_dev(h) for h in hosts]
            want = [oracle_mod.ecc(h, nbins, cons, value_range=r, threads=8) for h in hosts]
            for part in (slice(0, 15), slice(15, 24), slice(0, None)):
                say(f"case: parts {cons} {kind} {part} nbins={nbins}")
                plan = ctx.plan_batch(devs[part], nbins, [r] * len(devs[part]))
                for tuned in (False, True):
                    if tuned:
                        plan.autotune(1)
                    for o in plan.outs:
                        o.fill_(-1)
                    plan.launch()
                    torch.cuda.synchronize()
                    for h, g, w in zip(hosts[part], plan.outs, want[part]):
                        assert np.array_equal(g.cpu().numpy(), w), (cons, kind, h.shape, tuned)
                plan.close()
    finally:
        ctx.close()
