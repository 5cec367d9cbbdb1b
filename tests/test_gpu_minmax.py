"""GPU parity of the AUTO range of batches: the parts that the min/max pass cuts an
image into (16-byte groups, up to 32 parts per 2^20 elements) must cover every
element once, whatever the image's length and alignment.

Each image holds its smallest and its largest value at one position only, at the
ends of the image and around the edges of a part, so a missed element changes
the range and with it the curve."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def say(*args):
    print(*args, flush=True, file=sys.stderr)


@pytest.mark.parametrize("dtype", [np.uint16, np.float32])
@pytest.mark.parametrize("sizes", [
    [(1, 1), (1, 15), (17, 1), (3, 11)],
    [(1, 32767), (2, 16384), (1, 32769), (5, 6553)],
    [(1, 1 << 20), (3, 349525), (1025, 1023), (1, (1 << 20) + 17)],
])
def test_batch_auto_range_sees_every_element(oracle_mod, dtype, sizes):
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(77)
    hosts, devs = [], []
    for k, shape in enumerate(sizes * 3):
        n = int(np.prod(shape))
        if dtype == np.float32:
            a = rng.random(n).astype(np.float32)
            lo, hi = np.float32(-3.0), np.float32(5.0)
        else:
            a = rng.integers(1000, 2000, size=n).astype(np.uint16)
            lo, hi = 7, 60000
        edges = [0, n - 1, min(n - 1, 32768), min(n - 1, 32767), n // 2]
        a[edges[k % 5]] = lo
        a[edges[(k + 1) % 5]] = hi
        # an odd element offset into a larger buffer: unaligned 16-byte groups
        off = k % 3
        buf = np.zeros(n + 4, dtype=dtype)
        buf[off:off + n] = a
        base = torch.from_numpy(buf.view(np.int16) if dtype == np.uint16 else buf).cuda()
        hosts.append(a.reshape(shape))
        devs.append(base[off:off + n].view(shape))
    ctx = ecc.Context(0, "vertex")
    try:
        say(f"case: batch AUTO {np.dtype(dtype).name} {sizes}")
        got = ctx.compute_batch(devs, 500, value_ranges=["auto"] * len(devs))
        torch.cuda.synchronize()
        for h, g in zip(hosts, got):
            want = oracle_mod.ecc(h, 500, "vertex", value_range="auto", threads=8)
            assert np.array_equal(g.cpu().numpy(), want), h.shape
    finally:
        ctx.close()


@pytest.mark.parametrize("shape", [(1, 1), (1, 4096), (1, 4097), (3, 5, 700), (2050, 2049), (3, 2, 70, 90)])
def test_workgroups_fold_the_key_pairs(oracle_mod, shape):
    """A single image's AUTO range: 1 to 1024 key pairs, folded by workgroups of
    one to eight waves, the extremes at either end of the image."""
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(78)
    n = int(np.prod(shape))
    for cons in ("vertex", "top"):
        ctx = ecc.Context(0, cons)
        try:
            for ends in ((0, n - 1), (n - 1, 0)):
                a = rng.random(n).astype(np.float32)
                a[ends[1]] = 4.0
                a[ends[0]] = -2.0
                img = a.reshape(shape)
                d = torch.from_numpy(img).cuda()
                say(f"case: AUTO {cons} {shape} extremes at {ends}")
                want = oracle_mod.ecc(img, 700, cons, value_range="auto", threads=8)
                for waves in (0, 1, 3):
                    ctx.set_launch_shape(d, 700, waves=waves)
                    got = ctx.compute(d, 700, value_range="auto")
                    torch.cuda.synchronize()
                    assert np.array_equal(got.cpu().numpy(), want), (cons, shape, ends, waves)
        finally:
            ctx.close()
