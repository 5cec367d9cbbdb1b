"""GPU parity of volumes whose strips of 6 rows lie partly outside the image: 1 to 4
rows inside the last strip (and, top filtration, the first), alone and after whole
strips, against the oracle, bit for bit."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("cons", ["vertex", "top"])
@pytest.mark.parametrize("kind", ["u8", "u8levels", "u16", "u16wide", "f32"])
def test_few_rows_in_a_strip(oracle_mod, cons, kind):
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(4700)
    ctx = ecc.Context(0, cons)
    try:
        for rows in (1, 2, 3, 4, 7, 8, 9, 10, 13, 14, 15):
            for n0, n2 in ((5, 130), (17, 62)):
                shape = (n0, rows, n2)
                if kind == "f32":
                    img, nbins, r = rng.standard_normal(shape).astype(np.float32), 500, (-2.0, 2.0)
                    img[rng.random(shape) < 0.05] = np.nan
                elif kind == "u16wide":   # several windows
                    img, nbins, r = rng.integers(0, 65536, size=shape).astype(np.uint16), 40000, (0, 65535)
                elif kind == "u16":
                    img, nbins, r = rng.integers(0, 4096, size=shape).astype(np.uint16), 1000, (5, 4000)
                else:
                    img, nbins, r = rng.integers(0, 256, size=shape).astype(np.uint8), 256, (0, 255)
                    if kind == "u8levels":
                        nbins, r = 101, (100, 200)
                print(f"case: {cons} {kind} {shape}", flush=True, file=sys.stderr)
                dev = torch.from_numpy(img.view(np.int16) if img.dtype == np.uint16 else img).cuda()
                want = oracle_mod.ecc(img, nbins, cons, value_range=r, threads=8)
                for depth in (0, 3):
                    ctx.set_launch_shape(dev, nbins, depth=depth)
                    got = ctx.compute(dev, nbins, value_range=r)
                    torch.cuda.synchronize()
                    assert np.array_equal(got.cpu().numpy(), want), (cons, kind, shape, depth)
    finally:
        ctx.close()
