"""GPU: 2D images whose blocks of rows span more than 4 GiB, so that no 32-bit byte
offset reaches from a block's first row to its last one.

The reference is the same image as one plane of a 3D volume (equal curves: the
plane's cells are the image's, times a point), whose march starts every strip of 6
rows from a 64-bit address; a small image pins that identity to the oracle.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (dtype, rows, columns, set depth): the default block of the first three is 48, 512
# and 208 rows; a batch takes blocks of 48, 112 and 112 rows
CASES = [("u8", 48, 1 << 27, 0), ("f32", 600, (1 << 21) + 5, 0), ("u16", 200, 1 << 24, 0),
         ("u16", 1100, 1 << 21, 4096)]
BINS = 64


def _image(kind, rows, cols):
    gen = torch.Generator(device="cuda").manual_seed(rows)
    if kind == "f32":
        return torch.rand((rows, cols), generator=gen, device="cuda", dtype=torch.float32), (0.0, 1.0)
    if kind == "u8":
        return torch.randint(0, 256, (rows, cols), generator=gen, device="cuda", dtype=torch.uint8), (0, 255)
    return torch.randint(0, 1 << 15, (rows, cols), generator=gen, device="cuda", dtype=torch.int16), (0, (1 << 15) - 1)


@pytest.mark.parametrize("cons", ["vertex", "top"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_blocks_beyond_four_gigabytes(oracle_mod, cons, case):
    from paper_2203_09087_amd import ecc
    kind, rows, cols, depth = CASES[case]
    ctx = ecc.Context(0, cons)
    try:
        img, r = _image(kind, rows, cols)
        print(f"case: {cons} {kind} {rows} x {cols} depth={depth}", flush=True, file=sys.stderr)
        if depth:
            ctx.set_launch_shape(img, BINS, depth=depth)
        got = ctx.compute(img, BINS, value_range=r)
        want = ctx.compute(img.view(1, rows, cols), BINS, value_range=r)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), want.cpu().numpy())
        if not depth:
            batch = ctx.compute_batch([img], BINS, value_ranges=[r])[0]
            torch.cuda.synchronize()
            assert np.array_equal(batch.cpu().numpy(), want.cpu().numpy())
        del img
        small = torch.randint(0, 256, (rows, 67), device="cuda", dtype=torch.uint8)
        plane = ctx.compute(small.view(1, rows, 67), BINS)
        assert np.array_equal(plane.cpu().numpy(), oracle_mod.ecc(small.cpu().numpy(), BINS, cons, threads=8))
    finally:
        ctx.close()
