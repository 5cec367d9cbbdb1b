"""GPU parity of the one-launch smoothing at the edges of its tiles (64 x 32
outputs, a halo of 6), against the oracle and against the in-place passes, bit for
bit (the filter has one exact float32 result)."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [(1, 63), (31, 65), (32, 64), (33, 63), (38, 70), (39, 129), (64, 6), (7, 200),
                                   (97, 58)])
def test_tile_edges(oracle_mod, shape):
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(73)
    img = rng.standard_normal(shape).astype(np.float32)
    img[0, -1], img[-1, 0] = np.inf, -0.0
    taps = rng.uniform(-1, 1, 13).astype(np.float32)
    print(f"case: smooth tile {shape}", flush=True, file=sys.stderr)
    ctx = ecc.Context(0, "vertex")
    try:
        d = torch.from_numpy(img).cuda()
        got = ctx.smooth13(d, taps)
        torch.cuda.synchronize()
        want = oracle_mod.smooth13(img, taps)
        assert np.array_equal(got.cpu().numpy(), want, equal_nan=True)
        ctx.smooth13(d, taps, out=d)
        torch.cuda.synchronize()
        assert np.array_equal(d.cpu().numpy(), want, equal_nan=True)
    finally:
        ctx.close()
