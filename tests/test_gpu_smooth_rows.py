"""GPU parity of the one-launch smoothing at heights around its tiles of 16 rows (64
columns wide), against the oracle and the in-place passes, bit for bit."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [(15, 64), (16, 65), (17, 63), (22, 70), (23, 128), (48, 129), (49, 3)])
def test_tile_heights(oracle_mod, shape):
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(74)
    img = rng.standard_normal(shape).astype(np.float32)
    img[0, -1], img[-1, 0] = np.inf, -0.0
    taps = rng.uniform(-1, 1, 13).astype(np.float32)
    print(f"case: smooth {shape}", flush=True, file=sys.stderr)
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
