"""GPU: a batch of more images than a grid's second and third axes hold (65536)."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_batch_of_seventy_thousand_images():
    """Images of one pixel: the curve of value v is 0 below its bin and 1 from it on."""
    from paper_2203_09087_amd import ecc
    count, bins = 70000, 4
    values = torch.from_numpy(np.random.default_rng(31).integers(0, bins, size=count).astype(np.uint8)).cuda()
    out = torch.full((count, bins), -7, dtype=torch.int64, device="cuda")
    print(f"case: {count} images of 1 x 1", flush=True, file=sys.stderr)
    ctx = ecc.Context(0, "vertex")
    try:
        ctx.compute_batch(list(values.view(count, 1, 1)), bins, value_ranges=[(0, bins - 1)] * count, outs=list(out))
        torch.cuda.synchronize()
        want = (torch.arange(bins, device="cuda")[None, :] >= values[:, None].long()).long()
        assert torch.equal(out, want)
    finally:
        ctx.close()
