"""GPU: small images, whose last workgroup merges the rows of all of them, called back
to back on the same scratch: a row that the merge reads before its workgroup has
written it would hold the call before's counts."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape,nbins", [((16, 16), 256), ((64, 64), 300), ((150, 150), 256), ((300, 300), 256),
                                         ((9, 20, 20), 64), ((40, 37, 29), 16)])
def test_small_calls_back_to_back(oracle_mod, shape, nbins):
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(4500)
    # two images with few values in common bins: the rows of one differ from the other's
    hosts = [(rng.integers(0, 128, size=shape)).astype(np.uint8), (rng.integers(100, 256, size=shape)).astype(np.uint8)]
    devs = [torch.from_numpy(h).cuda() for h in hosts]
    print(f"case: {shape} nbins={nbins}, 400 calls", flush=True, file=sys.stderr)
    ctx = ecc.Context(0, "vertex")
    try:
        outs = torch.full((400, nbins), -7, dtype=torch.int64, device="cuda")
        for k in range(400):
            ctx.compute(devs[k % 2], nbins, out=outs[k])
        torch.cuda.synchronize()
        got = outs.cpu().numpy()
        for k in range(2):
            want = oracle_mod.ecc(hosts[k], nbins, "vertex", threads=8)
            assert (got[k::2] == want[None, :]).all()
    finally:
        ctx.close()
