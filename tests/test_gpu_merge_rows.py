"""GPU: the merge of batches whose images have few partial rows each (a thread per bin,
or per four bins), against the oracle, bit for bit: one row and several per image,
a batch with one image of more rows than that merge takes, bins that end inside a
block of 256 or 1024, several windows, and signed 4D volumes.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (images, bins): blocks of 256 bins; of 1024 from 4096 blocks of 256 bins on; several
# windows; up to 16 rows each, and more than 16 for one of them
BATCHES = [([(5, 7)] * 40 + [(40, 37, 29)], 1), ([(16, 16)] * 300, 257), ([(16, 16)] * 300 + [(60, 60, 60)], 4096),
           ([(3, 5)] * 1100, 1025), ([(20, 30)] * 30 + [(3, 8, 9, 10)], 5000), ([(1500, 1500)] + [(8, 8)] * 5, 300)]


@pytest.mark.parametrize("cons", ["vertex", "top"])
@pytest.mark.parametrize("case", range(len(BATCHES)))
def test_merge_of_few_rows(oracle_mod, cons, case):
    from paper_2203_09087_amd import ecc
    shapes, bins = BATCHES[case]
    rng = np.random.default_rng(4600 + case)
    hosts = [rng.integers(0, 65536, size=s).astype(np.uint16) for s in shapes]
    devs = [torch.from_numpy(h.view(np.int16)).cuda() for h in hosts]
    print(f"case: {cons} {len(shapes)} images, {bins} bins", flush=True, file=sys.stderr)
    ctx = ecc.Context(0, cons)
    try:
        out = torch.full((len(hosts), bins), -7, dtype=torch.int64, device="cuda")
        ctx.compute_batch(devs, bins, value_ranges=[(0, 65535)] * len(devs), outs=list(out))
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        for k, h in enumerate(hosts):
            want = oracle_mod.ecc(h, bins, cons, value_range=(0, 65535), threads=8 if h.size > 10000 else 1)
            assert np.array_equal(got[k], want), (k, h.shape)
    finally:
        ctx.close()
