"""GPU: calls that fit the documented scratch bound of ecc_reserve neither allocate
nor wait.  Growing the scratch waits for the whole device, so a call that grew it
would return only after the products that another stream is busy with."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def busy_stream():
    """A stream with about 100 ms of work on it, and the event that ends it."""
    a = torch.ones((8192, 8192), device="cuda", dtype=torch.bfloat16)
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(100):
            torch.mm(a, a, out=b)
        done = torch.cuda.Event()
        done.record(side)
    return done, (a, b, side)


def does_not_wait(call):
    done, keep = busy_stream()
    assert not done.query()
    out = call()
    waited = done.query()
    torch.cuda.synchronize()
    del keep
    assert not waited, "the call waited for the device"
    return out


def test_batch_of_three_types_and_few_bins():
    """Few images of three data types: as many workgroup segments as the bound has
    room for, each with the shortest row."""
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(61)
    vols = [torch.from_numpy(rng.integers(0, 100, size=(128, 128, 128)).astype(t)).cuda() for t in ("u1", "i2", "f4")]
    ranges = [(0, 99)] * 3
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    scratch, tables = ecc.batch_reserve_bytes(3, 3 * 128 ** 3, 1, cus)
    print(f"case: 3 volumes of 128^3, 1 bin, {scratch} bytes reserved", flush=True, file=sys.stderr)
    first, ctx = ecc.Context(0, "vertex"), ecc.Context(0, "vertex")
    try:
        first.compute_batch(vols, 1, value_ranges=ranges)   # loads the kernels
        ctx.reserve(scratch, tables)
        outs = torch.zeros((3, 1), dtype=torch.int64, device="cuda")
        does_not_wait(lambda: ctx.compute_batch(vols, 1, value_ranges=ranges, outs=list(outs)))
        assert outs.cpu().tolist() == [[1], [1], [1]]
    finally:
        first.close()
        ctx.close()


@pytest.mark.parametrize("wgs", [0, 1, 2, 16])
def test_wide_histogram_at_a_set_number_of_workgroups(oracle_mod, wgs):
    """16384 bins in one pass: 64 KB a workgroup row, two workgroups fit a CU, and the
    bound has room for one row per CU of that width."""
    from paper_2203_09087_amd import ecc
    rng = np.random.default_rng(62)
    host = rng.integers(0, 16384, size=(160, 160, 160)).astype(np.uint16)
    vol = torch.from_numpy(host.view(np.int16)).cuda()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    scratch, tables = ecc.batch_reserve_bytes(1, host.size, 16384, cus)
    print(f"case: 160^3 uint16, 16384 bins, {wgs} workgroups per CU, {scratch} bytes reserved", flush=True,
          file=sys.stderr)
    first, ctx = ecc.Context(0, "vertex"), ecc.Context(0, "vertex")
    try:
        first.compute(vol, 16384, value_range=(0, 16383))
        ctx.reserve(scratch, tables)
        ctx.set_launch_shape(vol, 16384, waves=4, depth=2, wgs_per_cu=wgs)   # 720 bricks
        out = torch.zeros(16384, dtype=torch.int64, device="cuda")
        does_not_wait(lambda: ctx.compute(vol, 16384, value_range=(0, 16383), out=out))
        assert np.array_equal(out.cpu().numpy(),
                              oracle_mod.ecc(host, 16384, "vertex", value_range=(0, 16383), threads=8))
    finally:
        first.close()
        ctx.close()


def test_a_tuned_shape_holds_no_window_above_4096_bins():
    """A shape tuned above 4096 bins is used for every such number of bins, so it names
    none of its own bins per pass (below, it may)."""
    from paper_2203_09087_amd import ecc
    vol = torch.randint(0, 16384, (6, 9, 20), device="cuda", dtype=torch.int16)
    ctx = ecc.Context(0, "vertex")
    try:
        for nbins in (4097, 5000, 16384, 40000):
            print(f"case: autotune at {nbins} bins", flush=True, file=sys.stderr)
            assert ctx.autotune(vol, nbins, value_range=(0, 16383), reps=1)["window"] == 0
    finally:
        ctx.close()
