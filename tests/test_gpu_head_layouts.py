"""The fused head by windows and by strips: launches on both sides of the line
between the two, and 9/7 strips, which take launches of more windows than fit
on the chip, at their edges. A window is 58 columns of level 2 by 18 rows
(forward) or 22 (inverse), so tall or wide thin images cross the line with few
pixels. Every output must equal the one-launch-per-level result bit for bit:
the per-quad arithmetic is the same.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1705_08266_amd as dwt  # noqa: E402
from paper_1705_08266_amd import batch as dwb  # noqa: E402

import test_gpu_head_batch as hb  # noqa: E402
from test_gpu_head_strips import DTYPES, HEAD, _both_ways, _crop  # noqa: E402


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("wavelet,dtype,inverse,eighths",
                         [("cdf97", torch.float32, False, 16), ("cdf97", torch.float16, False, 40),
                          ("cdf97", torch.float32, True, 16), ("cdf97", torch.bfloat16, True, 24),
                          ("cdf97", torch.float16, True, 48),
                          ("cdf53", torch.float16, True, 3), ("cdf53", torch.bfloat16, True, 11)])
def test_both_sides_of_the_line(wavelet, dtype, inverse, eighths):
    """Launches of exactly the windows of the line, and of one more."""
    windows = eighths * _cus() // 8
    for more in (0, 4):
        h = windows * (88 if inverse else 72) + more
        print(f"case line {wavelet} {dtype} inverse={inverse} {h} rows", flush=True)
        x = _crop(h, 68, 0, dtype, 11)
        one = dwt.inverse if inverse else dwt.forward
        assert torch.equal(one(x, wavelet, 2, tiles=[0, 0]), one(x, wavelet, 2, tiles=HEAD))


def _thin(k):
    """Windows of either direction beyond 6 per compute unit, and k pixels."""
    return (6 * _cus() + 1) * 88 + k


@pytest.mark.parametrize("width", [4, 192, 196, 584])
@pytest.mark.parametrize("dtype,pad", [(torch.float32, 0), (torch.float32, 7), (torch.float16, 0),
                                       (torch.float16, 7), (torch.bfloat16, 2)])
def test_strips_of_tall_images(dtype, pad, width):
    print(f"case tall {dtype} pad {pad} width {width}", flush=True)
    for scheme in ("nonseparable", "separable"):
        _both_ways(_crop(_thin(4), width, pad, dtype, 12), pad, "cdf97", scheme)


@pytest.mark.parametrize("height", [4, 8, 68, 100])
@pytest.mark.parametrize("dtype", DTYPES)
def test_strips_of_wide_images(dtype, height):
    print(f"case wide {dtype} height {height}", flush=True)
    w = (6 * _cus() + 1) * 58 * 4 + 4
    for pad in ((0,) if dtype == torch.float32 else (0, 7)):
        _both_ways(_crop(height, w, pad, dtype, 13), pad, "cdf97", "nonseparable")


@pytest.mark.parametrize("inverse", [False, True])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_planned_batch_by_strips(dtype, inverse):
    sizes = [(4, 4), (68, 196), (_thin(0), 60), (520, 1000), (132, 60)]
    xs = [_crop(h, w, 7 * (i % 2), dtype, 70 + i) for i, (h, w) in enumerate(sizes)]
    one = dwt.inverse if inverse else dwt.forward
    make = dwb.BatchPlan.inverse_of if inverse else dwb.BatchPlan.forward
    for persistent in (False, True):
        print(f"case batch {dtype} inverse={inverse} persistent={persistent}", flush=True)
        plan = make(xs, levels=2, fuse_head=True, persistent=persistent)
        plan.run()
        for x, y in zip(xs, plan.outputs):
            assert torch.equal(one(x.contiguous(), "cdf97", 2, tiles=[0, 0]), y)


@pytest.mark.parametrize("inverse", [False, True])
def test_head_level_batch_by_strips(monkeypatch, inverse):
    print(f"case head level batch inverse={inverse}", flush=True)
    monkeypatch.setattr(hb, "SIZES", [(60, 68), (200, _thin(0)), (4, 4), (392, 1028)])
    a = hb._requests(2, inverse, torch.float16, seed=300)
    b = hb._requests(2, inverse, torch.float16, seed=300)
    hb._run_levels(a, [0, 1], inverse)
    hb._run_head(b, (1, 2), 2, inverse)
    torch.cuda.synchronize()
    for ra, rb in zip(a, b):
        assert torch.equal(ra[1], rb[1]), tuple(ra[0].shape)


@pytest.mark.parametrize("pad", [0, 16, 7])
def test_windows_of_rows_off_the_sectors(pad):
    """FP32 forwards of more windows than the line, by windows where the band
    rows are off the 64-byte sectors, else by strips."""
    h, w = _thin(4), 128
    print(f"case off sectors pad {pad}", flush=True)
    x = _crop(h, w, pad, torch.float32, 14)
    out = torch.full((h, w + pad), -7.0, device="cuda")
    dwt.forward(x, "cdf97", 2, out=out[:, :w], tiles=HEAD)
    assert torch.equal(dwt.forward(x, "cdf97", 2, tiles=[0, 0]), out[:, :w])
    assert bool((out[:, w:] == -7).all())
