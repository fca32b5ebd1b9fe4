"""The fused head's strips and segments, and its ways of addressing rows.

A strip owns 48 columns of level 2 (192 pixels), a segment some of its rows; a
launch picks the segment by the image. Rows are reached from one resource per
segment, with 2-byte rows that are not word aligned shifted into place, or from
one resource per row where rows lie too far apart. Every output must equal the
one-launch-per-level result bit for bit: the per-quad arithmetic is the same.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1705_08266_amd as dwt  # noqa: E402
from paper_1705_08266_amd import _lib  # noqa: E402
from paper_1705_08266_amd import batch as dwb  # noqa: E402

HEAD = [_lib.TILE_HEAD] * 2
DTYPES = [torch.float32, torch.float16, torch.bfloat16]


def _crop(h, w, pad, dtype, seed):
    """A random image as a crop of a buffer whose rows are `pad` longer."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randint(0, 256, (h, w + pad), generator=g, device="cuda").to(dtype)
    return x[:, :w]


def _empty(h, w, pad, dtype):
    return torch.full((h, w + pad), -7.0, device="cuda", dtype=dtype)


def _both_ways(x, pad, wavelet, scheme):
    h, w = x.shape
    per, fus = _empty(h, w, 0, x.dtype), _empty(h, w, pad, x.dtype)
    dwt.forward(x, wavelet, 2, scheme, out=per, tiles=[0, 0])
    dwt.forward(x, wavelet, 2, scheme, out=fus[:, :w], tiles=HEAD)
    assert torch.equal(per, fus[:, :w])
    back, fback = _empty(h, w, 0, x.dtype), _empty(h, w, pad, x.dtype)
    dwt.inverse(fus[:, :w], wavelet, 2, scheme, out=back, tiles=[0, 0])
    dwt.inverse(fus[:, :w], wavelet, 2, scheme, out=fback[:, :w], tiles=HEAD)
    assert torch.equal(back, fback[:, :w])
    if pad:   # nothing beyond the rows' ends is written
        assert bool((fus[:, w:] == -7).all()) and bool((fback[:, w:] == -7).all())


@pytest.mark.parametrize("shape", [(4, 4), (4, 192), (196, 4), (64, 188), (72, 196), (100, 384),
                                   (388, 580), (1028, 768)])
@pytest.mark.parametrize("pad", [0, 2, 7])
@pytest.mark.parametrize("dtype", DTYPES)
def test_strip_edges_and_crops(dtype, pad, shape):
    print(f"case strips {dtype} pad {pad} {shape}", flush=True)
    x = _crop(*shape, pad, dtype, 3)
    for wavelet in ("cdf97", "cdf53"):
        for scheme in ("nonseparable", "separable"):
            _both_ways(x, pad, wavelet, scheme)


@pytest.mark.parametrize("shape,dtype", [((4100, 2052), torch.float32),     # streamed inverse
                                         ((4100, 4104), torch.float16),
                                         ((8196, 8196), torch.float32)])    # streamed bands
def test_many_segments(shape, dtype):
    print(f"case segments {shape} {dtype}", flush=True)
    _both_ways(_crop(*shape, 0, dtype, 4), 0, "cdf97", "nonseparable")


@pytest.mark.parametrize("dtype,pitch", [(torch.float32, 1 << 24), (torch.float16, (1 << 24) + 1)])
def test_rows_far_apart(dtype, pitch):
    """16 rows of 200 pixels, 64 or 32 MiB apart."""
    print(f"case far rows {dtype}", flush=True)
    h, w = 16, 200
    src = torch.zeros(h * pitch, device="cuda", dtype=dtype)
    x = torch.as_strided(src, (h, w), (pitch, 1))
    x.copy_(_crop(h, w, 0, dtype, 5))
    dst = torch.zeros(h * pitch, device="cuda", dtype=dtype)
    far = torch.as_strided(dst, (h, w), (pitch, 1))
    for wavelet in ("cdf97", "cdf53"):
        near = dwt.forward(x.contiguous(), wavelet, 2, tiles=[0, 0])
        dwt.forward(x, wavelet, 2, out=far, tiles=HEAD)
        assert torch.equal(near, far)
        back = torch.as_strided(src, (h, w), (pitch, 1))
        dwt.inverse(far, wavelet, 2, out=back, tiles=HEAD)
        assert torch.equal(dwt.inverse(near, wavelet, 2, tiles=[0, 0]), back)


@pytest.mark.parametrize("inverse", [False, True])
@pytest.mark.parametrize("persistent", [False, True])
def test_planned_batch_of_uneven_crops(persistent, inverse):
    """Workgroups whose strips belong to different images."""
    sizes = [(4, 4), (68, 196), (12, 388), (256, 192), (520, 1000), (132, 60), (1024, 64)]
    xs = [_crop(h, w, 7 * (i % 2), torch.float16, 60 + i) for i, (h, w) in enumerate(sizes)]
    print(f"case batch of crops inverse={inverse} persistent={persistent}", flush=True)
    make = dwb.BatchPlan.inverse_of if inverse else dwb.BatchPlan.forward
    plan = make(xs, levels=2, fuse_head=True, persistent=persistent)
    plan.run()
    one = dwt.inverse if inverse else dwt.forward
    for x, y in zip(xs, plan.outputs):
        assert torch.equal(one(x.contiguous(), "cdf97", 2, tiles=[0, 0]), y)
