"""Every layout of the fused head, each checked to be the one that runs: windows
and strips on both sides of the line between them, strips of rows at odd halves
of a word and of rows far apart, streamed bands and streamed pixels. Every
output must equal the one-launch-per-level result bit for bit, and nothing
outside a row may be written.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1705_08266_amd as dwt  # noqa: E402

from test_gpu_head_strips import DTYPES, HEAD, _crop, _empty  # noqa: E402

WINDOWS, STRIPS = "windows", "strips"
F32, F16, BF16 = DTYPES


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def _check(x, wavelet, inverse, layout, streamed=False, pad=0, out=None):
    """x is the image or the pyramid; the other has rows `pad` elements longer."""
    h, w = x.shape
    one = dwt.inverse if inverse else dwt.forward
    if out is None:
        out = _empty(h, w, pad, x.dtype)
    rows, tasks, stream = dwt.head_layout(x, out[:, :w], wavelet, 2, inverse)
    assert (STRIPS if rows else WINDOWS) == layout and stream == streamed, (rows, tasks, stream)
    for scheme in ("nonseparable", "separable"):
        print(f"case reach {tuple(x.shape)} {x.dtype} {wavelet} inverse={inverse} {layout} "
              f"streamed={streamed} pad={pad} {scheme}", flush=True)
        want = one(x, wavelet, 2, scheme, out=_empty(h, w, 0, x.dtype), tiles=[0, 0])
        one(x, wavelet, 2, scheme, out=out[:, :w], tiles=HEAD)
        assert torch.equal(want, out[:, :w])
    if pad:
        assert bool((out[:, w:] == -7).all())


# windows per compute unit up to which launches of one window across run by them
@pytest.mark.parametrize("wavelet,dtype,inverse,per_cu,pad", [
    ("cdf97", F32, False, 2, 0), ("cdf97", F32, True, 2, 0), ("cdf97", F16, False, 4.5, 0),
    ("cdf97", BF16, True, 5.25, 0), ("cdf53", F32, True, 1, 0), ("cdf53", F32, True, 2, 0),
    ("cdf53", F16, True, 2, 0), ("cdf97", F16, False, 8, 7), ("cdf97", BF16, True, 8, 7),
    ("cdf53", BF16, False, 2.5, 7), ("cdf53", F16, True, 4, 7)])
def test_both_sides_of_every_line(wavelet, dtype, inverse, per_cu, pad):
    h = int(per_cu * _cus()) * (88 if inverse else 72)
    for more, layout in ((0, WINDOWS), (4, STRIPS)):
        _check(_crop(h + more, 68, pad, dtype, 61), wavelet, inverse, layout, pad=pad)


@pytest.mark.parametrize("width", [4, 192, 196, 584])
@pytest.mark.parametrize("dtype,pad", [(F32, 0), (F32, 7), (F16, 0), (F16, 7), (BF16, 1)])
def test_strips_of_tall_images(dtype, pad, width):
    """Widths at the edges of a strip. FP32 forwards of rows off the 64-byte
    sectors run by windows there."""
    x = _crop((8 * _cus() + 1) * 88 + 4, width, pad, dtype, 62)
    for wavelet in ("cdf97", "cdf53"):
        off = dtype == F32 and wavelet == "cdf97" and (pad or width % 32)
        size = x.numel() * x.element_size()
        _check(x, wavelet, False, WINDOWS if off else STRIPS, not off and size > 256 << 20, pad)
        _check(x, wavelet, True, STRIPS, size >= 32 << 20, pad)


@pytest.mark.parametrize("height", [4, 8, 68, 100])
@pytest.mark.parametrize("dtype,pad", [(F32, 0), (F16, 0), (F16, 7), (BF16, 1)])
def test_strips_of_wide_images(dtype, pad, height):
    """Heights at the edges of an image."""
    w = (8 * _cus() + 1) * 232 + 28
    x = _crop(height, w, pad, dtype, 63)
    big = x.numel() * x.element_size() >= 32 << 20
    for inverse in (False, True):
        off = dtype == F32 and not inverse
        _check(x, "cdf97", inverse, WINDOWS if off else STRIPS, streamed=inverse and big, pad=pad)
        _check(x, "cdf53", inverse, STRIPS, streamed=inverse and big, pad=pad)


@pytest.mark.parametrize("dtype,pitch", [(F32, 1 << 24), (F16, 1 << 25), (F16, (1 << 24) + 1),
                                         (BF16, (1 << 24) + 1)])
@pytest.mark.parametrize("inverse", [False, True])
def test_strips_of_rows_far_apart(dtype, pitch, inverse):
    """8 rows, 32 or 64 MiB apart: no resource reaches a segment's rows."""
    w = ((8 * _cus() + 1) * 232 + 31) // 32 * 32
    x = torch.zeros(8 * pitch, device="cuda", dtype=dtype).as_strided((8, w), (pitch, 1))
    x.copy_(_crop(8, w, 0, dtype, 64))
    far = torch.full((8 * pitch,), -7.0, device="cuda", dtype=dtype).as_strided((8, w), (pitch, 1))
    for wavelet in ("cdf97", "cdf53"):
        _check(x, wavelet, inverse, STRIPS, out=far)


@pytest.mark.parametrize("dtype,shape", [(F32, (8200, 8192)), (F16, (16400, 8192)),
                                         (BF16, (16388, 8256))])
def test_streamed_bands(dtype, shape):
    """Forwards of more than 256 MiB by strips."""
    x = _crop(*shape, 0, dtype, 65)
    for wavelet in ("cdf97", "cdf53"):
        _check(x, wavelet, False, STRIPS, streamed=True)


@pytest.mark.parametrize("dtype,shape,layout", [(F32, (3076, 4096), STRIPS), (F32, (4100, 5508), STRIPS),
                                                (F16, (5124, 5636), STRIPS),
                                                (F16, (4100, 4104), WINDOWS),
                                                (BF16, (4104, 4096), WINDOWS)])
def test_streamed_pixels(dtype, shape, layout):
    """Inverses of 32 MiB and more."""
    _check(_crop(*shape, 0, dtype, 66), "cdf97", True, layout, streamed=True)
    _check(_crop(*shape, 0, dtype, 66), "cdf53", True, STRIPS, streamed=True)


@pytest.mark.parametrize("dtype", DTYPES)
def test_several_segments_not_streamed(dtype):
    for shape in ((3396, 3652), (2308, 5380)):
        for wavelet in ("cdf97", "cdf53"):
            layout = WINDOWS if dtype != F32 and wavelet == "cdf97" else STRIPS
            _check(_crop(*shape, 0, dtype, 67), wavelet, False, layout)


def test_head_layout_refuses_what_the_transform_refuses():
    x, y = _empty(64, 64, 0, F32), _empty(64, 64, 0, F32)
    assert dwt.head_layout(x, y)[0] == 0
    for bad in (lambda: dwt.head_layout(x, y, levels=1), lambda: dwt.head_layout(x, x),
                lambda: dwt.head_layout(x, y[:32]), lambda: dwt.head_layout(x, y, levels=7)):
        with pytest.raises(dwt.DWT2Error):
            bad()
