"""The rows per segment that a planned head launch gives its strips, read from
plans built on the host. A strip walks the rows of its segment and a few more,
so a launch of many images takes at least (segment + halo) row pairs per strip:
one tall image among thousands of small ones must not make theirs tall."""
import ctypes
import struct

import pytest
import torch

from paper_1705_08266_amd import _lib

from test_batch_plan_host import FAKE, HEADER, LAUNCH

# sizeof of the launch's parameters per image; the segment is their last field
PARAMS = {0: 216, 1: 200}
OWN, HALO = 48, 6


def _plan_of(sizes, dtype, wavelet, inverse, pad=0):
    """The plan of one head launch of images whose rows are `pad` elements longer."""
    lib = _lib.load()
    es = 4 if dtype == _lib.F32 else 2
    arr = (_lib.Image * len(sizes))()
    base = FAKE
    for i, (w, h) in enumerate(sizes):
        ws = lib.dwt2_workspace_bytes(w, h, 2, dtype)
        p, n = w + pad, (w + pad) * h * es
        arr[i] = _lib.Image(base, p, base + n, p, base + 2 * n + 2 * n % 4, ws, w, h)
        base += 2 * n + ws + 4096 - n % 4
    n = ctypes.c_size_t()
    args = (arr, len(sizes), dtype, wavelet, 2, inverse, 0, None, _lib.PLAN_HEAD)
    assert lib.dwt2_batch_plan_bytes(*args, ctypes.byref(n)) == 0
    buf = (ctypes.c_ubyte * n.value)()
    assert lib.dwt2_batch_plan(*args, buf, n.value) == 0
    assert HEADER.unpack_from(buf)[7] == 1
    return bytes(buf)


def _head(sizes, dtype, wavelet, inverse, pad=0):
    """(segment, 0 for windows, row pairs that a launch with it walks, and with 18)
    of a plan of images whose rows are `pad` elements longer."""
    buf = _plan_of(sizes, dtype, wavelet, inverse, pad)
    off = LAUNCH.unpack_from(buf, HEADER.size)[8]
    seg = struct.unpack_from("<i", buf, off + PARAMS[inverse] - 4)[0]

    def pairs(rows):
        return sum(-(-(w // 4) // OWN) * -(-(h // 4) // rows) * (rows + HALO) for w, h in sizes)

    return seg, pairs(seg) if seg else 0, pairs(18)


@pytest.mark.parametrize("inverse", [0, 1])
@pytest.mark.parametrize("dtype", [_lib.F32, _lib.F16, _lib.BF16])
@pytest.mark.parametrize("small,count", [(64, 4000), (64, 5000), (32, 6000), (128, 2500)])
def test_one_tall_image_among_small_ones(dtype, inverse, small, count):
    """At most twice the row pairs of segments of 18 rows."""
    seg, walked, short = _head([(small, small)] * count + [(4096, 4096)], dtype, 0, inverse)
    assert seg > 0 and walked <= 2 * short, (seg, walked, short)


@pytest.mark.parametrize("inverse", [0, 1])
@pytest.mark.parametrize("dtype", [_lib.F32, _lib.F16])
def test_small_images_alone(dtype, inverse):
    for count in (1100, 4200, 8000):
        seg, walked, short = _head([(32, 32)] * count, dtype, 0, inverse)
        assert seg == 8 or seg == 0, seg     # no taller than the images


@pytest.mark.parametrize("inverse", [0, 1])
@pytest.mark.parametrize("wavelet", [0, 1])
@pytest.mark.parametrize("dtype", [_lib.F16, _lib.BF16])
def test_rows_at_odd_halves_of_a_word(dtype, wavelet, inverse):
    """A launch of few windows runs by windows, whatever its rows start at."""
    for sizes in ([(256, 256)], [(608, 128)], [(1024, 960), (64, 64)], [(2048, 2048)]):
        assert _head(sizes, dtype, wavelet, inverse, pad=7)[0] == 0, sizes
    assert _head([(16384, 16384)], dtype, wavelet, inverse, pad=7)[0] > 0


@pytest.mark.parametrize("wavelet,dtype,inverse,windows,strips", [
    (0, _lib.F32, 0, [1, 2], [2.25]), (0, _lib.F32, 1, [1, 2], [2.25]),
    (0, _lib.F16, 0, [1, 4.5], [4.75]), (0, _lib.F16, 1, [3.25, 5.25], [5.5]),
    (1, _lib.F16, 1, [0.5, 1.5, 2], [0.25, 2.25]),
    (1, _lib.F32, 1, [0.875, 1, 1.75, 2], [0.5, 1.25, 2.25]),
    (1, _lib.F16, 0, [], [0.5, 2]), (1, _lib.F32, 0, [], [0.5, 2])])
def test_windows_or_strips(wavelet, dtype, inverse, windows, strips):
    """Windows per compute unit at which a launch runs by either, one window across."""
    cus = 256                      # where no device says otherwise
    if torch.cuda.is_available():
        cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows = 88 if inverse else 72
    for per_cu in windows + strips:
        seg = _head([(232, int(per_cu * cus) * rows)], dtype, wavelet, inverse)[0]
        assert (seg == 0) == (per_cu in windows), per_cu


@pytest.mark.parametrize("inverse", [0, 1])
@pytest.mark.parametrize("dtype", [_lib.F32, _lib.F16])
@pytest.mark.parametrize("sizes", [[(4096, 4096), (64, 96), (196, 52)], [(64, 64)] * 9])
def test_a_plan_holds_the_map_of_the_layout_that_runs(sizes, dtype, inverse):
    """And no other: its tasks, image by image, are all that its bytes hold
    beside the parameters."""
    plan = _plan_of(sizes, dtype, 0, inverse)
    images, total, img, start, params = LAUNCH.unpack_from(plan, HEADER.size)[4:]
    seg = struct.unpack_from("<i", plan, params + PARAMS[inverse] - 4)[0]
    tall = 22 if inverse else 18
    counts = [-(-(w // 4) // (OWN if seg else 58)) * -(-(h // 4) // (seg or tall))
              for w, h in sizes]
    assert images == len(sizes) and total == sum(counts)
    starts = [sum(counts[:i]) for i in range(images)]
    assert list(struct.unpack_from(f"<{images}i", plan, start)) == starts
    assert list(struct.unpack_from(f"<{total}i", plan, img)) == [
        i for i, c in enumerate(counts) for _ in range(c)]
    assert len(plan) <= HEADER.size + LAUNCH.size + 4 * (total + images) + \
        PARAMS[inverse] * images + 5 * 256
