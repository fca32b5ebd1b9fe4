"""Fused heads of 2-byte rows that start at odd halves of a word, by windows:
crops of odd pitches alone, in planned batches and in head level batches, with
and without images of whole words beside them, at the edges of a window (58
columns of level 2 by 18 rows forward, 22 inverse) and of an image. Every
output must equal the one-launch-per-level result bit for bit, and nothing
outside a row may be written.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1705_08266_amd as dwt  # noqa: E402
from paper_1705_08266_amd import batch as dwb  # noqa: E402
from paper_1705_08266_amd import serving as sv  # noqa: E402

import test_gpu_head_batch as hb  # noqa: E402
from test_gpu_head_strips import _both_ways, _crop  # noqa: E402

HALVES = [torch.float16, torch.bfloat16]


@pytest.mark.parametrize("shape", [(4, 4), (72, 232), (76, 236), (88, 228), (92, 468), (300, 700)])
@pytest.mark.parametrize("pad", [1, 7])
@pytest.mark.parametrize("dtype", HALVES)
def test_crops(dtype, pad, shape):
    print(f"case odd windows {dtype} pad {pad} {shape}", flush=True)
    h, w = shape
    x = _crop(h, w, pad, dtype, 31)
    off = _crop(h, w + 1, pad, dtype, 32)[:, 1:]     # pixels one column further on
    for wavelet in ("cdf97", "cdf53"):
        for scheme in ("nonseparable", "separable"):
            _both_ways(x, pad, wavelet, scheme)
            _both_ways(off, pad, wavelet, scheme)


@pytest.mark.parametrize("inverse", [False, True])
@pytest.mark.parametrize("wavelet", ["cdf97", "cdf53"])
@pytest.mark.parametrize("dtype", HALVES)
def test_batches_with_and_without_word_rows(dtype, wavelet, inverse):
    sizes = [(4, 4), (72, 232), (92, 468), (300, 700), (128, 64)]
    one = dwt.inverse if inverse else dwt.forward
    make = dwb.BatchPlan.inverse_of if inverse else dwb.BatchPlan.forward
    for odd in (1, len(sizes)):
        xs = [_crop(h, w, 7 if i < odd else 0, dtype, 40 + i) for i, (h, w) in enumerate(sizes)]
        expect = [one(x, wavelet, 2, tiles=[0, 0]) for x in xs]
        for persistent in (False, True):
            print(f"case odd batch {dtype} {wavelet} inverse={inverse} {odd} {persistent}",
                  flush=True)
            plan = make(xs, levels=2, wavelet=wavelet, fuse_head=True, persistent=persistent)
            plan.run()
            for want, got in zip(expect, plan.outputs):
                assert torch.equal(want, got)


@pytest.mark.parametrize("inverse", [False, True])
def test_head_level_batch(inverse):
    print(f"case odd head level batch inverse={inverse}", flush=True)

    def requests():
        out = []
        for i, (h, w) in enumerate([(68, 60), (232, 72), (4, 4), (700, 300)]):
            pad = 7 * (i % 2)
            src = _crop(h, w, pad, torch.float16, 50 + i)
            dst = torch.zeros(h, w + pad, dtype=src.dtype, device="cuda")[:, :w]
            ws = [torch.zeros(max(1, h * w // k), device="cuda") for k in (4, 16)]
            out.append((src, dst, *ws, sv.level_jobs(src, dst, *ws, 2, inverse)))
        return out

    a, b = requests(), requests()
    hb._run_levels(a, [0, 1], inverse)
    hb._run_head(b, (1, 2), 2, inverse)
    torch.cuda.synchronize()
    for ra, rb in zip(a, b):
        assert torch.equal(ra[1], rb[1]), tuple(ra[0].shape)
