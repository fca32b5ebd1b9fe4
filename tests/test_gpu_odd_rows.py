"""One-level transforms, tails and planned batches of rows that are not aligned
to the vectors: crops, odd pitches, detail bands at odd columns, and widths
that end inside a lane's vector. The same picture is transformed from an
aligned buffer with FP32 storage of the same 2-byte values, whose arithmetic
per quad is the same, so a result must be that one rounded once; and every
tile configuration must give the same bits.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1705_08266_amd as dwt  # noqa: E402
from paper_1705_08266_amd import batch as dwb  # noqa: E402

from test_gpu_head_strips import DTYPES, _crop, _empty  # noqa: E402

WIDTHS = [2, 4, 6, 10, 250, 254, 258, 502, 510]


@pytest.mark.parametrize("pad", [0, 1, 2, 7])
@pytest.mark.parametrize("width", WIDTHS)
@pytest.mark.parametrize("dtype", DTYPES)
def test_one_level(dtype, width, pad):
    print(f"case odd rows {dtype} width {width} pad {pad}", flush=True)
    for h in (2, 34):
        x = _crop(h, width, pad, dtype, 21)
        for wavelet in ("cdf97", "cdf53"):
            for scheme in ("nonseparable", "separable"):
                ref = dwt.forward(x.float().contiguous(), wavelet, 1, scheme).to(dtype)
                back = dwt.inverse(ref.float(), wavelet, 1, scheme).to(dtype)
                for tile in range(4):
                    out, rec = (_empty(h, width, pad, dtype) for _ in range(2))
                    dwt.forward(x, wavelet, 1, scheme, out=out[:, :width], tiles=[tile])
                    dwt.inverse(out[:, :width], wavelet, 1, scheme, out=rec[:, :width],
                                tiles=[tile])
                    assert torch.equal(ref, out[:, :width]), tile
                    assert torch.equal(back, rec[:, :width]), tile
                    if pad:   # nothing beyond the rows' ends is written
                        assert bool((out[:, width:] == -7).all())
                        assert bool((rec[:, width:] == -7).all())


@pytest.mark.parametrize("dtype", DTYPES)
def test_tails_and_batches(dtype):
    print(f"case odd rows in tails and batches {dtype}", flush=True)
    sizes = [(8, 8), (24, 504), (248, 136)]
    xs = [_crop(h, w, 3 * i + 1, dtype, 30 + i) for i, (h, w) in enumerate(sizes)]
    for levels in (1, 3):
        for inverse in (False, True):
            one = dwt.inverse if inverse else dwt.forward
            make = dwb.BatchPlan.inverse_of if inverse else dwb.BatchPlan.forward
            plan = make(xs, levels=levels)
            plan.run()
            for x, y in zip(xs, plan.outputs):
                ref = one(x.float().contiguous(), "cdf97", levels).to(dtype)
                assert torch.equal(ref, one(x, "cdf97", levels))
                assert torch.equal(ref, y)
