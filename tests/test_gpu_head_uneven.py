"""Planned heads of many short images and a tall one, by strips: a wavefront's
sweep ends with its own segment, so those of a workgroup pass its barriers
unevenly often, in persistent launches over several tasks too. Every output
must equal the one-launch-per-level result bit for bit.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1705_08266_amd as dwt  # noqa: E402
from paper_1705_08266_amd import batch as dwb  # noqa: E402

from test_gpu_head_strips import _crop  # noqa: E402


@pytest.mark.parametrize("inverse", [False, True])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("wavelet", ["cdf97", "cdf53"])
def test_short_images_and_a_tall_one(wavelet, dtype, inverse):
    # 9/7: more windows than any launch runs by windows, three to an image
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    sizes = [(4 * (1 + i % 5), 4 * (1 + i % 60)) for i in range(6 * cus)] + [(4096, 260)]
    xs = [_crop(h, w, 0, dtype, i) for i, (h, w) in enumerate(sizes)]
    one = dwt.inverse if inverse else dwt.forward
    make = dwb.BatchPlan.inverse_of if inverse else dwb.BatchPlan.forward
    expect = [one(x, wavelet, 2, tiles=[0, 0]) for x in xs]
    for persistent in (False, True):
        print(f"case uneven {wavelet} {dtype} inverse={inverse} persistent={persistent}",
              flush=True)
        plan = make(xs, levels=2, wavelet=wavelet, fuse_head=True, persistent=persistent)
        plan.run()
        for want, got in zip(expect, plan.outputs):
            assert torch.equal(want, got)
