"""Projections of geometries with more tasks than a block of 512 threads holds."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


# (L, n) of one and of several groups of 144 tasks, odd sides, a side of several strips
@pytest.mark.parametrize("L,n", [(256, 256), (255, 192), (200, 256), (162, 512), (73, 512)])
def test_images_per_block(tmp_path, L, n):
    """One image per block (as many as compute units at most), two (more) and
    the blocks of a small batch: the same bits, a NaN image among them."""
    import torch
    from paper_2503_13756_amd import api

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    _, imgs = synth.make_raw_stack(40 + L, L, 3)
    imgs[1, L // 3, L // 2] = np.nan
    x = torch.from_numpy(np.ascontiguousarray(imgs.astype(np.float32))).cuda()
    path = tmp_path / "large.json"
    path.write_text('{"small_batch": 0}')
    small, large = api.Context(0), api.Context(0, tune_json=str(path))
    few = api.project(small, x, n).view(torch.int32)
    for N in (1, 3, cus, cus + 1):
        at = torch.arange(N, device="cuda") % 3
        got = api.project(large, x[at].contiguous(), n).view(torch.int32)
        assert torch.equal(got, few[at]), N
    for c in (small, large):
        c.close()
