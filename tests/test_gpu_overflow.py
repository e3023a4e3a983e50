"""Values that overflow FP32 on the way (finite images, infinite filtered
projections)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def edge_pixel(L):
    """The pixel of the disk farthest from the centre: its projections reach the
    last bin."""
    a = 2 * np.arange(L) - L + 1
    r = a[:, None] ** 2 + a[None, :] ** 2
    return np.unravel_index(np.argmax(np.where(r <= (L - 2) ** 2, r, -1)), r.shape)


# columns by half waves, fused and staged, and by whole waves
@pytest.mark.parametrize("L,n,Q", [(64, 64, 32), (40, 96, 20), (130, 96, 16)])
@pytest.mark.parametrize("N", [1, 3])
def test_overflowed_filter_keeps_the_smallest_mass(tmp_path, L, n, Q, N):
    """One pixel whose ramp-filtered projections overflow in the last bins,
    where the scan of the column turns the infinity into a NaN: the smallest
    part mass (aux[0]) is the same finite number whether an image has many
    blocks or one, and so are the tables."""
    import torch
    from paper_2503_13756_amd import api

    imgs = np.zeros((N, L, L), np.float32)
    # between 1.4e39 / L, where bin L - 1 overflows at half weight, and 2.4e39 / L,
    # where contributions of both signs can overflow together and make a NaN
    imgs[N - 1][edge_pixel(L)] = 1.9e39 / L
    for k in range(N - 1):
        imgs[k, L // 2, L // 2 - k] = 1.0
    x = torch.from_numpy(imgs).cuda()
    out = {}
    for name, lim in (("small", 1 << 30), ("large", 0)):
        path = tmp_path / f"{name}.json"
        path.write_text('{"small_batch": %d}' % lim)
        ctx = api.Context(0, tune_json=str(path))
        q, a = api.tables(ctx, x, n, Q, ramp=True)
        out[name] = (q.cpu().numpy().view(np.uint32), a.cpu().numpy())
        if name == "small":
            pf = api.ramp(ctx, api.project(ctx, x, n))[N - 1].cpu().numpy()
        ctx.close()
    assert np.isinf(pf[:, L - 1]).any() and not np.isnan(pf).any()
    assert np.isfinite(out["large"][1][:, 0]).all()
    assert np.array_equal(out["small"][1].view(np.uint64), out["large"][1].view(np.uint64))
    assert np.array_equal(out["small"][0], out["large"][0])
