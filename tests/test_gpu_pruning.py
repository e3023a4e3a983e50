"""All-pairs BF16 form: candidates that its error bound rules out are not
rescored, and the records are those of rescoring every candidate."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def contexts(tmp_path_factory):
    """One context that prunes and one that is told not to."""
    from paper_2503_13756_amd import api

    path = tmp_path_factory.mktemp("tune") / "every.json"
    path.write_text('{"all_pairs_rescore": "every"}')
    pair = api.Context(0), api.Context(0, tune_json=str(path))
    yield pair
    for c in pair:
        c.close()


def images(L, count, seed):
    """Blobs, clean and noisy, and nearly symmetric images whose curves are
    almost flat."""
    import torch

    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ax = (torch.arange(L, device="cuda") - (L - 1) / 2) * (2.0 / L)

    def rand(*shape):
        return torch.rand(*shape, generator=gen, device="cuda")

    c = 1.2 * rand(count, 6, 2) - 0.6
    gx = torch.exp(-((ax - c[..., :1]) ** 2) / 0.02)
    gy = torch.exp(-((ax - c[..., 1:]) ** 2) / 0.02)
    x = torch.bmm(gy.transpose(1, 2).contiguous(), gx.contiguous())
    disc = torch.exp(-(ax[:, None] ** 2 + ax[None, :] ** 2) / 0.1)
    third = count // 3
    x[third:2 * third] += 0.3 * rand(third, L, L)
    x[2 * third:] = disc + 10.0 ** (-5.0 * rand(count - 2 * third, 1, 1)) * rand(
        count - 2 * third, L, L)
    return x.contiguous()


# few tables, whose spectra many blocks share; ragged tiles; more than one tile
# of references a block; every candidate count
@pytest.mark.parametrize("n", [32, 64])
@pytest.mark.parametrize("refs,count", [(1, 300), (17, 31), (200, 333)])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("top_k", [2, 4])
def test_records_of_every_candidate(contexts, n, refs, count, mode, top_k):
    import torch
    from paper_2503_13756_amd import api

    x = images(n, refs + count, 11 * n + refs)
    res = []
    for ctx in contexts:
        q, a = api.tables(ctx, x, n, n)
        r, _ = api.align_batch(ctx, q[:refs].contiguous(), a[:refs].contiguous(),
                               q[refs:].contiguous(), a[refs:].contiguous(), n, mode=mode, prec=1,
                               top_k=top_k)
        res.append(r)
    assert torch.equal(res[0], res[1])


@pytest.mark.parametrize("n", [32, 64])
@pytest.mark.parametrize("eps", [1e-2, 1e-3, 1e-4, 1e-5])
@pytest.mark.parametrize("mode", [0, 1])
def test_records_of_almost_flat_curves(contexts, n, eps, mode):
    """Tables of one quantile function whose columns differ by eps: the lags'
    objectives lie within the roundings of sums that are 1 / eps^2 larger."""
    import torch
    from paper_2503_13756_amd import api

    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    base = torch.linspace(-0.9, 0.9, n, device="cuda")[:, None]
    noise = torch.randn(500, n, n, generator=gen, device="cuda")
    q = (base + eps * noise.sort(dim=1).values).contiguous()
    d = q.double()
    th = 2 * np.pi * torch.arange(n, device="cuda", dtype=torch.float64) / n
    m = d.mean(1)
    a = torch.stack([torch.ones(500, dtype=torch.float64, device="cuda"), (d * d).sum((1, 2)),
                     (m * th.cos()).mean(1), -(m * th.sin()).mean(1)], 1).contiguous()
    res = [api.align_batch(ctx, q[:200].contiguous(), a[:200].contiguous(), q[200:].contiguous(),
                           a[200:].contiguous(), n, mode=mode, prec=1, top_k=4)[0]
           for ctx in contexts]
    assert torch.equal(res[0], res[1])


@pytest.mark.parametrize("n,count", [(64, 2026), (32, 2636)])
def test_scratch_between_the_two_needs(contexts, n, count):
    """The counts at which the no-alloc scratch holds what rescoring every
    candidate needs and not the norms besides lie where they were: one call
    more of either set fails."""
    import torch
    from paper_2503_13756_amd import api

    ctx = contexts[0]
    q, a = api.tables(ctx, images(n, count + 8, n), n, n)
    limit = 64 << 20
    spectra = 4 * (n // 2 + 1) * n  # bytes of a table
    need = 2 * spectra * count + 2 * 4 * count * count
    assert need <= limit < need + 2 * 24 * count

    def call(m):
        return api.align_batch(ctx, q[:m].contiguous(), a[:m].contiguous(), q[:m].clone(),
                               a[:m].clone(), n, prec=1, noalloc=True)[0]

    every, _ = api.align_batch(contexts[1], q[:count].contiguous(), a[:count].contiguous(),
                               q[:count].clone(), a[:count].clone(), n, prec=1)
    assert torch.equal(call(count), every)
    most = max(m for m in range(count, count + 9)
               if 2 * spectra * m + 2 * 4 * m * m <= limit)
    with pytest.raises(RuntimeError):
        call(most + 1)
