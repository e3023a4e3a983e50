"""Calls on few images or references, whose work is split over more blocks:
the splits never change a bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2503_13756_amd import api as A

    return A


def dev(x):
    import torch

    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# the packed rows per block of the reference spectra: one (Q/2 <= 512 / refs),
# several, with a ragged last block, all of them; n = 128 writes coefficients
@pytest.mark.parametrize("L,n,Q", [(24, 24, 20), (40, 48, 52), (32, 128, 36), (64, 256, 8)])
@pytest.mark.parametrize("refs", [1, 37, 130, 520])
def test_reference_spectra_row_split(api, L, n, Q, refs):
    _, imgs = synth.make_raw_stack(31 + L, L, 6)
    ctx = api.Context(0)
    q, a = api.tables(ctx, dev(imgs), n, Q)
    rep = (refs + 5) // 6
    rq = q.repeat(rep, 1, 1)[:refs].contiguous()
    ra = a.repeat(rep, 1)[:refs].contiguous()
    res, curve = api.align_batch(ctx, rq, ra, q[:2].contiguous(), a[:2].contiguous(), L,
                                 want_curve=True)
    res, curve = res.cpu().numpy(), curve.cpu().numpy()
    for r in range(min(6, refs)):
        one, c1 = api.align_batch(ctx, rq[r:r + 1].contiguous(), ra[r:r + 1].contiguous(),
                                  q[:2].contiguous(), a[:2].contiguous(), L, want_curve=True)
        for k in range(r, refs, 6):
            assert np.array_equal(res[2 * k:2 * k + 2], one.cpu().numpy()), (r, k)
            assert np.array_equal(curve[2 * k:2 * k + 2], c1.cpu().numpy()), (r, k)
    ctx.close()


# images per launch: one, several, one below and at the default small-batch
# limit of a 256-unit device; sides with one strip, with several, at the edges
# of the staging; columns by half waves (L <= 128) and by whole waves; (150,
# 192, 108) and (255, 512, 8): two images per 1024-thread block, fused and in
# several task groups
@pytest.mark.parametrize("L,n,Q", [(8, 8, 8), (39, 48, 48), (97, 24, 20), (128, 128, 128),
                                   (129, 96, 60), (256, 72, 256), (150, 192, 108),
                                   (255, 512, 8)])
@pytest.mark.parametrize("N", [1, 5, 255])
def test_small_batches_equal_large_ones(api, tmp_path, L, n, Q, N):
    """The launches of a small batch (several blocks per image) against those of
    a large one (one or two images per block): tables and aux, plain and
    ramp-filtered, bit for bit, with a NaN image, an empty one and an infinite
    pixel among them."""
    paths = {}
    for name, lim in (("small", 1 << 30), ("large", 0)):
        paths[name] = tmp_path / f"{name}.json"
        paths[name].write_text('{"small_batch": %d}' % lim)
    _, imgs = synth.make_raw_stack(77 + L, L, min(N, 5))
    imgs = np.concatenate([imgs] * ((N + 4) // 5))[:N].copy()
    if N >= 5:
        imgs[1, L // 2, L // 2] = np.nan
        imgs[2] = 0.0
        imgs[3, L // 2, L // 3] = np.inf
    x = dev(imgs)
    for ramp in (False, True):
        out = {}
        for name, p in paths.items():
            ctx = api.Context(0, tune_json=str(p))
            q, a = api.tables(ctx, x, n, Q, ramp=ramp)
            out[name] = (q.cpu().numpy().view(np.uint32), a.cpu().numpy().view(np.uint64))
            ctx.close()
        assert np.array_equal(out["small"][0], out["large"][0]), ramp
        assert np.array_equal(out["small"][1], out["large"][1]), ramp


# references per block of the FFT alignment: one (few pairs), runs of two to
# eight with an uneven last run; n = 512 never shares; bf16 rescores four lags
# of each reference, in batches of eight candidates
@pytest.mark.parametrize("L,n,Q,refs,images", [(16, 16, 12, 3, 700), (39, 48, 48, 9, 300),
                                               (24, 24, 20, 8, 1200), (40, 96, 44, 11, 200),
                                               (64, 256, 24, 5, 500), (24, 512, 8, 4, 600)])
@pytest.mark.parametrize("prec", [0, 1])
def test_references_sharing_a_block(api, oracle, L, n, Q, refs, images, prec):
    """All pairs of `refs` references and `images` images, whose blocks share an
    image's transforms between references, against the listed pairs, one per
    block, bit for bit (an empty image and a NaN reference among them), and
    against the oracle on a sample."""
    import torch
    from tests import parity

    _, imgs = synth.make_raw_stack(900 + L, L, 12)
    imgs[5] = 0.0
    imgs[1, L // 2, L // 2] = np.nan
    ctx = api.Context(0)
    q, a = api.tables(ctx, dev(imgs), n, Q)
    ri = [k % 5 for k in range(refs)]  # references: tables 0..4
    gi = [4 + k % 8 for k in range(images)]
    rq, ra, iq, ia = (x[torch.tensor(k, device="cuda")].contiguous()
                      for x, k in ((q, ri), (a, ri), (q, gi), (a, gi)))
    res, curve = api.align_batch(ctx, rq, ra, iq, ia, L, prec=prec, want_curve=True)
    pairs = np.array([(r, g) for r in range(refs) for g in range(images)], np.int64)
    one, c1 = api.align_batch(ctx, rq, ra, iq, ia, L, prec=prec, want_curve=True, pairs=dev(pairs))
    assert np.array_equal(res.cpu().numpy(), one.cpu().numpy())
    assert np.array_equal(curve.cpu().numpy().view(np.uint32), c1.cpu().numpy().view(np.uint32))
    s = np.r_[0:8, images:images + 8]
    ok = [p for p in s if ri[p // images] != 1 and gi[p % images] != 5]
    o = oracle.align(rq.cpu().numpy(), ra.cpu().numpy(), iq.cpu().numpy(), ia.cpu().numpy(), L,
                     pairs=pairs[ok], want_curve=True)
    g = api.unpack_results(res[torch.tensor(ok, device="cuda")])
    parity.check(g, o, L, parity.TAU_BF16 if prec else parity.TAU_FP32, o["curve"])
    ctx.close()


# 2,026 and 2,636: the most tables whose spectra and candidates fit the no-alloc
# scratch while the norms that prune candidates do not
@pytest.mark.parametrize("n,count", [(64, 2026), (32, 2636)])
@pytest.mark.parametrize("mode", [0, 1])
def test_pruned_candidates_never_win(api, n, count, mode):
    """All pairs with the candidates that cannot win pruned (the norms fit the
    call's scratch) against the same pairs with every candidate rescored (the
    no-alloc scratch has no room for the norms): the same records.  The images
    hold clean and noisy blobs, noise, nearly symmetric images whose curves are
    almost flat, copies, an empty image and a NaN."""
    import torch

    L = n
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5 + n)
    ax = (torch.arange(L, device="cuda") - (L - 1) / 2) * (2.0 / L)
    k = 6

    def blobs(m):
        c = 1.2 * torch.rand(m, k, 2, generator=gen, device="cuda") - 0.6
        gx = torch.exp(-((ax - c[..., :1]) ** 2) / 0.02)
        gy = torch.exp(-((ax - c[..., 1:]) ** 2) / 0.02)
        return torch.bmm(gy.transpose(1, 2).contiguous(), gx.contiguous())

    x = torch.cat([blobs(count // 2), torch.rand(count // 4, L, L, generator=gen, device="cuda")])
    disc = torch.exp(-(ax[:, None] ** 2 + ax[None, :] ** 2) / 0.1)
    rest = count - x.shape[0]
    x = torch.cat([x, disc + 1e-4 * torch.rand(rest, L, L, generator=gen, device="cuda")])
    x += 0.3 * torch.rand(count, 1, 1, generator=gen, device="cuda") * torch.rand(
        x.shape, generator=gen, device="cuda") * (torch.arange(count, device="cuda") % 2)[:, None, None]
    x[7] = 0.0
    x[11, L // 2, L // 2] = float("nan")
    x[13] = disc
    x[17] = x[3]
    y = x[torch.randperm(count, generator=gen, device="cuda")].contiguous()
    ctx = api.Context(0)
    q, a = api.tables(ctx, x.contiguous(), n, n)
    p, b = api.tables(ctx, y, n, n)
    pruned, _ = api.align_batch(ctx, q, a, p, b, L, mode=mode, prec=1)
    every, _ = api.align_batch(ctx, q, a, p, b, L, mode=mode, prec=1, noalloc=True)
    assert torch.equal(pruned, every)
    ctx.close()


# Fourier slices: a single round of columns with its slot in LDS (L <= 36; the
# slot in scratch at n = 512), several rounds with the last one short or taking
# column L along (L <= 64), a step of its own for column L; explicit angles
@pytest.mark.parametrize("L,n", [(8, 8), (12, 16), (16, 512), (32, 32), (36, 512), (36, 32),
                                 (48, 24), (54, 48), (72, 72), (108, 64), (128, 24), (162, 48),
                                 (256, 128)])
@pytest.mark.parametrize("theta", [False, True])
def test_fourier_rounds(api, oracle, tmp_path, L, n, theta):
    """The phases of an image over several blocks against one block per image
    bit for bit, and both against the oracle at the projector's tolerance
    (5e-6 of the largest value), with a NaN image among them."""
    _, imgs = synth.make_raw_stack(55 + L, L, 4)
    ang = synth.mc_angles(n, 3) if theta else None
    imgs[2, L // 2, L // 2] = np.nan
    x = dev(imgs)
    out = {}
    for name, lim in (("split", 1 << 30), ("whole", 0)):
        path = tmp_path / f"{name}.json"
        path.write_text('{"small_batch": %d}' % lim)
        ctx = api.Context(0, str(path))
        out[name] = api.project_fourier(ctx, x, n, theta=ang).cpu().numpy()
        ctx.close()
    assert np.array_equal(out["split"], out["whole"], equal_nan=True)
    got = out["split"]
    assert np.isnan(got[2]).all()
    keep = [0, 1, 3]
    P0 = np.maximum(oracle.fourier_project(imgs[keep], n, angles=ang)[0], 0.0)
    err = np.abs(got[keep] - P0).max(axis=(1, 2)) / P0.max(axis=(1, 2))
    assert err.max() < 5e-6, err
