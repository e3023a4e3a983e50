"""FFT alignment: the rescore of more candidates than one batch holds."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


# a batch is four candidates.  All Q rows of the image table in LDS at once, so
# that no staging lies between two batches, down to fewer lags than lanes and up
# to the most; and (96, 96, 96), staged in several chunks
@pytest.mark.parametrize("L,n,Q", [(16, 16, 16), (24, 24, 20), (39, 48, 48), (64, 64, 64),
                                   (96, 96, 96), (16, 8, 8), (64, 512, 8)])
@pytest.mark.parametrize("top_k", [5, 8])
@pytest.mark.parametrize("mode", [0, 1])
def test_batches_of_candidates_agree(oracle, L, n, Q, top_k, mode):
    """Eight references a block (up to 64 candidates), one pair a block and the
    stacks' queue give the same records; one batch of candidates (top_k = 1 and
    4) gives the same objective wherever it takes the same lag and never a
    smaller one; the records agree with the oracle."""
    import torch
    from paper_2503_13756_amd import api
    from tests import parity

    _, imgs = synth.make_raw_stack(300 + L, L, 20)
    refs, count = 8, 300
    ctx = api.Context(0)
    x = torch.from_numpy(np.ascontiguousarray(imgs)).cuda()
    q, a = api.tables(ctx, x, n, Q)
    rq, ra = q[:refs].contiguous(), a[:refs].contiguous()
    at = torch.arange(count, device="cuda") % 20
    iq, ia = q[at].contiguous(), a[at].contiguous()

    def align(k, pairs=None):
        r, _ = api.align_batch(ctx, rq, ra, iq, ia, L, mode=mode, prec=0, top_k=k, pairs=pairs)
        return r

    res = align(top_k)
    pairs = torch.tensor([(r, g) for r in range(refs) for g in range(count)], device="cuda")
    assert torch.equal(res, align(top_k, pairs))
    many = api.unpack_results(res)
    for k in (1, 4):
        few = api.unpack_results(align(k))
        same = many["rot_index"] == few["rot_index"]
        assert same.mean() > 0.9
        assert np.array_equal(many["sw2sq"][same], few["sw2sq"][same])
        assert (many["sw2sq"] <= few["sw2sq"]).all()
    if n == L and Q == L:
        out = api.align_stacks(ctx, [(x[0].contiguous(), x)], mode=mode, prec=0, top_k=top_k)
        assert torch.equal(out[0]["res"], res[:20])
    s = np.r_[0:20, count:count + 20]
    o = oracle.align(rq.cpu().numpy(), ra.cpu().numpy(), iq.cpu().numpy(), ia.cpu().numpy(), L,
                     pairs=pairs.cpu().numpy()[s], mode=mode, want_curve=True)
    g = api.unpack_results(res[torch.tensor(s, device="cuda")])
    parity.check(g, o, L, parity.TAU_FP32, o["curve"])
    ctx.close()
