"""Cost volumes of every D mod 4, bit-exact against the oracle: the smallest
ranges, both sides of the kernel's run lengths, rows that end inside and at the
end of a 128-pixel run, single calls and the work list of a batch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nd", [1, 2, 3, 5, 7, 9, 30, 33, 63, 66, 101, 127, 130, 131, 253, 254, 255])
def test_cost_ragged(nd):
    import torch

    import oracle
    from paper_2106_07927_amd import datagen, sgm
    prm = dict(ndisp=nd, win_w=9, win_h=7, npaths=4, p1=10, p2=120, lr_tolerance=-1, median3x3=False)
    pairs = []
    for w, h in ((1, 1), (5, 3), (127, 2), (128, 5), (129, 2), (500, 7)):
        print("cost", nd, w, h, flush=True)
        a, b = datagen.random_images(w, h, nd + w)
        pairs.append((a, b))
        cl, cr = oracle.census(a, 9, 7), oracle.census(b, 9, 7)
        dev = [torch.from_numpy(c.view(np.int64)).cuda().view(torch.uint64) for c in (cl, cr)]
        n = w * h * nd
        guarded = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda")      # bytes past the volume stay
        sgm.sgm_cost(*dev, nd, out=guarded[:n].view(h, w, nd))
        torch.cuda.synchronize()
        got = guarded.cpu().numpy()
        np.testing.assert_array_equal(got[:n].reshape(h, w, nd), oracle.cost(cl, cr, nd))
        assert (got[n:] == 0xA5).all()
    plan = sgm.BatchPlan([torch.from_numpy(a).cuda() for a, _ in pairs], [torch.from_numpy(b).cuda() for _, b in pairs],
                         [nd] * len(pairs), sgm.Params(**prm))
    plan.run()
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(pairs):
        np.testing.assert_array_equal(plan.disp[i].cpu().numpy(), oracle.run(a, b, oracle.Params(**prm))["disp"])
    plan.close()
