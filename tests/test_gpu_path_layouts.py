"""Every lane layout of the path pass gives the oracle's disparities: each
variant of each range of D, at whole, padded and cut lanes (D = 1 mod 2, 4, 8,
16 and multiples), one- and two-byte slices, as a work list of small frames
and as single frames.  Integers throughout: no tolerance."""
import json

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NDISP = [9, 13, 16, 17, 24, 32, 33, 40, 48, 50, 64, 65, 80, 100, 128, 129, 200, 208, 256]


@pytest.mark.parametrize("p1,p2,npaths", [(10, 120, 8), (90, 880, 8), (10, 120, 4), (7936, 7936, 8),
                                           (7937, 7937, 4)])
@pytest.mark.parametrize("nd", NDISP)
def test_every_variant_is_exact(nd, p1, p2, npaths):
    import torch

    import oracle
    from paper_2106_07927_amd import datagen, sgm
    prm = sgm.Params(ndisp=0, win_w=9, win_h=7, npaths=npaths, p1=p1, p2=p2, lr_tolerance=-1, median3x3=False)
    # the last one is large enough for kernels of its own
    shapes = [(61, 43), (34, 90), (400, 251)]
    pairs = [datagen.random_images(w, h, 7 * nd + i) for i, (w, h) in enumerate(shapes)]
    want = [oracle.run_threaded(a, b, oracle.Params(ndisp=nd, win_w=9, win_h=7, npaths=npaths, p1=p1, p2=p2,
                                                    lr_tolerance=-1, median3x3=False), 8) for a, b in pairs]
    lefts = [torch.from_numpy(a).cuda() for a, _ in pairs]
    rights = [torch.from_numpy(b).cuda() for _, b in pairs]
    n = sgm.load_library().sgm_aggregate_variants(nd)
    for v in [None] + list(range(n)):
        print("layout", nd, p2, npaths, v, flush=True)
        table = json.dumps({} if v is None else {f"{w}x{h}x{nd}": v for w, h in shapes})
        plan = sgm.BatchPlan(lefts, rights, [nd] * len(shapes), prm, tune_table=table, want_right=True)
        plan.run()
        torch.cuda.synchronize()
        for i, w in enumerate(want):
            np.testing.assert_array_equal(plan.disp[i].cpu().numpy(), w["disp"], err_msg=f"{shapes[i]} variant {v}")
            np.testing.assert_array_equal(plan.disp_right[i].cpu().numpy(), w["disp_right"])
        plan.close()


@pytest.mark.parametrize("p1,p2,npaths", [(127, 128, 8), (3000, 7936, 8), (7936, 7936, 8), (7936, 7936, 4), (1, 7937, 4),
                                          (16128, 16128, 4)])
@pytest.mark.parametrize("nd", [3, 13, 16, 30, 64, 100, 128, 200, 256])
def test_large_penalties(nd, p1, p2, npaths):
    """S_bar with path states as large as they get: costs of 255 over whole
    lines, a few small ones, and P1 up to P2."""
    import torch

    import oracle
    from paper_2106_07927_amd import sgm
    for w, h in ((70, 40), (33, 50)):
        print("penalties", nd, p1, p2, npaths, w, h, flush=True)
        rng = np.random.Generator(np.random.PCG64(nd + w))
        cost = np.full((h, w, nd), 255, np.uint8)
        some = rng.random(cost.shape)
        cost[some < 0.2] = rng.integers(0, 256, int((some < 0.2).sum()))
        cost[:, : w // 2][some[:, : w // 2] >= 0.001] = 255
        got = sgm.sgm_aggregate(torch.from_numpy(cost).cuda(), npaths, p1, p2)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.view(torch.int16).cpu().numpy().view(np.uint16),
                                      oracle.aggregate(cost, npaths, p1, p2))
