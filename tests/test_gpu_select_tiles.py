"""The selection's tile pass at segment (8 / 16 pixels) and tile (32 / 64)
edges, for every class of disparity range, from pair slices of both widths and
from S_bar, with and without the subpixel output, against the oracle.  Integer
maps exactly; the refined values within 2^-15 (one float32 division of exact
integers, an offset of at most 1/2 added to d < 256: half an ulp of 2^-16 and
2^-25)."""
import numpy as np
import pytest

from paper_2106_07927_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nd", [1, 2, 3, 7, 15, 16, 17, 31, 32, 48, 63, 64, 65, 80, 100, 101, 127, 128, 129, 144, 200,
                                203, 255, 256])
def test_selection_at_tile_edges(nd):
    import torch

    import oracle
    from paper_2106_07927_amd import sgm
    print("selection, D =", nd, flush=True)
    for w, h in ((1, 1), (15, 2), (16, 3), (17, 1), (33, 2), (63, 1), (65, 3), (130, 2)):
        c = datagen.random_cost(w, h, nd, seed=nd + w, high=6)              # many ties
        dc = torch.from_numpy(c).cuda()
        for npaths, p1, p2 in ((8, 3, 20), (4, 90, 880)):
            s = oracle.aggregate(c, npaths, p1, p2)
            dl, dr = oracle.wta(s), oracle.right_disparity(s)
            d = oracle.lr_check(dl, dr, 1)
            a = sgm.sgm_aggregate_select(dc, npaths, p1, p2, 1, False, want_right=True)
            b = sgm.sgm_wta_lrc(torch.from_numpy(s).cuda(), 1, False, want_right=True)
            fine, fr = sgm.sgm_aggregate_select_subpixel(dc, npaths, p1, p2, 1, False, want_right=True)
            torch.cuda.synchronize()
            for got in (a, b):
                np.testing.assert_array_equal(got[0].cpu().numpy(), d, err_msg=f"{w}x{h} P2 {p2}")
                np.testing.assert_array_equal(got[1].cpu().numpy(), dr, err_msg=f"{w}x{h} P2 {p2}")
            np.testing.assert_array_equal(fr.cpu().numpy(), dr)
            fine = fine.cpu().numpy()
            ok = d != 0xFFFF
            np.testing.assert_array_equal(fine >= 0, ok)
            np.testing.assert_allclose(fine[ok], oracle.refine_subpixel(s, dl)[ok], rtol=0, atol=2.0 ** -15)


@pytest.mark.parametrize("nd", [33, 64, 100, 200, 256])
def test_selection_of_costs_without_a_winner(nd):
    """S_bar of one value everywhere, the largest uint16 included: d = 0."""
    import torch

    from paper_2106_07927_amd import sgm
    for v in (0, 65535):
        s = torch.full((3, 70, nd), v, dtype=torch.int32).to(torch.uint16).cuda()
        got, right = sgm.sgm_wta_lrc(s, -1, False, want_right=True)
        torch.cuda.synchronize()
        assert not got.cpu().numpy().any() and not right.cpu().numpy().any()
