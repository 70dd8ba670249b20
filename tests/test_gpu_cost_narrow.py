"""Cost volumes of images narrower than a block's run of 128 pixels, whose runs
per thread depend on the width: every run length, D a multiple of 4 and not,
bit-exact against the oracle; bytes past the volume stay."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nd", [4, 13, 21, 64, 101, 128, 250, 256])
@pytest.mark.parametrize("w", [2, 4, 9, 16, 17, 33, 65, 85, 100, 126])
def test_cost_narrow(w, nd):
    import torch

    import oracle
    from paper_2106_07927_amd import datagen, sgm
    print("cost", w, nd, flush=True)
    h = 5
    a, b = datagen.random_images(w, h, nd + w)
    cl, cr = oracle.census(a, 9, 7), oracle.census(b, 9, 7)
    dev = [torch.from_numpy(c.view(np.int64)).cuda().view(torch.uint64) for c in (cl, cr)]
    n = w * h * nd
    guarded = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    sgm.sgm_cost(*dev, nd, out=guarded[:n].view(h, w, nd))
    torch.cuda.synchronize()
    got = guarded.cpu().numpy()
    np.testing.assert_array_equal(got[:n].reshape(h, w, nd), oracle.cost(cl, cr, nd))
    assert (got[n:] == 0xA5).all()
