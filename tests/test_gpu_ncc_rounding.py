"""The NCC cost where its quick form and its definition could round apart:
bit-exact against the oracle on textured, two-level, nearly flat and saturated
images, at run and tile edges of the kernel and every residue of D mod 4."""
import numpy as np
import pytest

from paper_2106_07927_amd import datagen

pytestmark = pytest.mark.gpu


def images(kind, w, h, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    if kind == "texture":
        p = datagen.make_pair(w, h, 32, seed)
        return p["left"], p["right"]
    if kind == "two levels":
        return tuple((rng.integers(0, 2, (h, w)) * 255).astype(np.uint8) for _ in range(2))
    if kind == "nearly flat":
        return tuple((100 + (rng.random((h, w)) < 0.02)).astype(np.uint8) for _ in range(2))
    a = rng.integers(0, 256, (h, w)).astype(np.uint8)          # one gain and offset of the other
    return a, np.clip(a.astype(int) // 2 + 60, 0, 255).astype(np.uint8)


@pytest.mark.parametrize("win", [5, 9])
@pytest.mark.parametrize("kind", ["texture", "two levels", "nearly flat", "scaled"])
def test_ncc_cost_is_the_definition(kind, win):
    import torch

    import oracle
    from paper_2106_07927_amd import sgm
    for w, h, nd in ((1, 1, 4), (127, 3, 13), (128, 4, 64), (129, 2, 130), (300, 12, 128), (260, 5, 255), (520, 9, 3)):
        print("ncc", kind, win, w, h, nd, flush=True)
        a, b = images(kind, w, h, w + nd)
        got = sgm.sgm_cost_ncc(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), win, nd)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(got.cpu().numpy(), oracle.ncc_cost(a, b, win, nd))
