"""The path pass keeps one step per chunk of the first half and walks the
partner's steps again from it.

CPU model: for every line kind, length and chunk length, each wave's second
half recomputes the partner's values of a chunk from the step stored at the
chunk's last pixel, with zeros outside the line and restarts where a diagonal
wraps; they must equal the partner's own walk.  GPU: S_bar at lengths around
the chunk and lane-group edges, all of P2's slice widths, against the oracle.
Integers throughout: no tolerance.
"""
import numpy as np
import pytest

from paper_2106_07927_amd import datagen

DIRS = [(1, 0), (0, 1), (1, 1), (-1, 1)]


def step(L, c, p1, p2):
    m = L.min()
    p = np.concatenate(([1 << 30], L, [1 << 30]))
    V = np.minimum(np.minimum(L, np.minimum(p[:-2], p[2:]) + p1), m + p2)
    return V - m, V + c                               # A, next state (any offset)


def pixels(q, W, H, line, sign):
    """Pixels of the line in walking order and where the recursion restarts."""
    dx, dy = DIRS[q]
    if q == 0:
        seq = [(x, line) for x in range(W)]
    elif q == 1:
        seq = [(line, y) for y in range(H)]
    else:
        seq = [((line + dx * y) % W, y) for y in range(H)]
    seq = seq if sign > 0 else seq[::-1]
    fresh = [i == 0 or seq[i][0] - seq[i - 1][0] != sign * dx for i in range(len(seq))]
    return seq, fresh


@pytest.mark.parametrize("K", [8, 16])
@pytest.mark.parametrize("W,H", [(1, 1), (7, 9), (8, 16), (17, 8), (16, 33), (3, 40), (41, 2)])
def test_partner_steps_from_checkpoints(W, H, K):
    D, p1, p2 = 5, 3, 11
    C = datagen.random_cost(W, H, D, seed=W * 100 + H).astype(np.int64)
    for q in range(4):
        for line in range(H if q == 0 else W):
            n = W if q == 0 else H
            T = n + (K - n % K) % K
            delta = T - n
            split = K * (T // (2 * K))
            A = {}                                     # position (forward order) -> A, per direction
            for sign in (1, -1):
                seq, fresh = pixels(q, W, H, line, sign)
                L = np.zeros(D, np.int64)
                for i, (x, y) in enumerate(seq):
                    if fresh[i]:
                        L = np.zeros(D, np.int64)
                    a, L = step(L, C[y, x], p1, p2)
                    A[sign, i if sign > 0 else n - 1 - i] = a
            for sign, first in ((1, split // K), (-1, (T - split) // K)):
                # positions of the wave's step s: s (forward) or T - 1 - s (reverse)
                for c in range(first, T // K):
                    pos = [s if sign > 0 else T - 1 - s for s in range(c * K, c * K + K)]
                    stored = [k for k in range(0, split if sign < 0 else T - split, K)]
                    last = pos[-1]                     # the partner's first step of the chunk
                    partner_step = last if sign < 0 else T - 1 - last
                    assert partner_step in stored      # it was stored before the barrier
                    cost = lambda p: C[xy(p)[1], xy(p)[0]] if p < n else np.zeros(D, np.int64)  # noqa: E731
                    seq, _ = pixels(q, W, H, line, 1)
                    xy = lambda p: seq[p]              # noqa: E731
                    a = A[-sign, last] if last < n else np.zeros(D, np.int64)
                    P = a + cost(last)
                    for p, before in zip(pos[-2::-1], pos[:0:-1]):
                        if p < n and before < n and abs(seq[p][0] - seq[before][0]) != abs(DIRS[q][0]):
                            P = np.zeros(D, np.int64)  # the line wraps between the two
                        elif p < n and before < n and DIRS[q][0] and \
                                seq[before][0] - seq[p][0] != DIRS[q][0] * (before - p):
                            P = np.zeros(D, np.int64)
                        a, P = step(P, cost(p), p1, p2)
                        if p < n:
                            np.testing.assert_array_equal(a, A[-sign, p], err_msg=f"{q} {line} {sign} {p}")
            assert delta == T - n


@pytest.mark.gpu
@pytest.mark.parametrize("w,h,nd,npaths,p1,p2", [
    (16, 8, 64, 8, 10, 120), (15, 7, 64, 8, 10, 127), (17, 9, 64, 8, 10, 128), (33, 17, 64, 4, 7, 86),
    (32, 16, 128, 8, 10, 120), (31, 24, 100, 8, 90, 880), (49, 25, 128, 8, 10, 7936),
    (2, 70, 256, 8, 10, 120), (70, 2, 256, 8, 10, 127), (65, 33, 250, 8, 3000, 7936),
    (48, 40, 203, 4, 16128, 16128), (5, 64, 16, 8, 10, 120), (64, 5, 1, 8, 0, 120), (1200, 40, 128, 8, 10, 120),
    (700, 700, 128, 4, 10, 120), (1000, 500, 64, 8, 10, 120), (600, 700, 192, 8, 10, 120),
])
def test_aggregate_at_chunk_edges(w, h, nd, npaths, p1, p2):
    import torch

    import oracle
    from paper_2106_07927_amd import sgm
    print("aggregate", w, h, nd, npaths, p1, p2, flush=True)
    c = datagen.random_cost(w, h, nd, seed=w + h, high=256)
    got = sgm.sgm_aggregate(torch.from_numpy(c).cuda(), npaths, p1, p2)
    torch.cuda.synchronize()
    if w * h * nd > 4_000_000:                         # per-pixel line recursions of the oracle
        g = got.cpu().numpy()
        for x, y in ((0, 0), (w - 1, h - 1), (w // 2, h // 2), (w - 1, 0), (7, h - 9), (w - 17, 8)):
            np.testing.assert_array_equal(g[y, x], oracle.aggregate_at(c, npaths, p1, p2, x, y))
    else:
        np.testing.assert_array_equal(got.cpu().numpy(), oracle.aggregate(c, npaths, p1, p2))


@pytest.mark.gpu
@pytest.mark.parametrize("nd", [1, 3, 5, 7, 9, 11, 15, 17, 23, 31, 33, 41, 63, 65, 66, 97, 100, 101, 102, 103, 127, 129,
                                130, 131, 136, 203, 255])
def test_aggregate_where_d_cuts_a_lane(nd):
    """The lane that holds d = D - 1 stores in parts, the volume's last pixel
    is loaded byte by byte; nothing past a slice or a pixel is touched."""
    import torch

    import oracle
    from paper_2106_07927_amd import sgm
    print("aggregate, D =", nd, flush=True)
    for w, h in ((1, 1), (9, 17), (33, 6)):
        c = datagen.random_cost(w, h, nd, seed=nd, high=256)
        for npaths, p1, p2 in ((8, 10, 120), (8, 90, 880)):
            need = sgm.aggregate_work_bytes(w, h, nd, npaths, p2)
            work = torch.full((need + 256,), 0xA5, dtype=torch.uint8, device="cuda")
            got = sgm.sgm_aggregate(torch.from_numpy(c).cuda(), npaths, p1, p2, work=work[:need])
            torch.cuda.synchronize()
            np.testing.assert_array_equal(got.cpu().numpy(), oracle.aggregate(c, npaths, p1, p2))
            assert bool((work[need:] == 0xA5).all())
