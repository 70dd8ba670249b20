"""CPU model of the two halves of a line pair in the path pass.

In its first half a wave keeps one step of every chunk of K steps, the chunk's
first; in its second half it reads the partner's kept steps and completes the
pixels that the partner walked first.  For every length: chunks of both waves
cover the same pixels, the two second halves complete every pixel of the line
exactly once, and every kept step that is read was stored before the barrier.
"""
import pytest

from test_path_schedule import schedule


@pytest.mark.parametrize("K", [8, 16])
def test_second_halves_complete_every_pixel_once(K):
    for n in range(1, 6 * K + 2):
        T, delta, split_fwd, split_rev = schedule(n, K)
        assert T % K == 0 and 0 <= delta < K and T == n + delta
        assert split_fwd % K == 0 and split_rev % K == 0 and split_fwd + split_rev == T
        done = [0] * n
        # position of a wave's step s along the forward line, and the split
        for position, first, partner_first in ((lambda s: s, split_fwd, split_rev),
                                               (lambda s: T - 1 - s, split_rev, split_fwd)):
            for c in range(first, T, K):
                kept = T - 1 - (c + K - 1)             # the partner's step at the chunk's last pixel
                assert kept % K == 0 and kept < partner_first
                for s in range(c, c + K):
                    if position(s) < n:
                        done[position(s)] += 1
        assert done == [1] * n, (n, K, done)
