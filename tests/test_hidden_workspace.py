"""Workspace of the hidden-state statistics on the host: the bytes for the
largest problem serve every smaller one, and hold its partial sums."""
import ctypes
import random

import pytest

import paper_2607_22586_amd.binding as bd


def _need(B, T, D):
    return bd.load_library().mmshiftkv_hidden_stats_workspace(ctypes.byref(bd.HShape(B, T, D)))


@pytest.mark.parametrize("D", [8, 512, 520, 2048, 3584, 8192])
def test_workspace_never_falls(D):
    rng = random.Random(D)
    lengths = sorted({1, 32, 33, 4096, 16384, 18000, 37376, 37888} | {int(2 ** rng.uniform(0, 20)) for _ in range(400)})
    for B in (1, 3, 4):
        sizes = [_need(B, T, D) for T in lengths]
        assert sizes == sorted(sizes)
    for T in lengths[::25]:
        sizes = [_need(B, T, D) for B in range(1, 40)]
        assert sizes == sorted(sizes)
        sizes = [_need(2, T, d) for d in range(8, 9000, 256)]
        assert sizes == sorted(sizes)


def test_workspace_holds_the_partial_sums():
    """(sum, sum of squares) in fp64 per batch row, feature and chunk, with
    chunks of 256 tokens, halved down to 32 while the chunk sums have fewer
    than 1024 waves of 512 features."""
    rng = random.Random(0)
    for _ in range(4000):
        B, T, D = rng.choice((1, 1, 2, 4, 7, 64)), int(2 ** rng.uniform(0, 20)), 8 * int(2 ** rng.uniform(0, 11))
        chunk = 256
        while chunk > 32 and B * -(-D // 512) * -(-T // chunk) < 1024:
            chunk //= 2
        assert _need(B, T, D) >= B * D * -(-T // chunk) * 16
