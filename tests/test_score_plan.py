"""The score passes' plan on the host: the allocation-free entry point takes
every problem that the largest key blocks let fit its scratch memory."""
import ctypes

import pytest

import paper_2607_22586_amd.binding as bd

# B, Hq, Hkv, T, d, P, G: problems whose partials fit with 1024-key blocks
# and would not with 256-key ones, then one of every size class that does not
# depend on the block size
SHAPES = [(16, 32, 8, 4148, 128, 1024, 32), (1, 56, 8, 132144, 64, 256, 16), (16, 96, 8, 1298, 64, 512, 16),
          (2, 256, 32, 2558, 64, 1024, 32), (16, 192, 16, 550, 64, 512, 32), (8, 28, 4, 33578, 128, 256, 16),
          (1, 128, 8, 167073, 128, 128, 8), (4, 28, 4, 16384, 128, 512, 32), (1, 28, 4, 4096, 128, 512, 32)]


@pytest.fixture(scope="module")
def lib():
    return bd.load_library()


def _up(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("B,Hq,Hkv,T,d,P,G", SHAPES)
def test_workspace_stays_within_the_scratch_where_large_blocks_fit(lib, B, Hq, Hkv, T, d, P, G):
    shape = bd._shape(B, Hq, Hkv, T, 64, d)
    params = bd.SelectionConfig(P=P, G=G).c_params()
    need = lib.mmshiftkv_score_workspace(ctypes.byref(shape), ctypes.byref(params))
    Gh = Hq // Hkv
    rows = Gh * P + 32 * ((Gh + 31) // 32)
    least = _up(B * Hkv * ((T + 1023) // 1024) * rows * 8) + _up(B * Hkv * rows * 4)
    assert least <= need
    if least <= bd.NOALLOC_SCRATCH_BYTES:
        assert need <= bd.NOALLOC_SCRATCH_BYTES
