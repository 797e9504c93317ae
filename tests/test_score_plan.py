"""The score passes' plan on the host: the allocation-free entry point takes
every problem that the largest key blocks let fit its scratch memory, and the
workspace for the largest prompt serves every shorter one."""
import ctypes
import random

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


HEADS = [(28, 4, 128, 512, 32), (32, 32, 128, 512, 32), (64, 8, 128, 512, 32), (4, 1, 64, 512, 32), (16, 2, 64, 64, 4),
         (96, 16, 64, 1024, 32), (128, 8, 128, 128, 8), (7, 7, 128, 96, 2)]
FAKE = ctypes.c_void_p(0x10000)


def _need(lib, B, Hq, Hkv, T, d, P, G):
    shape, params = bd._shape(B, Hq, Hkv, T, 64, d), bd.SelectionConfig(P=P, G=G).c_params()
    return shape, params, lib.mmshiftkv_score_workspace(ctypes.byref(shape), ctypes.byref(params))


@pytest.mark.parametrize("Hq,Hkv,d,P,G", HEADS)
def test_workspace_never_falls_with_the_prompt_or_the_batch(lib, Hq, Hkv, d, P, G):
    rng = random.Random(Hq * P + d)
    lengths = sorted({1, 2, 255, 256, 257, 8192, 8256, 16384, 32767, 32768, 131072, 1 << 20} |
                     {int(2 ** rng.uniform(0, 20)) for _ in range(400)})
    for B in (1, 3, 16):
        sizes = [_need(lib, B, Hq, Hkv, T, d, P, G)[2] for T in lengths]
        assert sizes == sorted(sizes)
    for T in lengths[::20]:
        sizes = [_need(lib, B, Hq, Hkv, T, d, P, G)[2] for B in range(1, 40)]
        assert sizes == sorted(sizes)


@pytest.mark.parametrize("Hq,Hkv,d,P,G", HEADS)
def test_workspace_of_the_query_is_accepted(lib, Hq, Hkv, d, P, G):
    """The plan of every problem fits the queried bytes (the call below stops
    at the missing group masses, before any launch)."""
    rng = random.Random(Hq + P)
    for _ in range(600):
        B, T = rng.choice((1, 1, 2, 4, 16, 64)), int(2 ** rng.uniform(0, 19))
        shape, params, need = _need(lib, B, Hq, Hkv, T, d, P, G)
        for dtype in (bd.MMSKV_BF16, bd.MMSKV_F32):
            strides = bd.Strides(Hkv * T * d, T * d, d)
            call = lambda nbytes: lib.mmshiftkv_score_mass(  # noqa: E731
                ctypes.byref(shape), ctypes.byref(params), FAKE, FAKE, FAKE, dtype, ctypes.byref(strides), None, FAKE,
                FAKE, FAKE, nbytes, None)
            assert call(need) == bd.MMSKV_EINVAL
            assert call(need - 1) == bd.MMSKV_EWORKSPACE
