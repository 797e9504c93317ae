"""Score passes whose key blocks are shared by several workgroups (row parts)
and blocks that straddle T, against fp64 softmax sums in plain torch.

The sizes sit on the edges of the key sub-tiles (32), waves (64, 128) and
blocks (256, 512, 1024), and on group sizes whose proxy blocks can and cannot
be split (16, 32, 48 and 64 proxies per group)."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = [
    # B, Hq, Hkv, T, d, P, G, dtype
    (1, 4, 1, 1, 64, 64, 4, "bf16"),
    (1, 4, 1, 31, 64, 64, 2, "f32"),
    (1, 7, 1, 33, 128, 512, 32, "bf16"),
    (1, 7, 1, 255, 128, 512, 32, "bf16"),
    (2, 2, 2, 257, 64, 96, 2, "bf16"),          # 48 per group
    (1, 7, 1, 300, 128, 768, 16, "bf16"),       # 48 per group, split in units of two groups
    (1, 8, 1, 545, 128, 192, 4, "f32"),
    (1, 7, 1, 1024, 128, 512, 32, "bf16"),      # full blocks, 15 and 16 parts
    (1, 12, 2, 1027, 128, 512, 8, "bf16"),      # 64 per group
    (4, 32, 32, 300, 64, 64, 4, "bf16"),        # two tiles a head: hardly anything to split
    (1, 28, 4, 4095, 128, 512, 32, "bf16"),     # 8 and 4 parts
    (1, 28, 4, 5000, 128, 512, 32, "f32"),      # 8-wave mass blocks with parts
    (1, 16, 2, 8000, 64, 512, 32, "bf16"),      # the same at d = 64
    (1, 28, 4, 12000, 128, 512, 32, "bf16"),    # 8-wave blocks with parts and early phases in both passes
    (1, 28, 4, 16001, 128, 512, 32, "bf16"),    # the same with a ragged last block
    (16, 28, 4, 4001, 128, 512, 32, "bf16"),    # 1024-key blocks, the last one ragged
    (16, 28, 4, 4064, 128, 64, 4, "bf16"),      # the same with a last sub-tile that is full
]


def _reference(proxies, q_last, k, G):
    B, Hq, P, d = proxies.shape
    Hkv, T = k.shape[1], k.shape[2]
    Gh = Hq // Hkv
    keys = k.bfloat16().double()
    anc = (q_last.double() * (math.log2(math.e) / math.sqrt(d))).float().bfloat16().double()
    gm = torch.zeros((B, Hkv, G, T), dtype=torch.float64, device=k.device)
    an = torch.zeros((B, Hkv, T), dtype=torch.float64, device=k.device)
    for b in range(B):
        for h in range(Hq):
            kt = keys[b, h // Gh].t().contiguous()
            p = torch.softmax((proxies[b, h].double() @ kt) * math.log(2.0), dim=-1)
            gm[b, h // Gh] += p.reshape(G, P // G, T).sum(1)
            an[b, h // Gh] += torch.softmax((anc[b, h] @ kt) * math.log(2.0), dim=-1) / Gh
    return gm, gm.sum(2), an


@pytest.mark.parametrize("B,Hq,Hkv,T,d,P,G,dtype", SIZES)
def test_parts_and_ragged_blocks(B, Hq, Hkv, T, d, P, G, dtype):
    import paper_2607_22586_amd as mm
    from paper_2607_22586_amd import workloads as wl
    print("score parts", B, Hq, Hkv, T, d, P, G, dtype, flush=True)
    x = wl.custom_layer(B, Hq, Hkv, T, 8, d, dtype, seed=T, device="cuda:0")
    cfg = mm.SelectionConfig(P=P, G=G, gamma=3.0, seed=1)
    prox, ql = mm.build_proxies(x["q_win"], cfg, T, Hkv)
    a, b = (mm.score(prox, ql, x["k"], cfg, 8) for _ in range(2))
    for want, got, again in zip(_reference(prox, ql, x["k"], G), (a.group_mass, a.mass, a.anchor),
                                (b.group_mass, b.mass, b.anchor)):
        assert torch.equal(got, again)           # no order depends on timing
        # fp32 logits of up to ~60 (d products, each rounded at 2^-24) move a
        # probability by < 60 * d * 2^-24 = 5e-4 in the worst case; sums of up
        # to 1024 fp32 terms add 6e-5
        err = (got.double() - want).abs()
        assert bool((err <= 6e-4 * want + 1e-30).all()), float((err / (want + 1e-30)).max())


@pytest.mark.parametrize("B,Hq,Hkv,T,d,P,G", [(1, 7, 1, 1024, 128, 512, 32), (1, 28, 4, 4095, 128, 512, 32),
                                              (1, 4, 1, 700, 64, 512, 32)])
def test_merge_again_after_a_mass_pass(B, Hq, Hkv, T, d, P, G):
    """The mass pass leaves the other stages' results in the workspace: the
    merge and a second mass pass after it give the first one's bits."""
    import paper_2607_22586_amd as mm
    from paper_2607_22586_amd import workloads as wl
    print("merge again", B, Hq, Hkv, T, d, P, G, flush=True)
    x = wl.custom_layer(B, Hq, Hkv, T, 8, d, "bf16", seed=T, device="cuda:0")
    cfg = mm.SelectionConfig(P=P, G=G, gamma=3.0, seed=1)
    prox, ql = mm.build_proxies(x["q_win"], cfg, T, Hkv)
    ws = torch.empty(mm.score_workspace(B, Hq, Hkv, T, 8, d, cfg), dtype=torch.uint8, device="cuda:0")
    mm.score_lse(prox, ql, x["k"], cfg, ws, 8)
    first = mm.score_mass(prox, ql, x["k"], cfg, ws, 8)
    mm.score_lse(prox, ql, x["k"], cfg, ws, 8, stage="merge")
    again = mm.score_mass(prox, ql, x["k"], cfg, ws, 8)
    for a, b in ((first.group_mass, again.group_mass), (first.mass, again.mass), (first.anchor, again.anchor)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("B,Hq,Hkv,T,d,P,G,dtype", [
    (1, 7, 1, 255, 128, 512, 32, "bf16"), (2, 28, 4, 1000, 128, 512, 32, "f32"), (1, 28, 4, 4095, 128, 512, 32, "bf16"),
    (1, 32, 32, 777, 128, 512, 32, "bf16"), (1, 16, 2, 3000, 64, 64, 4, "f32"), (2, 8, 2, 12001, 64, 512, 32, "bf16")])
def test_strides_do_not_change_the_bits(B, Hq, Hkv, T, d, P, G, dtype):
    """Token-major and padded caches give the contiguous head-major result's
    bits (which the test above holds to fp64)."""
    import paper_2607_22586_amd as mm
    from paper_2607_22586_amd import workloads as wl
    print("strides", B, Hq, Hkv, T, d, P, G, dtype, flush=True)
    x = wl.custom_layer(B, Hq, Hkv, T, 8, d, dtype, seed=T, device="cuda:0")
    cfg = mm.SelectionConfig(P=P, G=G, gamma=3.0, seed=1)
    prox, ql = mm.build_proxies(x["q_win"], cfg, T, Hkv)
    k = x["k"]
    want = mm.score(prox, ql, k, cfg, 8)
    tokens = k.transpose(1, 2).contiguous().transpose(1, 2)
    slack = torch.full((B, Hkv, T + 3, d + 16), float("nan"), dtype=k.dtype, device=k.device)
    slack[:, :, :T, :d] = k
    for view in (tokens, slack[:, :, :T, :d]):
        got = mm.score(prox, ql, view, cfg, 8)
        for a, b in ((want.group_mass, got.group_mass), (want.mass, got.mass), (want.anchor, got.anchor)):
            assert torch.equal(a, b)
