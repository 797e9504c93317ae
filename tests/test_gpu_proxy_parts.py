"""Query proxies bit-exact against the oracle where a head's proxies are shared
by several workgroups and at the edges of the window staging: window rows
around the batches of 16 and the chunks of 64, head counts with one, two, four
and sixteen parts, fp32 and bf16 queries, rotary pairs, strided windows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_22586_amd import binding as bd
from paper_2607_22586_amd import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("B,Hq,d,W,P,dtype,rope,ddof", [
    (1, 1, 64, 1, 32, "bf16", False, 0), (1, 4, 64, 15, 512, "f32", False, 1), (1, 4, 64, 16, 512, "bf16", True, 0),
    (1, 28, 128, 17, 512, "bf16", False, 0), (1, 2, 128, 63, 96, "f32", True, 0), (2, 7, 128, 64, 64, "bf16", False, 1),
    (1, 3, 64, 65, 160, "bf16", False, 0), (1, 5, 128, 129, 512, "f32", True, 1), (4, 28, 128, 32, 64, "f32", False, 0)])
@pytest.mark.parametrize("strided", [False, True])
def test_proxies_bit_exact_over_parts(B, Hq, d, W, P, dtype, rope, ddof, strided):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gen = torch.Generator().manual_seed(W * 1000 + P)
    q = torch.randn((B, Hq, W, d), generator=gen) + 2.0 * torch.randn((B, Hq, 1, d), generator=gen)
    q = q if dtype == "f32" else q.bfloat16()
    cfg = bd.SelectionConfig(P=P, G=2, seed=99, layer=3, std_ddof=ddof)
    tab = wl.rope_tables(d, 777) if rope else None
    x = q.to(DEV)
    if strided:                                  # a token-major window, one row of slack per head
        wide = torch.empty((B, W, Hq, d + 8), dtype=x.dtype, device=DEV)
        wide[..., :d] = x.transpose(1, 2)
        x = wide[..., :d].transpose(1, 2)
    prox, ql, st = bd.build_proxies(x, cfg, 100, Hq, tab, tab, with_stats=True)
    torch.cuda.synchronize()
    tn = None if tab is None else tuple(t.numpy() for t in tab)
    rp, rq, rs = oracle.build_proxies(wl.to_numpy_bits(q), P, cfg.gamma, cfg.seed, cfg.layer, ddof, tn, tn)
    assert np.array_equal(wl.to_numpy_bits(prox), rp)
    assert np.array_equal(wl.to_numpy_bits(ql), rq)
    assert np.array_equal(st.cpu().numpy(), rs)
