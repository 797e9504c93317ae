"""The top-k on scores at the limits of its first-digit buckets, against numpy:
scores of every sign."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _select(cfg, budget, mass=None, gm=None, anchor=None):
    import paper_2607_22586_amd as mm
    dev = lambda x: None if x is None else torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")  # noqa: E731
    B, Hkv, T = mass.shape
    sel = mm.select_topk(mm.ScoreOut(dev(gm), dev(mass), dev(anchor)), cfg, budget, Hq=Hkv)
    return sel.idx.cpu().numpy(), sel.counts.cpu().numpy()


def _best(score, want):
    """The `want` best by (score bits as an unsigned number desc, index asc), ascending."""
    bits = score.astype(np.float64).view(np.uint64)
    return np.sort(np.lexsort((np.arange(len(bits)), ~bits))[:want])


@pytest.mark.parametrize("T,budget,n_neg", [(1000, 200, 200), (1000, 150, 200), (1000, 260, 200), (9000, 700, 700),
                                            (9000, 5000, 4500), (40001, 300, 300), (40001, 6000, 7000)])
@pytest.mark.parametrize("low", [0.0, 1.0])
def test_every_sign_has_a_place(T, budget, n_neg, low):
    """Masses of -0 and below: min(C, T) keys are kept whatever the bits."""
    import paper_2607_22586_amd as mm
    print("signs", T, budget, n_neg, low, flush=True)
    rng = np.random.default_rng(T + n_neg)
    mass = np.zeros((1, 2, T), np.float32)
    for c in range(2):
        mass[0, c, rng.permutation(T)[:n_neg]] = -low * rng.random(n_neg) if low else -0.0
        mass[0, c, rng.permutation(T)[:10]] = rng.random(10)
    cfg = mm.SelectionConfig(mode=mm.MMSKV_MASS, keep_last=False)
    idx, counts = _select(cfg, budget, mass)
    for c in range(2):
        assert counts[0, c] == budget
        assert np.array_equal(idx[0, c], _best(mass[0, c], budget))
