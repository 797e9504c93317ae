"""The top-k on scores at the limits of its first-digit buckets, against numpy:
scores of every sign, thousands of scores tied at the cut, and buckets of nearly
all keys."""
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


@pytest.mark.parametrize("T,above,tied,budget", [
    (300, 5, 200, 100), (1000, 0, 129, 128), (4096, 100, 2000, 1100), (4096, 0, 4096, 256), (4097, 1, 4096, 4000),
    (8192, 300, 4000, 2301), (16384, 20, 1500, 700), (16384, 0, 16384, 5000), (32768, 7, 4096, 8), (40001, 90, 3000, 91),
    (40001, 90, 4096, 4000), (40001, 0, 9000, 4500), (100003, 50, 2500, 2000), (524288, 9, 4000, 3000),
    (524289, 9, 4000, 3000)])
@pytest.mark.parametrize("run", [False, True])
def test_ties_at_the_cut(T, above, tied, budget, run):
    """Equal scores enter by index, spread over the row or in one run."""
    import paper_2607_22586_amd as mm
    print("ties", T, above, tied, budget, run, flush=True)
    rng = np.random.default_rng(T + tied)
    mass = (0.25 * rng.random((1, 2, T))).astype(np.float32)
    for c in range(2):
        order = rng.permutation(T) if not run else np.roll(np.arange(T), int(rng.integers(T)))
        mass[0, c, order[:tied]] = 0.5
        mass[0, c, order[tied:tied + above]] = 1.0 + rng.random(len(order[tied:tied + above]))
    for keep_last in (False, True):
        cfg = mm.SelectionConfig(mode=mm.MMSKV_MASS, keep_last=keep_last)
        idx, counts = _select(cfg, budget, mass)
        for c in range(2):
            want = _best(mass[0, c, :-1], budget - 1).tolist() + [T - 1] if keep_last else _best(mass[0, c], budget)
            assert counts[0, c] == budget and np.array_equal(idx[0, c], want)


@pytest.mark.parametrize("T,G,budget", [(700, 4, 300), (4000, 32, 409), (16384, 8, 2000), (40000, 3, 1024)])
def test_votes_alone(T, G, budget):
    """lambda = 0: the score is the bare vote count, so that whole vote classes tie."""
    import paper_2607_22586_amd as mm
    print("votes", T, G, budget, flush=True)
    rng = np.random.default_rng(T)
    gm = (rng.integers(1, 1 << 12, (1, 2, G, T)) * 2.0 ** -24).astype(np.float32)   # exact sums below 32
    anchor = rng.random((1, 2, T)).astype(np.float32) / T
    cfg = mm.SelectionConfig(P=32 * G, G=G, tau=0.75, lam=0.0)
    idx, counts = _select(cfg, budget, gm.sum(2), gm, anchor)
    for c in range(2):
        votes = np.zeros(T)
        for g in range(G):
            order = np.lexsort((np.arange(T), -gm[0, c, g]))
            run = np.cumsum(gm[0, c, g][order].astype(np.float64))
            votes[order[:int(np.searchsorted(run, 0.75 * run[-1])) + 1]] += 1
        want = np.append(_best(votes[:-1], budget - 1), T - 1)
        assert counts[0, c] == budget and np.array_equal(idx[0, c], want)


@pytest.mark.parametrize("T,budget", [(129, 64), (1000, 256), (1025, 300), (4097, 409), (8193, 512), (16384, 8000),
                                      (32768, 256), (32769, 256), (70001, 1024), (524289, 700)])
@pytest.mark.parametrize("kind", ["near", "peaked", "tiny"])
def test_large_buckets(T, budget, kind):
    """Masses within 1%, masses over hundreds of octaves, and masses below the digits' range."""
    import paper_2607_22586_amd as mm
    print("buckets", T, budget, kind, flush=True)
    rng = np.random.default_rng(T)
    x = rng.standard_normal((1, 2, T))
    mass = {"near": 0.3 * (1 + 0.01 * x), "peaked": np.exp2(-30 * np.abs(x)), "tiny": 2.0 ** -60 * np.exp2(x)}[kind]
    mass = mass.astype(np.float32)
    idx, counts = _select(mm.SelectionConfig(mode=mm.MMSKV_MASS, keep_last=False), budget, mass)
    # the same as votes: one group whose tau-set is its largest mass, ranked by the anchor
    gm = np.zeros((1, 2, 1, T), np.float32)
    gm[..., T // 3] = 1.0
    cfg = mm.SelectionConfig(P=32, G=1, keep_last=False)
    vidx, vcounts = _select(cfg, budget, gm.sum(2), gm, mass)
    for c in range(2):
        assert counts[0, c] == budget and np.array_equal(idx[0, c], _best(mass[0, c], budget))
        score = mass[0, c].astype(np.float64) + gm[0, c, 0]
        assert vcounts[0, c] == budget and np.array_equal(vidx[0, c], _best(score, budget))
