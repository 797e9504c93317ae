"""Selection over rows at the edges of its kernels' ranges, against numpy:
the register-resident tau cut (512 and 1024 threads, up to 64 masses a
thread), the sweep tau cut above 65536 keys, the register-resident top-k up to
32768 keys and the sweep top-k above, with ties, zero masses and every budget
form.  Masses are multiples of 2^-30 below 2^-12, so that a row of 100003 totals less
than its 32 proxies (the bound of the fixed-point sums) and every sum is exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    # T, G, tau, keep_last, budget, levels (distinct masses; few = many ties)
    (1, 1, 0.95, True, 4, 8), (31, 3, 0.5, True, 7, 4), (1025, 33, 0.95, False, 64, 1 << 18),
    (4097, 32, 0.95, True, 409, 16), (8192, 32, 1.0, True, 1, 1 << 18), (16384, 5, 0.9, True, 256, 3),
    (16385, 2, 0.95, True, 300, 1 << 18), (32768, 2, 0.95, False, 1024, 1 << 18), (32769, 3, 0.95, True, 1, 5),
    (40001, 2, 0.95, True, 1024, 1 << 18), (65536, 2, 0.6, False, 777, 2), (65537, 2, 0.95, True, 2000, 1 << 18),
    (100003, 3, 0.95, True, 512, 40),
]


def _expected(gm, anchor, tau, lam, keep_last, budget):
    G, T = gm.shape
    votes = np.zeros(T, np.int64)
    for g in range(G):
        order = np.lexsort((np.arange(T), -gm[g]))
        run = np.cumsum(gm[g][order])            # exact integers
        n = int(np.searchsorted(run, np.ceil(tau * run[-1]))) + 1 if run[-1] else 0
        votes[order[:n]] += 1
    score = votes.astype(np.float64) + lam * anchor.astype(np.float64)
    if T <= budget:
        return votes, np.arange(T)
    pool, want = (T - 1, budget - 1) if keep_last else (T, budget)
    best = np.lexsort((np.arange(pool), -score[:pool]))[:want]
    return votes, np.sort(np.concatenate([best, [T - 1]]) if keep_last else best)


@pytest.mark.parametrize("T,G,tau,keep_last,budget,levels", CASES)
def test_rows_at_range_edges(T, G, tau, keep_last, budget, levels):
    import paper_2607_22586_amd as mm
    print("select", T, G, tau, keep_last, budget, levels, flush=True)
    rng = np.random.default_rng(T)
    units = rng.integers(0, levels, (1, 2, G, T))        # mass in units of 2^-30
    anchor = (rng.integers(0, min(levels, 1 << 10), (1, 2, T)) * 2.0 ** -11).astype(np.float32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")  # noqa: E731
    gm = (units * 2.0 ** -30).astype(np.float32)
    cfg = mm.SelectionConfig(P=32 * G, G=G, tau=tau, keep_last=keep_last)
    sc = mm.ScoreOut(dev(gm), dev(gm.sum(2)), dev(anchor))
    budgets = torch.tensor([[budget, max(1, budget // 2)]], dtype=torch.int32, device="cuda:0")
    sel = mm.select_topk(sc, cfg, budget, None, budgets, Hq=2, want_votes=True)
    idx, counts, votes = (x.cpu().numpy() for x in (sel.idx, sel.counts, sel.votes))
    for c in range(2):
        want_votes, want = _expected(units[0, c], anchor[0, c], tau, 1.0, keep_last, int(budgets[0, c]))
        assert np.array_equal(votes[0, c], want_votes)
        assert counts[0, c] == len(want)
        assert np.array_equal(idx[0, c, :len(want)], want) and (idx[0, c, len(want):] == -1).all()
