"""The work that a program selecting KV caches with this package does, as
measurable cases: whole layers, the score passes alone, the selection alone,
the hidden-state proxies, the decode-time check and the baseline selectors,
from one small layer to the largest batch of the benchmark.

Every case goes through the package's public calls.  Inputs come from the
package's seeded generator (low-rank visual rows and wider text rows) or, for
the selection alone, from seeded softmax rows.  ``exact`` recomputes the
outputs in 64 bits with plain torch.
"""
from __future__ import annotations

import math

import torch

import paper_2607_22586_amd.binding as mm
from paper_2607_22586_amd import workloads

DEV = "cuda:0"
LOG2E = math.log2(math.e)
P, G, GAMMA, TAU = 512, 32, 10.0, 0.95        # the paper's settings
SINKS, POOL, WINDOW = 4, 5, 32                # the baselines' settings

_LAYER = dict(kind="layer", d=128, dtype="bf16", rope=False, mode="vote")
_SCORE = dict(kind="score", d=128, dtype="bf16", layout="heads", mode="vote", W=64)


def listed():
    return [
        # one small fp32 layer, allocating its outputs: latency and launches
        dict(_LAYER, name="layer_tiny_f32", B=1, Hq=4, Hkv=1, d=64, T=1024, W=16, budget=64, dtype="f32"),
        # one layer of a 7B model after a single image, proxies at a future position
        dict(_LAYER, name="layer_4k_rope", B=1, Hq=28, Hkv=4, T=4096, W=32, budget=409, rope=True),
        # a few images in one prompt of odd length
        dict(_LAYER, name="layer_8k", B=1, Hq=28, Hkv=4, T=8191, W=32, budget=512),
        # a serving batch of long prompts, the benchmark's layer
        dict(_LAYER, name="layer_16k_b4", B=4, Hq=28, Hkv=4, T=16384, W=64, budget=256),
        # every query head with its own KV head, keys in a token-major cache
        dict(_SCORE, name="score_mha_2880", B=1, Hq=32, Hkv=32, T=2880, layout="tokens"),
        # unquantised fp32 cache of an odd length, ranked by mass
        dict(_SCORE, name="score_f32_12k", B=1, Hq=28, Hkv=4, T=12345, dtype="f32", mode="mass"),
        # a large model's layer at the longest prompt of the efficiency sweep
        dict(_SCORE, name="score_32k", B=1, Hq=64, Hkv=8, T=32768),
        # selection and gather of a very long prompt, one budget per head
        dict(kind="select", name="select_40k", B=1, Hq=28, Hkv=4, d=128, T=40000, budget=1024, dtype="bf16",
             mode="vote", per_head=True),
        # statistics, samples and projection from the hidden states
        dict(kind="hidden", name="hidden_16k_b4", B=4, T=16384, Hq=28, d=128, dtype="bf16", rope=True),
        # decode queries against the full and the compacted cache
        dict(kind="decode", name="decode_16k_b4", B=4, Hq=28, Hkv=4, d=128, T=16384, n_dec=16, c_max=256,
             dtype="bf16"),
        # the same check on an fp32 cache of one image
        dict(kind="decode", name="decode_4k_f32", B=1, Hq=28, Hkv=4, d=128, T=4096, n_dec=4, c_max=409,
             dtype="f32"),
        # the window-attention baseline on the benchmark's layer
        dict(kind="baseline", name="snapkv_16k_b4", which="snapkv", B=4, Hq=28, Hkv=4, d=128, T=16384, W=64,
             budget=256, dtype="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


HEADS = ((4, 1, 64), (28, 4, 128), (28, 4, 128), (32, 8, 128), (32, 32, 128), (64, 8, 128), (16, 2, 64))
MOST_ROWS = 4 * 28 * 16384                     # query heads x keys of the largest listed layer


def draw(rng):
    kind = rng.choice(("layer", "layer", "score", "score", "select", "hidden", "decode", "baseline"))
    dtype = rng.choice(("bf16", "bf16", "bf16", "f32"))
    hq, hkv, d = rng.choice(HEADS)
    b = rng.choice((1, 1, 2, 4))
    if kind == "hidden":
        hq, d = rng.choice(((28, 128), (16, 128), (32, 64), (12, 64)))
        return dict(kind=kind, B=b, T=_log(rng, 256, 16384), Hq=hq, d=d, dtype="bf16" if b > 2 else dtype,
                    rope=rng.random() < 0.5)
    if kind == "select":
        t = _log(rng, 512, 100000)
        while b * hkv * t > 1 << 19:
            t = t // 2 + 1
        return dict(kind=kind, B=b, Hq=hq, Hkv=hkv, d=d, T=t, budget=_log(rng, 32, 2048), dtype=dtype,
                    mode=rng.choice(("vote", "vote", "mass")), per_head=rng.random() < 0.5)
    t = _log(rng, 256, 32768)
    while b * hq * t > MOST_ROWS:
        t = t // 2 + 1
    if kind == "decode":
        return dict(kind=kind, B=b, Hq=hq, Hkv=hkv, d=d, T=t, n_dec=rng.randint(1, min(32, 256 * hkv // hq)),
                    c_max=_log(rng, 32, 1024), dtype=dtype)
    if kind == "baseline":
        return dict(kind=kind, which=rng.choice(("snapkv", "expected", "streaming")), B=b, Hq=hq, Hkv=hkv, d=d,
                    T=t, W=rng.randint(32, 96), budget=_log(rng, 48, 1024), dtype=dtype)
    mode = rng.choice(("vote", "vote", "mass"))
    if kind == "layer":
        return dict(kind=kind, B=b, Hq=hq, Hkv=hkv, d=d, T=t, W=rng.randint(8, 128), budget=_log(rng, 32, 1024),
                    dtype=dtype, rope=rng.random() < 0.5, mode=mode)
    return dict(kind=kind, B=b, Hq=hq, Hkv=hkv, d=d, T=t, W=64, dtype=dtype, mode=mode,
                layout=rng.choice(("heads", "tokens")))


# ---------------------------------------------------------------- inputs
def _inputs(case, seed, W, n_dec=0):
    n_text = max(1, min(512, case["T"] // 8))
    w = workloads.Workload("case", 11, case["B"], 1, case["Hq"], case["Hkv"], case["d"], case["T"], W, 0,
                           case["dtype"], "lowrank", n_text)
    return workloads.make_layer(w, seed, DEV, n_dec=n_dec)


def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 7919 + stream * 104_729 + 17) & 0x7FFFFFFF)
    return g


def _mode(case):
    return mm.MMSKV_MASS if case.get("mode") == "mass" else mm.MMSKV_VOTE


def _config(case, seed):
    return mm.SelectionConfig(P=P, G=G, gamma=GAMMA, tau=TAU, layer=seed % 80, seed=1000 + seed, mode=_mode(case))


def _rope(case, position):
    return [t.to(DEV) for t in workloads.rope_tables(case["d"], position)] if case["rope"] else None


def _scale(d):
    return LOG2E / math.sqrt(d)


def _bf16(x64):
    """fp64 -> fp32 -> bf16, the rounding of every query row."""
    return x64.float().bfloat16()


def _token_major(x):
    return x.transpose(1, 2).contiguous().transpose(1, 2)


def prepare(case, seed):
    with torch.no_grad():
        return _PREPARE[case["kind"]](case, seed)


def _prepare_layer(case, seed):
    x = _inputs(case, seed, case["W"])
    return dict(case=case, q=x["q_win"], k=x["k"], v=x["v"], cfg=_config(case, seed),
                rope_f=_rope(case, case["T"] + 256), rope_l=_rope(case, case["T"] - 1))


def _prepare_score(case, seed):
    # proxies of the paper's law, drawn by torch; the workspace and the
    # outputs are kept, as a program that scores layer after layer keeps them
    x = _inputs(case, seed, case["W"])
    q = x["q_win"].double()
    z = torch.randn((case["B"], case["Hq"], P, case["d"]), generator=_gen(seed, 1), device=DEV, dtype=torch.float32)
    rows = q.mean(2, keepdim=True) + GAMMA * q.std(2, correction=0, keepdim=True) * z.double()
    cfg = _config(case, seed)
    k = _token_major(x["k"]) if case["layout"] == "tokens" else x["k"]
    B, Hq, Hkv, T, d = (case[n] for n in ("B", "Hq", "Hkv", "T", "d"))
    ws = torch.empty(mm.score_workspace(B, Hq, Hkv, T, case["W"], d, cfg), dtype=torch.uint8, device=DEV)
    gm = torch.empty((B, Hkv, G, T), dtype=torch.float32, device=DEV) if cfg.mode == mm.MMSKV_VOTE else None
    out = mm.ScoreOut(gm, torch.empty((B, Hkv, T), dtype=torch.float32, device=DEV),
                      torch.empty((B, Hkv, T), dtype=torch.float32, device=DEV))
    return dict(case=case, proxies=_bf16(rows * _scale(d)), q_last=x["q_win"][:, :, -1].bfloat16().contiguous(),
                k=k, cfg=cfg, ws=ws, out=out)


def _prepare_select(case, seed):
    # masses like those of the proxies: sums of peaked softmax rows
    B, Hq, Hkv, T, d = (case[n] for n in ("B", "Hq", "Hkv", "T", "d"))
    g = _gen(seed, 2)
    rows = (P // G) * (Hq // Hkv)
    gm = torch.zeros((B, Hkv, G, T), device=DEV)
    for _ in range(4):
        gm += torch.softmax(3.0 * torch.randn((B, Hkv, G, T), generator=g, device=DEV), dim=-1)
    gm *= rows / 4.0
    anchor = torch.softmax(2.0 * torch.randn((B, Hkv, T), generator=g, device=DEV), dim=-1)
    cfg = _config(case, seed)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    k, v = (torch.randn((B, Hkv, T, d), generator=g, device=DEV).to(dt) for _ in range(2))
    budgets = None
    if case["per_head"]:
        budgets = torch.randint(case["budget"] // 2, case["budget"] + 1, (B, Hkv), generator=g, device=DEV,
                                dtype=torch.int32)
    ws = torch.empty(mm.select_workspace(B, Hq, Hkv, T, 1, d, cfg), dtype=torch.uint8, device=DEV)
    c = case["budget"]
    votes = torch.empty((B, Hkv, T), dtype=torch.uint8, device=DEV) if cfg.mode == mm.MMSKV_VOTE else None
    out = mm.Selected(torch.empty((B, Hkv, c), dtype=torch.int32, device=DEV),
                      torch.empty((B, Hkv), dtype=torch.int32, device=DEV), votes)
    kv = tuple(torch.empty((B, Hkv, c, d), dtype=dt, device=DEV) for _ in range(2))
    return dict(case=case, cfg=cfg, scores=mm.ScoreOut(gm, gm.sum(2), anchor), k=k, v=v, budgets=budgets, ws=ws,
                out=out, kv=kv)


def _prepare_hidden(case, seed):
    x = workloads.custom_hidden(case["B"], case["T"], case["Hq"] * case["d"], case["Hq"], case["d"], case["dtype"],
                                seed, DEV)
    return dict(case=case, hidden=x["hidden"], wq=x["wq"], cfg=_config(case, seed),
                rope=_rope(case, case["T"] + 256))


def _prepare_decode(case, seed):
    x = _inputs(case, seed, 32, n_dec=case["n_dec"])
    B, Hkv, T, c_max = case["B"], case["Hkv"], case["T"], case["c_max"]
    n = min(c_max, T)
    keep = torch.argsort(torch.rand((B, Hkv, T), generator=_gen(seed, 3), device=DEV), dim=-1)[:, :, :n]
    keep = keep.sort(dim=-1).values
    idx = torch.full((B, Hkv, c_max), -1, dtype=torch.int32, device=DEV)
    idx[:, :, :n] = keep.int()
    rows = keep.unsqueeze(-1).expand(B, Hkv, n, case["d"])
    kv = []
    for t in (x["k"], x["v"]):
        o = torch.zeros((B, Hkv, c_max, case["d"]), dtype=t.dtype, device=DEV)
        o[:, :, :n] = torch.gather(t, 2, rows)
        kv.append(o)
    ws = torch.empty(max(256, mm.decode_workspace(B, case["Hq"], Hkv, T, case["d"], case["n_dec"])),
                     dtype=torch.uint8, device=DEV)
    out = (torch.empty((B, case["Hq"], case["n_dec"]), dtype=torch.float32, device=DEV),
           torch.empty((B, case["Hq"], case["n_dec"], case["d"]), dtype=torch.float32, device=DEV))
    sel = mm.Selected(idx, torch.full((B, Hkv), n, dtype=torch.int32, device=DEV), None)
    return dict(case=case, q_dec=x["q_dec"], k=x["k"], sel=sel, k_out=kv[0], v_out=kv[1], ws=ws, out=out)


def _prepare_baseline(case, seed):
    x = _inputs(case, seed, case["W"])
    return dict(case=case, q=x["q_win"], k=x["k"], v=x["v"], seed=1000 + seed, layer=seed % 80)


_PREPARE = dict(layer=_prepare_layer, score=_prepare_score, select=_prepare_select, hidden=_prepare_hidden,
                decode=_prepare_decode, baseline=_prepare_baseline)


# ---------------------------------------------------------------- the pass
def run(state):
    return _RUN[state["case"]["kind"]](state)


def _run_layer(s):
    r = mm.select_layer(s["q"], s["k"], s["v"], s["case"]["budget"], s["cfg"], rope_f=s["rope_f"],
                        rope_l=s["rope_l"])
    return dict(proxies=r.proxies, q_last=r.q_last, group_mass=r.scores.group_mass, mass=r.scores.mass,
                anchor=r.scores.anchor, idx=r.sel.idx, counts=r.sel.counts, k_out=r.k_out, v_out=r.v_out)


def _run_score(s):
    r = mm.score(s["proxies"], s["q_last"], s["k"], s["cfg"], s["case"]["W"], out=s["out"], workspace=s["ws"])
    return dict(group_mass=r.group_mass, mass=r.mass, anchor=r.anchor)


def _run_select(s):
    c = s["case"]
    sel = mm.select_topk(s["scores"], s["cfg"], c["budget"], None, s["budgets"], c["Hq"], out=s["out"],
                         workspace=s["ws"])
    ko, vo = mm.gather_kv(s["k"], s["v"], sel, out=s["kv"])
    return dict(idx=sel.idx, counts=sel.counts, votes=sel.votes, k_out=ko, v_out=vo)


def _run_hidden(s):
    stats = mm.hidden_stats(s["hidden"])
    hp = mm.hidden_proxies(stats, s["cfg"], s["case"]["T"])
    return dict(stats=stats, hp=hp, proxies=mm.project_proxies(hp, s["wq"], s["case"]["Hq"], s["rope"]))


def _run_decode(s):
    cov, out = mm.decode_check(s["q_dec"], s["k"], s["sel"], s["k_out"], s["v_out"], workspace=s["ws"],
                               out=s["out"])
    return dict(coverage=cov, out=out)


def _run_baseline(s):
    c = s["case"]
    sel, score, mass, ko, vo = mm.baseline_select(c["which"], s["q"], s["k"], s["v"], c["budget"], s["seed"],
                                                  s["layer"], window=WINDOW, pool=POOL, sinks=SINKS, P=P)
    return dict(idx=sel.idx, counts=sel.counts, score=score, mass=mass, k_out=ko, v_out=vo)


_RUN = dict(layer=_run_layer, score=_run_score, select=_run_select, hidden=_run_hidden, decode=_run_decode,
            baseline=_run_baseline)


# ---------------------------------------------------------------- its size
def work(case):
    """Bytes of the inputs and outputs, each once, and the matrix products
    each formed once (the logits are needed twice, before and after their row
    sums, but how they come back the second time is the kernel's choice)."""
    kind, B, Hq, T, d = case["kind"], case["B"], case["Hq"], case["T"], case["d"]
    eb = 4 if case["dtype"] == "f32" else 2
    if kind == "hidden":
        D = Hq * d
        return dict(bytes=B * T * D * eb + D * D * 2 + 16 * B * D + 4 * B * P * D, flops=2 * B * P * D * D)
    Hkv = case["Hkv"]
    keys = B * Hkv * T
    if kind == "decode":
        kept = B * Hkv * min(case["c_max"], T)
        rows = B * Hq * case["n_dec"]
        return dict(bytes=keys * d * eb + kept * (4 + 2 * d * eb) + rows * (2 * d + 4 + 4 * d),
                    flops=2 * rows * d * (T + 2 * min(case["c_max"], T)))
    vote = _mode(case) == mm.MMSKV_VOTE and kind != "baseline"
    rows = {"baseline": {"snapkv": WINDOW, "expected": P, "streaming": 0}.get(case.get("which"), 0)}.get(kind, P)
    masses = keys * (4 * G if vote else 0) + 8 * keys
    kept = 0 if kind == "score" else B * Hkv * min(case["budget"], T)
    moved = kept * (4 + 4 * d * eb)
    if kind == "select":
        return dict(bytes=keys * ((4 * G + 4 + 1) if vote else 4) + moved, flops=keys * (G if vote else 1))
    flops = 2 * B * Hq * (rows + 1) * d * T if rows else keys
    proxies = 2 * B * Hq * (rows + 1) * d
    if kind == "score":
        return dict(bytes=keys * d * eb + proxies + masses, flops=flops)
    window = B * Hq * case["W"] * d * eb
    if kind == "baseline":
        return dict(bytes=(keys * d * eb + window if rows else 0) + 8 * keys + moved, flops=flops)
    return dict(bytes=keys * d * eb + proxies + window + masses + moved, flops=flops)


def tolerance(case):
    kind = case["kind"]
    if kind == "select":
        return "exact"
    if kind == "hidden":
        # bf16 proxies of a reduction over D values
        return dict(rel=5e-4, max=0.01, differ=0.0)
    if kind == "decode":
        # fp32 logits and sums; the attention's values come from bf16 products
        return dict(rel=5e-6, max=2e-4)
    # fp32 logits of up to ~100 and fp32 sums of their powers; a key whose
    # vote sits on a group's cut may change places with another
    return dict(rel=2e-5, max=1e-3, differ=0.005)


# ---------------------------------------------------------------- in 64 bits
def exact(case, seed):
    if case["kind"] == "select" or case.get("which") == "streaming":
        return None
    with torch.no_grad():
        return _EXACT[case["kind"]](case, prepare(case, seed))


def _philox(counter, key):
    """Philox4x32-10 (Salmon et al., SC 2011) on int64 tensors holding 32-bit words."""
    c = [x.to(torch.int64) for x in counter]
    k0, k1 = key

    def mul(m, x):
        lo, hi = m * (x & 0xFFFF), m * (x >> 16)
        return (lo + ((hi & 0xFFFF) << 16)) & 0xFFFFFFFF, (hi + (lo >> 16)) >> 16

    for _ in range(10):
        l0, h0 = mul(0xD2511F53, c[0])
        l1, h1 = mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _normals(cfg, B, heads, rows, dims):
    """[B, heads, rows, dims] fp64 Box-Muller normals of the package's counter
    layout; `heads` lists the head fields."""
    def ax(v, i):
        return torch.as_tensor(v, dtype=torch.int64, device=DEV).reshape([-1 if j == i else 1 for j in range(4)])
    shape = (B, len(heads), rows, dims // 4)
    b = ax(list(range(B)), 0)
    counter = [t.expand(shape) for t in (ax(list(range(dims // 4)), 3), ax(list(range(rows)), 2), ax(heads, 1),
                                         (b << 16) | cfg.layer)]
    w = _philox(counter, (cfg.seed & 0xFFFFFFFF, cfg.seed >> 32))
    u = [(2 * (x >> 9) + 1).double() * 2.0 ** -24 for x in w]
    z = []
    for p in (0, 2):
        r, turn = torch.sqrt(-2.0 * torch.log(u[p])), 2.0 * math.pi * u[p + 1]
        z += [r * torch.cos(turn), r * torch.sin(turn)]
    return torch.stack(z, dim=-1).reshape(B, len(heads), rows, dims)


def _rotate(x, rope):
    if rope is None:
        return x
    c, s = (t.double() for t in rope)
    h = x.shape[-1] // 2
    return torch.cat([x[..., :h] * c - x[..., h:] * s, x[..., h:] * c + x[..., :h] * s], dim=-1)


def _masses(proxies, q_last, k, groups):
    """fp64 group masses, masses and anchor of bf16 query rows against bf16 keys."""
    B, Hq, rows, d = proxies.shape
    Hkv, T = k.shape[1], k.shape[2]
    Gh = Hq // Hkv
    keys = k.bfloat16().double()
    anc = _bf16(q_last.double() * _scale(d)).double()
    gm = torch.empty((B, Hkv, groups, T), dtype=torch.float64, device=DEV)
    an = torch.empty((B, Hkv, T), dtype=torch.float64, device=DEV)
    for b in range(B):
        for c in range(Hkv):
            kt = keys[b, c].t().contiguous()
            tot = torch.zeros((groups, T), dtype=torch.float64, device=DEV)
            for h in range(c * Gh, (c + 1) * Gh):
                p = torch.softmax((proxies[b, h].double() @ kt) * math.log(2.0), dim=-1)
                tot += p.reshape(groups, rows // groups, T).sum(1)
            gm[b, c] = tot
            an[b, c] = torch.softmax((anc[b, c * Gh:(c + 1) * Gh] @ kt) * math.log(2.0), dim=-1).mean(0)
    return gm, gm.sum(2), an


def _proxy_rows(case, s, gamma, cfg, rope):
    q = s["q"].double()
    z = _normals(cfg, case["B"], list(range(case["Hq"])), P, case["d"])
    x = q.mean(2, keepdim=True) + gamma * q.std(2, correction=0, keepdim=True) * z
    return _rotate(x, rope) * _scale(case["d"])


def _exact_layer(case, s):
    rows = _proxy_rows(case, s, GAMMA, s["cfg"], s["rope_f"])
    last = _rotate(s["q"][:, :, -1].double(), s["rope_l"])
    gm, mass, an = _masses(_bf16(rows), _bf16(last), s["k"], G)
    return dict(proxies=rows, q_last=last, group_mass=gm if _mode(case) == mm.MMSKV_VOTE else None, mass=mass,
                anchor=an, idx=None, counts=None, k_out=None, v_out=None)


def _exact_score(case, s):
    gm, mass, an = _masses(s["proxies"], s["q_last"], s["k"], G)
    return dict(group_mass=gm if _mode(case) == mm.MMSKV_VOTE else None, mass=mass, anchor=an)


def _exact_hidden(case, s):
    D = case["Hq"] * case["d"]
    stats = torch.empty((case["B"], 2, D), dtype=torch.float64, device=DEV)
    for b in range(case["B"]):
        h = s["hidden"][b].double()
        stats[b, 0], stats[b, 1] = h.mean(0), h.std(0, correction=0)
    z = _normals(s["cfg"], case["B"], [0xFFFFFFFF], P, D)[:, 0]
    hp = stats[:, 0:1] + GAMMA * stats[:, 1:2] * z
    q = _bf16(hp).double() @ s["wq"].double().t()
    q = q.reshape(case["B"], P, case["Hq"], case["d"]).transpose(1, 2)
    return dict(stats=stats, hp=hp, proxies=_rotate(q, s["rope"]) * _scale(case["d"]))


def _exact_decode(case, s):
    B, Hq, n, d = s["q_dec"].shape
    Hkv = case["Hkv"]
    Gh, kept = Hq // Hkv, min(case["c_max"], case["T"])
    q = _bf16(s["q_dec"].double() * _scale(d)).double()
    cov = torch.empty((B, Hq, n), dtype=torch.float64, device=DEV)
    out = torch.empty((B, Hq, n, d), dtype=torch.float64, device=DEV)
    for b in range(B):
        for h in range(Hq):
            c = h // Gh
            p = torch.softmax((q[b, h] @ s["k"][b, c].bfloat16().double().t().contiguous()) * math.log(2.0), dim=-1)
            cov[b, h] = p[:, s["sel"].idx[b, c, :kept].long()].sum(-1)
            kc = s["k_out"][b, c, :kept].bfloat16().double().t().contiguous()
            out[b, h] = torch.softmax((q[b, h] @ kc) * math.log(2.0), dim=-1) @ s["v_out"][b, c, :kept].double()
    return dict(coverage=cov, out=out)


def _exact_baseline(case, s):
    if case["which"] == "snapkv":
        rows = s["q"][:, :, -WINDOW:].bfloat16().double() * _scale(case["d"])
    else:
        cfg = mm.SelectionConfig(P=P, gamma=1.0, seed=s["seed"], layer=s["layer"])
        rows = _proxy_rows(case, s, 1.0, cfg, None)
    mass = _masses(_bf16(rows), s["q"][:, :, -1].bfloat16(), s["k"], 1)[1]
    return dict(idx=None, counts=None, score=None, mass=mass, k_out=None, v_out=None)


_EXACT = dict(layer=_exact_layer, score=_exact_score, hidden=_exact_hidden, decode=_exact_decode,
              baseline=_exact_baseline)
