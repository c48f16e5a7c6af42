"""Performance cases: the work a user of this library has it do, one dict of plain sizes per case.

Every case goes through the Python binding's public calls (paper_2608_25230_amd.fw) on
device tensors.  The kinds are the library's entry points:

  subset   best_subset: the exhaustive best kept set of small rows
  topk     dense_topk: dense output, forced outputs, gaps and top-k indices per budget
  swap     swap: the balancing selector over the full neighbourhood
  pool     pool_subset: candidate sets, ES_pool, balancing, certificates
  vote     group_vote: one kept set per key/value head and position
  curve    dropped_mass_curve: observation-window importance and the per-cell curve
  compact  ragged_compact (after maxpool_scores when pooled): allocation and K/V compaction

Inputs are drawn on the GPU from the seed, by the recipes of workloads.py: standard normal
queries, keys and values, a sink logit, outlier key channels, heavy keys, per-cell
temperatures, keys that share a row direction.
"""
import itertools
import math

import numpy as np
import torch

from paper_2608_25230_amd import fw

BF16, F32 = "bf16", "f32"
PROTOCOL = ((4, 24), (8, 12), (16, 6), (32, 4))  # (s, extra) of the enumeration protocol


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # 256 sixteen-key rows: the smallest call, where launches and latency count
        dict(name="subset_tiny", kind="subset", dtype=F32, H=256, G=1, n=16, d=64, k=4, sink=True, shift=0.0),
        # the enumeration workload: every 6-subset of 24 keys for 168,192 rows
        dict(name="subset_exhaustive", kind="subset", dtype=F32, H=168192, G=1, n=24, d=128, k=6, sink=False,
             shift=1.5),
        # one decoding position of a layer at batch 8: 64 key/value heads of 4 query rows, a ragged cache
        dict(name="topk_decode", kind="topk", dtype=BF16, H=64, G=4, n=5003, d=128, ks="128,512,1024", idx=True),
        # the headline: 32 layers x 8 heads, 256 rows each, three budgets, no index list
        dict(name="topk_prefill", kind="topk", dtype=BF16, H=256, G=256, n=4096, d=128, ks="128,512,1024",
             idx=False),
        # float32 rows of 64-wide heads, sizes that no tile divides
        dict(name="topk_f32", kind="topk", dtype=F32, H=16, G=90, n=1999, d=64, ks="64,250,999", idx=True),
        # long rows, one budget
        dict(name="topk_long", kind="topk", dtype=BF16, H=8, G=128, n=32768, d=128, ks="1024", idx=True),
        # balancing on mid-size float32 rows
        dict(name="swap_mid", kind="swap", dtype=F32, H=4, G=30, n=2001, d=64, k=128, iters=16, heavy=8),
        # balancing on long rows: 8 heads of 128 rows, 32,768 keys, 1,024 kept, at most 64 swaps
        dict(name="swap_long", kind="swap", dtype=BF16, H=8, G=128, n=32768, d=128, k=1024, iters=64, heavy=16),
        # the enumeration protocol on full-length rows, six sampled rows per query head
        dict(name="pool_protocol", kind="pool", dtype=BF16, H=256, G=24, n=4096, d=128, budgets="4:24,8:12,16:6,32:4",
             swaps=64),
        # the group vote on the same rows
        dict(name="vote", kind="vote", dtype=BF16, H=256, G=24, n=4096, d=128, s=8, group=4),
        # ContourKV's scores and curves: 256 cells of 131,072 keys, 64 window queries
        dict(name="curve_long", kind="curve", dtype=BF16, H=256, G=64, n=131072, d=128, order=False),
        # ContourKV's allocation and compaction of the same cells at a tenth of the entries
        dict(name="compact_long", kind="compact", dtype=BF16, H=256, per_layer=8, n=131072, d=128, keep=0.1, floor=32,
             cap=0.0, pool=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["topk", "topk", "topk", "subset", "swap", "pool", "vote", "curve", "compact"])
    c = dict(kind=kind, dtype=rng.choice([BF16, BF16, F32]), d=rng.choice([64, 80, 128, 128, 128]))
    if kind == "subset":
        c["dtype"], c["d"] = F32, rng.choice([16, 64, 128])
        c["n"] = rng.randint(8, 36)
        c["k"] = rng.randint(1, max(1, min(8, c["n"] - 1)))
        while math.comb(c["n"], c["k"]) > 140000:
            c["k"] -= 1
        work = math.comb(c["n"], c["k"]) + 4 * c["n"] ** 2
        c["H"], c["G"] = min(_log(rng, 64, 160000), max(16, int(6e9 / work))), 1
        c.update(sink=rng.random() < 0.5, shift=rng.choice([0.0, 1.5]))
    elif kind == "topk":
        # decode: a few rows of each head; prefill: blocks of rows
        c["G"] = rng.choice([1, 4, 8, 16 * _log(rng, 1, 16), _log(rng, 9, 256)])
        c["n"] = _log(rng, 100, 32768)
        if rng.random() < 0.4:
            c["n"] = rng.choice([1024, 2048, 4096])
        c["H"] = min(_log(rng, 4, 256), max(1, int(1.3e8 / (c["G"] * c["n"]))))
        c["idx"] = rng.random() < 0.5
        c["ks"] = ",".join(str(max(1, c["n"] // f)) for f in rng.choice([(32, 8, 4), (4,), (16, 2), (64, 32, 16, 8, 4)]))
    elif kind == "swap":
        c["n"] = _log(rng, 48, 16000)
        c["k"] = max(1, int(c["n"] * rng.uniform(0.03, 0.3)))
        c["iters"] = _log(rng, 4, 64)
        c["heavy"] = rng.choice([0, min(16, c["n"] // 8)])
        rows = max(4, min(1024, int(8e11 / (c["k"] * c["n"] * c["iters"]))))
        c["G"] = rng.choice([1, 4, 8, 30, 32])
        c["H"] = max(1, min(16, rows // c["G"]))
    elif kind == "pool":
        c["n"] = _log(rng, 128, 8192)
        c["budgets"] = ",".join("%d:%d" % b for b in sorted(rng.sample(PROTOCOL, rng.randint(1, 4))))
        c["G"] = rng.choice([4, 6, 24])
        c["H"] = min(_log(rng, 4, 256), max(1, int(2.5e7 / (c["G"] * c["n"]))))
        c["swaps"] = 64
    elif kind == "vote":
        c["n"] = _log(rng, 128, 8192)
        c["group"] = rng.choice([1, 4, 8])
        c["G"] = c["group"] * rng.choice([1, 6, 7])
        c["s"] = min(_log(rng, 4, 64), c["n"] // 2)
        c["H"] = min(_log(rng, 4, 256), max(1, int(2.5e7 / (c["G"] * c["n"]))))
    elif kind == "curve":
        c["n"] = _log(rng, 500, 131072)
        c["G"] = rng.choice([16, 32, 64, 64, 40])
        c["H"] = min(_log(rng, 4, 256), max(1, int(6e8 / (c["G"] * c["n"]))))
        # neighbours in the order of a long cell are nearer than float32 rounds their scores
        c["order"] = c["n"] <= 8192 and rng.random() < 0.7
    else:
        c["n"] = _log(rng, 500, 131072)
        c["per_layer"] = rng.choice([2, 4, 8])
        c["H"] = c["per_layer"] * max(1, min(_log(rng, 1, 32), int(3e7 / (c["per_layer"] * c["n"]))))
        c["keep"], c["floor"] = rng.choice([0.05, 0.1, 0.3]), rng.choice([0, 8, 16])
        c["pool"] = rng.choice([1, 7])
        c["cap"] = rng.choice([0.0, 1.0, 1.5])  # of the mean kept count; 0: no cap
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _dtype(case):
    return torch.bfloat16 if case["dtype"] == BF16 else torch.float32


def _normal(g, shape, dtype):
    """Standard normal values drawn in float32, in blocks, and rounded to dtype."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    step = 1 << 28
    for lo in range(0, flat.numel(), step):
        m = min(step, flat.numel() - lo)
        flat[lo:lo + m] = torch.randn(m, generator=g, device="cuda")
    return out


def _ks(case):
    return tuple(int(x) for x in case["ks"].split(","))


def _budgets(case):
    return tuple(tuple(int(x) for x in b.split(":")) for b in case["budgets"].split(","))


def _alloc(case):
    """(entries kept in all, cap per cell) of a compaction case."""
    H, n, floor = case["H"], case["n"], case["floor"]
    budget = max(H * floor, int(case["keep"] * H * n))
    cap = 0 if not case["cap"] else min(n, max(floor, int(math.ceil(case["cap"] * budget / H))))
    return budget, cap


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    H, n, d, dt = case["H"], case["n"], case["d"], _dtype(case)
    st = {"case": case}
    if case["kind"] == "compact":
        st["k"], st["v"] = _normal(g, (H, n, d), dt), _normal(g, (H, n, d), dt)
        # window scores: softmax weights of normal logits, a temperature per cell
        t = torch.empty(H, 1, device="cuda").uniform_(0.5, 2.0, generator=g)
        st["score"] = torch.softmax(torch.randn((H, n), generator=g, device="cuda") / (8.0 * t), dim=1).contiguous()
        return st
    G = case["G"]
    st["q"] = _normal(g, (H, G, d), dt)
    st["k"] = _normal(g, (H, n, d), dt)
    st["scale"] = torch.full((H,), 1.0 / math.sqrt(d), device="cuda")
    st["bias"] = None
    if case["kind"] in ("topk", "pool", "vote"):  # four outlier key channels
        ch = torch.randperm(d, generator=g, device="cuda")[:4]
        st["k"][:, :, ch] *= 8
    if case["kind"] in ("topk", "pool", "vote", "swap") or case.get("sink"):
        st["bias"] = torch.zeros(n, device="cuda")
        st["bias"][0] = 4.0
    if case["kind"] == "subset" and case["shift"]:  # keys share a row direction
        u = torch.randn((H, 1, d), generator=g, device="cuda")
        st["k"] += case["shift"] * u / u.norm(dim=2, keepdim=True)
    if case.get("heavy"):
        at = torch.randint(1, n, (H, case["heavy"]), generator=g, device="cuda")
        for h in range(H):
            st["k"][h, at[h].unique()] *= 3
    if case["kind"] == "curve":  # a temperature per cell; the values are not read
        st["scale"] /= torch.empty(H, device="cuda").uniform_(0.5, 2.0, generator=g)
    else:
        st["v"] = _normal(g, (H, n, d), dt)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "compact":
        budget, cap = _alloc(c)
        score = st["score"] if c["pool"] == 1 else fw.maxpool_scores(st["score"], c["pool"])
        out = fw.ragged_compact(st["k"], st["v"], score, budget, c["floor"], c["per_layer"], cap=cap)
    elif kind == "curve":
        out = fw.dropped_mass_curve(st["q"], st["k"], st["scale"], st["bias"], want_order=c["order"])
    else:
        rows = (st["q"], st["k"], st["v"])
        kw = dict(scale=st["scale"], bias=st["bias"])
        if kind == "subset":
            out = fw.best_subset(*rows, c["k"], **kw)
        elif kind == "topk":
            out = fw.dense_topk(*rows, _ks(c), **kw, want_idx=c["idx"])
        elif kind == "swap":
            out = fw.swap(*rows, c["k"], c["iters"], **kw)
        elif kind == "pool":
            out = fw.pool_subset(*rows, _budgets(c), c["swaps"], **kw)
        else:
            out = fw.group_vote(*rows, c["s"], c["group"], **kw)
    return {k: v for k, v in out.items() if k != "_ws" and v is not None}


def work(case):
    H, n, d = case["H"], case["n"], case["d"]
    e = 2 if case["dtype"] == BF16 else 4
    if case["kind"] == "compact":
        budget, _ = _alloc(case)
        # scores read, kept rows read and written, kept positions written
        return {"bytes": 4 * H * n + 4 * budget * d * e + 4 * budget, "flops": 0}
    G = case["G"]
    R = H * G
    rows = R * d * e + 2 * H * n * d * e
    if case["kind"] == "curve":
        return {"bytes": R * d * e + H * n * d * e + 4 * H * n * (3 if case["order"] else 2), "flops": 2 * R * n * d}
    if case["kind"] == "topk":
        ks = _ks(case)
        out = 4 * R * (d * (1 + len(ks)) + 2 * len(ks)) + (4 * R * max(ks) if case["idx"] else 0)
        return {"bytes": rows + out, "flops": 2 * R * n * d + 2 * R * n * d}
    if case["kind"] == "subset":
        return {"bytes": rows + 4 * R * (2 * case["k"] + 4), "flops": 5 * R * math.comb(n, case["k"]) + 2 * R * n * n * d}
    if case["kind"] == "swap":
        # per sweep: one dot per key
        return {"bytes": rows + 4 * R * (case["k"] + case["iters"] + 3), "flops": 2 * R * n * d * (2 + case["iters"])}
    if case["kind"] == "pool":
        b = _budgets(case)
        subsets = sum(math.comb(s + x, s) for s, x in b)
        return {"bytes": rows + 4 * R * sum(4 * s + x + 17 for s, x in b), "flops": 6 * R * n * d + 5 * R * subsets}
    return {"bytes": rows + 4 * R * (3 + case["s"] // case["group"]), "flops": 4 * R * n * d}


def tolerance(case):
    """About four times the error against 64 bits, and room for keys whose logits
    agree to the last bits of float32 and change places: at a budget's cut such a
    pair moves one row's set, at most max of the output's scale in that row."""
    kind = case["kind"]
    if kind == "compact":
        # positions, offsets and copies are exact; the evicted mass is a float32 of a float64 sum
        return {"rel": 1e-7, "max": 1e-6, "differ": 0.0}
    if kind == "topk":
        if case["dtype"] == F32:
            return {"rel": 5e-5, "max": 0.1, "differ": 2e-3}
        return {"rel": 5e-3, "max": 0.2, "differ": 5e-3}  # bf16 weights in the matrix products
    if kind == "swap":
        # long rows score swaps in float32; two swaps that tie there end in different sets
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-2}
    if kind == "curve":
        return {"rel": 2e-6, "max": 2e-5, "differ": 1e-2}
    # float64 throughout, float32 outputs
    return {"rel": 5e-7, "max": 1e-3, "differ": 1e-3}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------
def _weights(st, h):
    """Logits and softmax weights of the rows of units h (a slice), float64."""
    z = torch.matmul(st["q"][h].double(), st["k"][h].double().transpose(1, 2).contiguous())
    z = z * st["scale"][h].double()[:, None, None]
    if st["bias"] is not None:
        z = z + st["bias"].double()
    return z, torch.softmax(z, dim=2)


def _slices(st, limit):
    """Slices of units whose [units][G][n] arrays stay under `limit` values."""
    c = st["case"]
    step = max(1, int(limit // (c["G"] * c["n"])))
    return [slice(lo, min(c["H"], lo + step)) for lo in range(0, c["H"], step)]


def _rank(x):
    return torch.sort(x, dim=-1, descending=True, stable=True).indices


def _gather_rows(v, idx):
    """v [U][n][d], idx [U][G][m] -> [U][G][m][d]."""
    U, G, m = idx.shape
    return torch.gather(v, 1, idx.reshape(U, G * m, 1).expand(-1, -1, v.shape[2])).view(U, G, m, v.shape[2])


def _set_error(p, v, o, idx):
    """es of the kept sets idx [U][G][m]."""
    w = torch.gather(p, 2, idx)
    return ((_gather_rows(v, idx) - o[:, :, None]) * w[..., None]).sum(2).norm(dim=2) / w.sum(2)


def _combos(n, k):
    flat = np.fromiter(itertools.chain.from_iterable(itertools.combinations(range(n), k)), np.int64)
    return torch.from_numpy(flat.reshape(-1, k)).cuda()


def _best_of(gram, mass, k):
    """Least sqrt(1'G1)/mass over the k-subsets of P keys, and the first subset
    that takes it (lexicographic); gram [R][P][P], mass [R][P]."""
    R, P = mass.shape
    sets = _combos(P, k)
    ind = torch.zeros((len(sets), P), dtype=torch.float64, device="cuda").scatter_(1, sets, 1.0)
    i, j = torch.triu_indices(P, P, device="cuda")
    pairs = ind[:, i] * ind[:, j]
    tri = gram[:, i, j] * torch.where(i == j, 1.0, 2.0).double()
    es, at = [], []
    step = max(1, (1 << 26) // len(sets))
    for lo in range(0, R, step):
        s = torch.matmul(tri[lo:lo + step], pairs.t()).clamp_min(0) / torch.matmul(mass[lo:lo + step], ind.t()) ** 2
        m = s.min(dim=1)
        es.append(m.values.sqrt())
        at.append(m.indices)
    return torch.cat(es), sets[torch.cat(at)]


def _ratio(a, b):
    return torch.where(b > 0, a / b, torch.where(a == 0, 1.0, math.inf).double())


def _exact_topk(case, st):
    ks = _ks(case)
    parts = []
    for h in _slices(st, 1 << 26):
        z, p = _weights(st, h)
        v = st["v"][h].double()
        o = torch.matmul(p, v)
        order = _rank(z)
        os_, gap, drop = [], [], []
        for k in ks:
            rest = order[:, :, k:]
            kept = p.scatter(2, rest, 0.0)
            m_s = torch.matmul(kept, v) / kept.sum(2, keepdim=True)
            os_.append(m_s)
            gap.append((m_s - o).norm(dim=2))
            drop.append(torch.gather(p, 2, rest).sum(2))
        parts.append(dict(o=o, o_s=torch.stack(os_), gap=torch.stack(gap), dropped=torch.stack(drop),
                          topk_idx=order[:, :, :max(ks)].int()))
    out = {k: torch.cat([x[k] for x in parts], dim=0 if k in ("o", "topk_idx") else 1) for k in parts[0]}
    if not case["idx"]:
        del out["topk_idx"]
    return out


def _exact_subset(case, st):
    k, parts = case["k"], []
    for h in _slices(st, 1 << 18):
        z, p = _weights(st, h)
        v = st["v"][h].double()
        dev = (v - torch.matmul(p, v)) * p.transpose(1, 2)
        gram = torch.matmul(dev, dev.transpose(1, 2).contiguous())
        parts.append((gram, p[:, 0], _rank(z)[:, 0, :k]))
    gram, p, top = (torch.cat(x) for x in zip(*parts))
    es, sets = _best_of(gram, p, k)
    ind = torch.zeros_like(p).scatter_(1, top, 1.0)
    kept = (p * ind).sum(1)
    es_top = torch.matmul(ind[:, None], torch.matmul(gram, ind[:, :, None]))[:, 0, 0].clamp_min(0).sqrt() / kept
    closed = torch.where(es_top > 0, 1 - es / es_top, 0.0)
    out = dict(best_idx=sets.int(), best_gap=es, topk_gap=es_top, closed=closed, dropped_topk=(p * (1 - ind)).sum(1),
               topk_idx=top.int())
    return {k: x[:, None] for k, x in out.items()}


def _exact_swap(case, st):
    H, G, n, d, k, iters = (case[x] for x in ("H", "G", "n", "d", "k", "iters"))
    if 2.0 * H * G * k * n * d * iters > 5e13:
        return None
    traj = torch.full((H, G, iters + 1), math.nan, dtype=torch.float64, device="cuda")
    count = torch.zeros((H, G), dtype=torch.int32, device="cuda")
    final, drop = [], []
    for h in range(H):
        z, p = _weights(st, slice(h, h + 1))
        v = st["v"][h].double()
        for r in range(G):
            w = p[0, r]
            order = _rank(z[0, r])
            u = (v - w @ v) * w[:, None]
            keep, rest = order[:k].sort().values, order[k:].sort().values
            cur = u[keep].sum(0).norm() / w[keep].sum()
            traj[h, r, 0] = cur
            for it in range(iters if k < n else 0):
                g, m = u[keep].sum(0), w[keep].sum()
                a, b = g - u[keep], u[rest]
                num = (a * a).sum(1)[:, None] + (b * b).sum(1) + 2 * a @ b.t()
                err = num.clamp_min(0).sqrt() / (m - w[keep][:, None] + w[rest])
                at = int(err.argmin())
                i, j = divmod(at, n - k)
                new = torch.cat([keep[:i], keep[i + 1:], rest[j:j + 1]]).sort().values
                es = u[new].sum(0).norm() / w[new].sum()
                if not es < cur:
                    break
                rest = torch.cat([rest[:j], rest[j + 1:], keep[i:i + 1]]).sort().values
                keep, cur = new, es
                traj[h, r, it + 1] = cur
                count[h, r] = it + 1
            final.append(keep)
            drop.append(w[rest].sum())
    return dict(s_idx=torch.stack(final).view(H, G, k).int(), gap_traj=traj, n_swaps=count,
                dropped=torch.stack(drop).view(H, G))


def _exact_pool(case, st):
    """Sets, medians and certificates; the Frank-Wolfe columns too."""
    budgets, parts = _budgets(case), []
    for h in _slices(st, 1 << 24):
        z, p = _weights(st, h)
        v = st["v"][h].double()
        o = torch.matmul(p, v)
        dev = ((v * v).sum(2)[:, None] - 2 * torch.matmul(o, v.transpose(1, 2).contiguous())
               + (o * o).sum(2)[:, :, None]).clamp_min(0).sqrt()
        order = _rank(z)
        one = dict(stats=[], cell_median=[], cell_flat=[], pool_idx=[], best_idx=[], bal_idx=[], geo_idx=[],
                   n_swaps=[])
        for s, extra in budgets:
            top = order[:, :, :s]
            ext = _rank((p * dev).scatter(2, top, -1.0))[:, :, :extra]
            pool = torch.cat([top, ext], 2)
            keys, place = pool.sort(dim=2)
            U, G, P = keys.shape
            x = (_gather_rows(v, keys) - o[:, :, None]).view(U * G, P, -1)
            w = torch.gather(p, 2, keys).view(U * G, P)
            y = torch.matmul(x, x.transpose(1, 2).contiguous())
            gram = y * w[:, :, None] * w[:, None]
            _, best = _best_of(gram, w, s)
            in_top = (place < s).view(U * G, P)
            bal, swaps = _balance(gram, w, in_top, case["swaps"])
            ef, geo, steps = _frank_wolfe(x, y, in_top, place.view(U * G, P), s, 64)
            flat_keys = keys.view(U * G, P)
            sets = [torch.gather(flat_keys, 1, q).view(U, G, s) for q in (best, bal, geo)]
            e_top, e_best, e_bal, e_geo = (_set_error(p, v, o, q) for q in [top.sort(2).values] + sets)
            drop = torch.gather(p, 2, order[:, :, s:]).sum(2)
            diam, sigma = dev.max(2).values, (p * dev * dev).sum(2).sqrt()
            ef, steps = ef.view(U, G), steps.view(U, G).double()
            c_hat = torch.where(e_top > 0, 1 - e_best / e_top, 0.0)
            one["stats"].append(torch.stack([
                e_top, e_best, e_bal, _ratio(e_top, e_best), c_hat, _ratio(e_bal, e_best), drop, e_top * (1 - drop),
                diam, sigma, 2 * diam * drop, (drop / (1 - drop)).sqrt() * sigma, ef, e_geo, _ratio(e_best, ef),
                steps], dim=2))
            srt = drop.sort(1).values
            med = (srt[:, (G - 1) // 2] + srt[:, G // 2]) / 2
            one["cell_median"].append(med)
            one["cell_flat"].append((med > 0.25).to(torch.uint8))
            one["pool_idx"].append(pool.int())
            for name, q in zip(("best_idx", "bal_idx", "geo_idx"), sets):
                one[name].append(q.int())
            one["n_swaps"].append(swaps.view(U, G).int())
        parts.append(one)
    out = {}
    for name in parts[0]:
        lists = [torch.cat([one[name][b] for one in parts]) for b in range(len(budgets))]
        out[name] = lists if name.endswith("idx") else torch.stack(lists)
    return out


def _balance(gram, w, member, most):
    """The balancing selector within a pool: final sets (ascending) and swap counts."""
    R, P = w.shape
    member = member.clone()
    swaps = torch.zeros(R, dtype=torch.int64, device="cuda")
    live = torch.ones(R, dtype=torch.bool, device="cuda")
    rows = torch.arange(R, device="cuda")
    diag = torch.diagonal(gram, dim1=1, dim2=2)
    for _ in range(most):
        m = member.double()
        col = torch.matmul(gram, m[:, :, None])[:, :, 0]
        total, mass = (col * m).sum(1), (w * m).sum(1)
        num = (total[:, None, None] - 2 * col[:, :, None] + 2 * col[:, None] + diag[:, :, None] + diag[:, None]
               - 2 * gram)
        val = num.clamp_min(0) / (mass[:, None, None] - w[:, :, None] + w[:, None]) ** 2
        val = val.masked_fill(~(member[:, :, None] & ~member[:, None]), math.inf).view(R, P * P)
        best = val.min(1)
        live &= best.values < total / mass ** 2
        if not live.any():
            break
        i, j = best.indices // P, best.indices % P
        member[rows[live], i[live]] = False
        member[rows[live], j[live]] = True
        swaps += live
    s = int(member[0].sum())
    return member.nonzero()[:, 1].view(R, s), swaps


def _frank_wolfe(x, y, in_top, place, s, most):
    """EF_FW over a pool of deviations x (Gram matrix y), the geometric sets and the steps taken."""
    R, P = in_top.shape
    rows = torch.arange(R, device="cuda")
    w = torch.zeros((R, P), dtype=torch.float64, device="cuda")
    w[rows, torch.diagonal(y, dim1=1, dim2=2).argmin(1)] = 1.0
    steps = torch.zeros(R, dtype=torch.int64, device="cuda")
    live = torch.ones(R, dtype=torch.bool, device="cuda")
    for _ in range(most):
        t = torch.matmul(y, w[:, :, None])[:, :, 0]
        j = t.argmin(1)
        tj, sq = t[rows, j], (t * w).sum(1)
        gap = sq - tj
        live &= (gap > 0) & ~((w[rows, j] == 0) & ((w > 0).sum(1) >= s))
        if not live.any():
            break
        eta = (gap / (sq - 2 * tj + y[rows, j, j])).clamp_max(1.0)
        new = w * (1 - eta)[:, None]
        new[rows, j] += eta
        w = torch.where(live[:, None], new, w)
        steps += live
    ef = torch.matmul(w[:, None], x)[:, 0].norm(dim=1)
    # the support first, then top-mass keys in rank order
    order = torch.where(w > 0, -1, torch.where(in_top, place, 4 * P))
    geo = order.sort(dim=1, stable=True).indices[:, :s].sort(1).values
    return ef, geo, steps


def _exact_vote(case, st):
    s, m, parts = case["s"], case["group"], []
    T = case["G"] // m
    for h in _slices(st, 1 << 25):
        z, p = _weights(st, h)
        v = st["v"][h].double()
        o = torch.matmul(p, v)
        U, G, n = p.shape
        vote = _rank(p.view(U, m, T, n).sum(1))[:, :, :s]
        own = vote[:, None].expand(U, m, T, s).reshape(U, G, s)
        drop = p.scatter(2, own, 0.0).sum(2)
        parts.append(dict(vote_idx=vote.int(), es_vote=_set_error(p, v, o, own),
                          es_top=_set_error(p, v, o, _rank(z)[:, :, :s]), dropped=drop))
    return {k: torch.cat([x[k] for x in parts]) for k in parts[0]}


def _exact_curve(case, st):
    imp = torch.cat([_weights(st, h)[1].mean(1) for h in _slices(st, 1 << 26)])
    srt = imp.sort(dim=1, descending=True, stable=True)
    tail = srt.values.flip(1).cumsum(1).flip(1)
    out = dict(importance=imp, curve=torch.cat([tail, torch.zeros_like(tail[:, :1])], 1))
    if case["order"]:
        out["order"] = srt.indices.int()
    return out


def _exact_compact(case, st):
    H, n, d, floor = case["H"], case["n"], case["d"], case["floor"]
    budget, cap = _alloc(case)
    r = st["score"]
    if case["pool"] > 1:
        half = case["pool"] // 2
        r = torch.nn.functional.max_pool1d(r[:, None], case["pool"], 1, half)[:, 0]
    quota, f = budget - H * min(floor, n), min(floor, n)
    offer = r[:, :n - f].double()
    if cap:
        late = _rank(offer)[:, cap - f:]
        offer = offer.scatter(1, late, -1.0)
    pick = _rank(offer.reshape(-1))[:quota]
    keep = torch.zeros((H, n), dtype=torch.bool, device="cuda")
    keep[:, n - f:] = True
    keep[pick // max(n - f, 1), pick % max(n - f, 1)] = True
    counts = keep.sum(1)
    offsets = torch.cat([counts.new_zeros(1), counts.cumsum(0)])
    pos = keep.nonzero()
    widest = counts.view(-1, case["per_layer"]).max(1).values.sum() * case["per_layer"]
    row = 2 * d * st["k"].element_size()
    tau = offer.reshape(-1)[pick[-1:]] if quota > 0 else torch.full((1,), math.inf, dtype=torch.float64, device="cuda")
    held = torch.stack([counts.sum() * row, widest * row, torch.full_like(widest, H * n * row)])
    return dict(offsets=offsets, kept_pos=pos[:, 1].int(), k_out=st["k"][pos[:, 0], pos[:, 1]],
                v_out=st["v"][pos[:, 0], pos[:, 1]], tau=tau, dropped=r.double().masked_fill(keep, 0.0).sum(1),
                bytes_held=held)


def exact(case, seed):
    if case["kind"] == "subset" and case["H"] * math.comb(case["n"], case["k"]) * case["n"] ** 2 > 3e13:
        return None
    st = prepare(case, seed)
    return {"topk": _exact_topk, "subset": _exact_subset, "swap": _exact_swap, "pool": _exact_pool,
            "vote": _exact_vote, "curve": _exact_curve, "compact": _exact_compact}[case["kind"]](case, st)
