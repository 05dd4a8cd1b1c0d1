"""Performance cases: batched filtered searches and index builds through the
public binding (paper_2609_16175_amd.Index), over the sizes, data types,
options and entry points a program uses.

A case is a dict of plain values. Search cases hold a resident index and a
batch of device queries with their ranges; build cases hold host arrays and
run the whole construction. Inputs are Gaussian mixtures of low intrinsic
dimension with range attributes (the recipes of workloads/gen.py), drawn and
linked on the GPU so that they are made quickly.
"""
import math

import numpy as np
import torch

import paper_2609_16175_amd as boa

PAD = 0xFFFFFFFF


def _search(name, **kw):
    case = dict(op="search", name=name, u8=False, integer=False, attrs="uniform", sel=0.1, k=10, L0=16, Lmax=512,
                alpha=2.0, eps=0.05, mode="phased", pq=0, no_alloc=False, counters=False, esc=1.0)
    case.update(kw)
    return case


def _build(name, **kw):
    case = dict(op="build", name=name, u8=False, integer=False, attrs="uniform", sel=0.1, nq=1)
    case.update(kw)
    return case


# esc: share of the queries that go past the first width (work() counts with
# it; measured once per recipe, no search reads it).
def listed():
    return [
        # one interactive request to a small collection, default arguments
        _search("request-1", n=10_000, d=32, R=16, m=1, clusters=16, attrs="tiny", sel=0.5, nq=1, Lmax=128),
        # a small batch on the small collection, survivors in a launch of their own
        _search("tiny-100-split", n=10_000, d=32, R=16, m=1, clusters=16, attrs="tiny", sel=0.5, nq=100, Lmax=128,
                alpha=32.0, eps=0.001, mode="split", counters=True),
        # a serving loop that may not allocate: 64 uint8 queries with a warm start
        _search("serve-64-noalloc", n=100_000, d=128, u8=True, R=32, m=2, clusters=100, nq=64, alpha=32.0, eps=0.005,
                mode="warm", no_alloc=True),
        # descriptor search, a full batch; nearly every query settles at the first width
        _search("sift-split", n=1_000_000, d=128, integer=True, R=64, m=2, clusters=1000, sel=0.0, nq=10_000, alpha=32.0,
                eps=0.2, mode="split", esc=0.02),
        # image features, three typed attributes, one launch per width
        _search("deep-phased", n=500_000, d=96, R=64, m=3, clusters=500, attrs="mixed", sel=0.05, nq=5_000,
                counters=True, esc=0.5),
        # the largest index and batch: uint8 descriptors, nearly every query escalates
        _search("u8-warm", n=10_000_000, d=128, u8=True, R=32, m=2, clusters=10_000, nq=10_000, alpha=32.0, eps=0.005,
                mode="warm"),
        # text embeddings under attributes that follow the clusters, phases overlapped on two streams
        _search("dblp-plus", n=300_000, d=768, R=48, m=4, clusters=600, attrs="cluster", sel=0.01, nq=2_000, Lmax=1024,
                mode="plus", esc=0.2),
        # the same embeddings traversed by product-quantised codes with an exact re-rank
        _search("dblp-pq", n=300_000, d=768, R=48, m=4, clusters=600, attrs="cluster", sel=0.01, nq=2_000, Lmax=1024,
                alpha=32.0, eps=0.005, mode="warm", pq=192, esc=0.75),
        # a fixed wide beam over odd sizes, the non-adaptive baseline
        _search("fixed-ragged", n=234_567, d=100, R=50, m=5, clusters=234, sel=0.1, nq=777, k=17, mode="fixed",
                Lmax=500),
        # index construction on the GPU: float32 with typed attributes, uint8, wide float32 rows
        _build("build-f32", n=30_000, d=96, R=64, m=3, clusters=30, attrs="mixed"),
        _build("build-u8", n=60_000, d=128, u8=True, R=32, m=2, clusters=60),
        _build("build-wide", n=10_007, d=768, R=48, m=4, clusters=20, attrs="cluster"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "f32", "f32", "u8", "u8", "wide", "pq", "build"])
    m = rng.randint(1, 8)
    mode = rng.choice(["phased", "fused", "warm", "split", "plus", "fixed"])
    common = dict(m=m, k=rng.randint(1, 16), attrs=rng.choice(["uniform", "mixed"]) if m >= 3 else "uniform",
                  sel=rng.choice([0.01, 0.05, 0.1, 0.5]), mode=mode, alpha=rng.choice([2.0, 4.0, 32.0]),
                  eps=rng.choice([0.005, 0.05, 0.2]), counters=rng.random() < 0.3,
                  no_alloc=mode != "plus" and rng.random() < 0.2)
    if kind == "build":
        u8 = rng.random() < 0.5
        c = _build("", n=_log(rng, 3_000, 40_000), d=16 * rng.randint(2, 12) if u8 else 4 * rng.randint(6, 40), u8=u8,
                   R=rng.randint(12, 64), m=m, attrs=common["attrs"])
    elif kind == "small":
        c = _search("", n=_log(rng, 5_000, 50_000), d=4 * rng.randint(4, 32), R=rng.randint(12, 48), nq=_log(rng, 1, 500),
                    Lmax=_log(rng, 32, 256), **common)
    elif kind == "f32":
        c = _search("", n=_log(rng, 50_000, 300_000), d=4 * rng.randint(16, 64), integer=rng.random() < 0.5,
                    R=rng.randint(24, 64), nq=_log(rng, 100, 3_000), Lmax=_log(rng, 64, 512), **common)
    elif kind == "u8":
        c = _search("", n=_log(rng, 50_000, 1_000_000), d=16 * rng.randint(2, 16), u8=True, R=rng.randint(16, 64),
                    nq=_log(rng, 100, 5_000), Lmax=_log(rng, 64, 512), **common)
    elif kind == "wide":
        c = _search("", n=_log(rng, 30_000, 100_000), d=64 * rng.randint(5, 16), R=rng.randint(24, 64),
                    nq=_log(rng, 100, 1_000), Lmax=_log(rng, 64, 1024), **common)
    else:
        pq = 2 * rng.randint(8, 96)
        c = _search("", n=_log(rng, 30_000, 100_000), d=4 * pq, pq=pq, R=rng.randint(24, 64), nq=_log(rng, 100, 1_000),
                    Lmax=_log(rng, 64, 1024), **common)
    c["clusters"] = max(4, c["n"] // 1000)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs

def _mixture(case, gen, dev):
    """(vectors, cluster of each point, queries, cluster of each query):
    cluster centres in an 8-dimensional subspace, 99% of the noise on 8
    directions of each cluster (isotropic for the small recipe)."""
    n, d, C, nq = case["n"], case["d"], case["clusters"], case["nq"]
    S = -(-n // C)
    normal = lambda *s: torch.randn(*s, generator=gen, device=dev)  # noqa: E731
    tiny = case["attrs"] == "tiny"
    ints = case["u8"] or case["integer"]
    if tiny:
        centre = normal(C, d)
    else:
        centre = normal(C, 8) @ normal(8, d)
        centre *= 1.0 / centre.std()
    axes = normal(C, 8, d) / math.sqrt(8)
    sigma = 0.3 if tiny else (0.5 if ints else 0.2)

    def rows(c, per):   # `per` rows of each cluster c
        iso = normal(len(c), per, d)
        x = iso if tiny else 0.1 * iso + 0.995 * (normal(len(c), per, 8) @ axes[c])
        x = centre[c][:, None, :] + sigma * x
        if ints:
            return (128 + 40 * x).round_().clamp_(0, 255)
        return x if tiny else x / x.norm(dim=-1, keepdim=True)

    at = torch.randperm(n, generator=gen, device=dev)   # id of the i-th row made
    x = torch.empty(n, d, dtype=torch.uint8 if case["u8"] else torch.float32, device=dev)
    cid = torch.empty(n, dtype=torch.int64, device=dev)
    step = max(1, (1 << 26) // (S * d))
    for c0 in range(0, C, step):
        c = torch.arange(c0, min(C, c0 + step), device=dev)
        part = rows(c, S).reshape(-1, d)
        i0 = c0 * S
        part = part[:max(0, n - i0)]
        where = at[i0:i0 + len(part)]
        x[where] = part.to(x.dtype)
        cid[where] = c.repeat_interleave(S)[:len(part)]
    qc = torch.randint(0, C, (nq,), generator=gen, device=dev)
    q = torch.cat([rows(qc[i:i + 4096], 1)[:, 0] for i in range(0, nq, 4096)]).to(x.dtype)
    return x, cid, q, qc


def _attributes(case, cid, qc, gen, dev):
    """(attribute cells n x m, types, ranges nq x m x 2) as int32 cells."""
    n, m, C, nq = case["n"], case["m"], case["clusters"], case["nq"]
    kind = case["attrs"]
    cells, types, ranges = [], [], []
    sel = torch.full((nq,), case["sel"], device=dev, dtype=torch.float64)
    if case["sel"] == 0.0:   # each query draws its joint selectivity
        sel = torch.tensor([0.5, 0.1, 0.01], device=dev, dtype=torch.float64)[
            torch.randint(0, 3, (nq,), generator=gen, device=dev)]
    free = m - 2 if kind == "cluster" else m
    frac = sel ** (1.0 / max(1, free)) if kind != "cluster" else sel.clamp(min=0.1) ** (1.0 / max(1, free))
    for j in range(m):
        if kind == "cluster" and j < 2:   # follows the cluster; the window holds the query's own
            col = cid + torch.randint(0, 100, (n,), generator=gen, device=dev)
            width = max(130, 3 * C // 20)
            lo = (qc - torch.randint(0, width - 99, (nq,), generator=gen, device=dev)).clamp(min=0)
            cells.append(col.int())
            types.append(0)
            ranges.append(torch.stack([lo, lo + width - 1], 1).int())
            continue
        as_float = kind == "mixed" and j == 2
        if as_float:
            col = torch.rand(n, generator=gen, device=dev)
        elif kind == "mixed" and j == 1:   # Zipf(1.1) over 0..999
            p = torch.arange(1, 1001, device=dev, dtype=torch.float64) ** -1.1
            cdf = (p / p.sum()).cumsum(0)
            col = torch.searchsorted(cdf, torch.rand(n, generator=gen, device=dev, dtype=torch.float64)).clamp(max=999).int()
        else:
            col = torch.randint(0, 1000 if kind == "tiny" else 10_000, (n,), generator=gen, device=dev).int()
        s = col.sort().values
        u = torch.rand(nq, generator=gen, device=dev, dtype=torch.float64) * (1 - frac)
        lo = s[(u * n).long().clamp(0, n - 1)]
        hi = s[((u + frac) * n).long().clamp(0, n - 1)]
        r = torch.stack([lo, hi], 1)
        cells.append(col.view(torch.int32) if as_float else col)
        ranges.append(r.view(torch.int32) if as_float else r)
        types.append(1 if as_float else 0)
    return torch.stack(cells, 1).contiguous(), types, torch.stack(ranges, 1).contiguous()


def _nearest_in_blocks(x, order, B, t):
    """For each point, its t nearest among the B points of its block of `order`."""
    n, dev = len(order), x.device
    B = max(2, min(B, n))
    t = min(t, B - 1)
    nb = -(-n // B)
    full = torch.cat([order, order[:nb * B - n]]).view(nb, B)
    out = torch.empty(n, t, dtype=torch.int64, device=dev)
    step = max(1, (1 << 27) // (B * max(B, x.shape[1])))
    for b0 in range(0, nb, step):
        ids = full[b0:b0 + step]
        y = x[ids].float()
        dist = (y * y).sum(-1)[:, None, :] - 2 * torch.bmm(y, y.transpose(1, 2).contiguous())
        dist.masked_fill_(ids[:, :, None] == ids[:, None, :], float("inf"))
        near = dist.topk(t, dim=-1, largest=False).indices
        got = ids.gather(1, near.reshape(len(ids), -1)).view(len(ids), B, t)
        keep = (torch.arange(len(ids) * B, device=dev) + b0 * B < n).view(len(ids), B)
        out[ids[keep]] = got[keep]
    return out


def _graph(case, x, cid, cells, gen):
    """n x R rows: near and spread neighbours of the own cluster, members of
    the nearest clusters, neighbours close in an attribute too, neighbours in
    random subsets of a few sizes (which span the data), and one free slot."""
    n, R, C, dev = case["n"], case["R"], case["clusters"], x.device
    perm = lambda: torch.randperm(n, generator=gen, device=dev)  # noqa: E731
    p = perm()
    by_cluster = p[cid[p].sort(stable=True).indices]
    size = -(-n // C)                      # (all clusters but the last are this large)
    share = lambda f: max(1, round(R * f))  # noqa: E731
    parts = [_nearest_in_blocks(x, by_cluster, size, share(0.34)), _nearest_in_blocks(x, by_cluster, max(8, size // 8), share(0.1))]
    members = torch.cat([by_cluster, by_cluster[-1:].expand(-n % size)]).view(-1, size)
    mean = torch.cat([x[i].float().mean(1) for i in members.split(max(1, (1 << 25) // (size * case["d"])))])
    gap = torch.cdist(mean, mean)
    gap.fill_diagonal_(float("inf"))
    close = gap.topk(min(8, len(mean) - 1), largest=False).indices
    t = share(0.1)
    other = close[cid[:, None].clamp(max=len(mean) - 1), torch.randint(0, close.shape[1], (n, t), generator=gen, device=dev)]
    parts.append(by_cluster[(other * size + torch.randint(0, size, (n, t), generator=gen, device=dev)).clamp(max=n - 1)])
    for j in range(min(2, case["m"])):
        rank = torch.empty_like(p)
        rank[cells[:, j].sort(stable=True).indices] = torch.arange(n, device=dev)
        bucket = rank * max(1, size // 16) // n
        parts.append(_nearest_in_blocks(x, (bucket * C + cid).sort(stable=True).indices, 256, share(0.12)))
    parts += [_nearest_in_blocks(x, perm(), B, share(0.04)) for B in (512, 64, 8)]
    rows = torch.cat(parts, 1)[:, :max(1, R - 1)]
    rows = torch.where(rows == torch.arange(n, device=dev)[:, None], rows[:, :1], rows).sort(1).values
    rows[:, 1:][rows[:, 1:] == rows[:, :-1]] = -1
    adj = torch.full((n, R), -1, dtype=torch.int32, device=dev)
    adj[:, :rows.shape[1]] = rows.int()
    return adj


def _entry(x):
    """The point nearest the centroid (float64)."""
    mean = sum(p.double().sum(0) for p in x.split(1 << 18)) / len(x)
    return int(torch.cat([(p.double() - mean).square().sum(1) for p in x.split(1 << 18)]).argmin())


def _codes(x, M, gen):
    """4-bit product quantisation: (codebook M x 16 x ds, centroid of each
    point and subspace n x M); 3 rounds of k-means on a sample."""
    n, d = x.shape
    y = x.float().view(n, M, d // M)
    s = y[torch.randint(0, n, (8192,), generator=gen, device=x.device)]
    cb = s[:16].transpose(0, 1).contiguous()
    nearest = lambda z: (z[:, :, None, :] - cb[None]).square().sum(-1).argmin(-1)  # noqa: E731
    for _ in range(3):
        one = torch.nn.functional.one_hot(nearest(s), 16).float()            # s x M x 16
        count = one.sum(0)
        sums = torch.bmm(one.permute(1, 2, 0).contiguous(), s.transpose(0, 1).contiguous())
        cb = torch.where(count[..., None] > 0, sums / count[..., None].clamp(min=1), cb)
    return cb, torch.cat([nearest(z) for z in y.split(4096)])


def _inputs(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    x, cid, q, qc = _mixture(case, gen, dev)
    cells, types, ranges = _attributes(case, cid, qc, gen, dev)
    if case["op"] == "build":
        return x, cells, types
    adj = _graph(case, x, cid, cells, gen)
    pq = _codes(x, case["pq"], gen) if case["pq"] else None
    return x, cells, types, adj, _entry(x), q, ranges, pq


def prepare(case, seed):
    got = _inputs(case, seed)
    if case["op"] == "build":
        x, cells, types = got
        return dict(op="build", R=case["R"], x=x.cpu().numpy(), cells=cells.cpu().numpy(),
                    types=np.array(types, dtype=np.int32))
    x, cells, types, adj, entry, q, ranges, pq = got
    ix = boa.Index(x.cpu().numpy(), cells.cpu().numpy(), np.array(types, dtype=np.int32),
                   adj.cpu().numpy().view(np.uint32), entry)
    if pq is not None:
        codes = (pq[1][:, 0::2] | (pq[1][:, 1::2] << 4)).to(torch.uint8)
        ix.set_pq(pq[0].cpu().numpy(), codes.cpu().numpy())
    mode = case["mode"]
    kw = dict(k=case["k"], L0=case["L0"], Lmax=case["Lmax"], alpha=case["alpha"], eps=case["eps"],
              fixed_L=case["Lmax"] if mode == "fixed" else 0, fused=mode in ("fused", "warm"), split=mode == "split",
              warm=mode == "warm", boa_plus=mode == "plus", pq=case["pq"] > 0, counters=case["counters"],
              no_alloc=case["no_alloc"])
    if case["no_alloc"]:   # such a program keeps its output buffers too
        new = lambda *s, t=torch.int32: torch.zeros(*s, dtype=t, device=q.device)  # noqa: E731
        nq, k, n_ = case["nq"], case["k"], case["counters"]
        kw["out"] = (new(nq, k), new(nq, k, t=torch.float32), new(nq), new(nq) if n_ else None, new(nq) if n_ else None)
    return dict(op="search", ix=ix, q=q, ranges=ranges, kw=kw)


def run(state):
    if state["op"] == "build":
        ix = boa.Index(state["x"], state["cells"], state["types"], None, -1, R=state["R"])
        adj, entry, repaired = ix.graph()
        ix.close()
        return dict(adjacency=adj.view(np.int32), entry=entry, repaired=repaired)
    r = state["ix"].search(state["q"], state["ranges"], **state["kw"])
    out = dict(ids=r.ids, dists=r.dists, final_L=r.final_L)
    if r.expansions is not None:
        out.update(expansions=r.expansions, scored=r.scored)
    return out


def _widths(case):
    if case["mode"] == "fixed":
        return [case["Lmax"]]
    L = [case["L0"]]
    while L[-1] < case["Lmax"]:
        L.append(min(math.ceil(case["alpha"] * L[-1]), case["Lmax"]))
    return L


def work(case):
    """Search: a beam of width L expands about L + 10 nodes and scores about
    0.4 R new ones for each; a row, an attribute record and a vector (or code)
    are read for each once, in the widest phase a query reaches. Build: every
    pair's distance once."""
    n, d, R, m = case["n"], case["d"], case["R"], case["m"]
    e = 1 if case["u8"] else 4
    if case["op"] == "build":
        return dict(bytes=n * (d * e + 4 * m + 4 * R), flops=2.0 * n * n * d)
    w = _widths(case)
    L = w[0] if len(w) == 1 else case["esc"] * w[-1] + (1 - case["esc"]) * w[0]
    exp = case["nq"] * min(n, L + 10)
    scored = min(0.4 * R * exp, case["nq"] * n)
    per = 4 * m + (case["pq"] // 2 if case["pq"] else d * e)
    return dict(bytes=exp * 4 * R + scored * per + case["nq"] * (d * e + 8 * m + 8 * case["k"] + 4),
                flops=scored * (case["pq"] if case["pq"] else 3 * d))


def tolerance(case):
    # ids, widths and counts are whole numbers; distances have one documented
    # summation order (include/boa.h), so every correct search gives their bits
    return "exact"


# ---------------------------------------------------------------------------
# the search in plain torch and 64 bits: batched over queries, one expansion
# per step

def exact(case, seed):
    if case["op"] == "build":
        return None   # whole numbers only
    w = _widths(case)
    steps = case["nq"] * (w[0] + case["esc"] * (sum(w[1:]) if case["mode"] != "warm" else w[-1])) * (w[-1] + case["R"])
    if steps > 2.5e9:
        return None
    x, cells, types, adj, entry, q, ranges, pq = _inputs(case, seed)
    dev, n, k, nq = x.device, case["n"], case["k"], case["nq"]
    as_float = torch.tensor([t == 1 for t in types], device=dev)
    val = torch.where(as_float, cells.view(torch.float32).double(), cells.double())
    lo = torch.where(as_float, ranges[..., 0].contiguous().view(torch.float32).double(), ranges[..., 0].double())
    hi = torch.where(as_float, ranges[..., 1].contiguous().view(torch.float32).double(), ranges[..., 1].double())
    rows = adj.long()
    qd = q.double()
    if pq is not None:
        M = case["pq"]
        table = (qd.view(nq, M, 1, -1) - pq[0].double()[None]).square().sum(-1)   # nq x M x 16

    def true_dist(qi, ids):
        return (x[ids].double() - qd[qi][:, None, :]).square().sum(-1)

    def dist(qi, ids):
        if pq is None:
            return true_dist(qi, ids)
        c = pq[1][ids]                                                            # b x r x M
        return table[qi].transpose(1, 2).gather(1, c).sum(-1)

    out_ids = torch.full((nq, k), -1, dtype=torch.int32, device=dev)
    out_d = torch.full((nq, k), float("inf"), dtype=torch.float64, device=dev)
    out_L = torch.zeros(nq, dtype=torch.int32, device=dev)
    E = torch.zeros(nq, dtype=torch.int64, device=dev)
    S = torch.zeros(nq, dtype=torch.int64, device=dev)
    FAR = (1 << 62) + 1

    def score(qi, ids):   # keys: violations, then the distance's bits
        phi = ((val[ids] < lo[qi][:, None, :]) | (val[ids] > hi[qi][:, None, :])).sum(-1)
        return (phi << 58) | (dist(qi, ids).view(torch.int64) >> 5)

    def chunk(c):
        live, carried = c, None
        for p, L in enumerate(w):
            b = len(live)
            warm = case["mode"] == "warm" and p > 0
            cap = w[p + 1] if case["mode"] == "warm" and p + 1 < len(w) else L
            ar = torch.arange(b, device=dev)
            if warm:
                seen, ids, key, done = carried
            else:
                seen = torch.zeros(b, n + 1, dtype=torch.bool, device=dev)
                seen[:, entry] = True
                seen[:, n] = True
                ids = torch.full((b, 1), entry, device=dev)
                key, done = score(live, ids), torch.zeros(b, 1, dtype=torch.bool, device=dev)
                S[live] += 1
            while True:
                open_ = ~done[:, :L] & (key[:, :L] < FAR)
                some = open_.any(1)
                if not bool(some.any()):
                    break
                j = open_.to(torch.uint8).argmax(1)
                done[ar[some], j[some]] = True
                E[live[some]] += 1
                new = rows[ids[ar, j].clamp(max=n - 1)]
                new = torch.where((new < 0) | ~some[:, None], n, new)
                fresh = ~seen.gather(1, new)
                seen.scatter_(1, new, True)
                S[live] += fresh.sum(1)
                nk = torch.where(fresh, score(live, new.clamp(max=n - 1)), FAR)
                ids, key = torch.cat([ids, new], 1), torch.cat([key, nk], 1)
                done = torch.cat([done, torch.zeros_like(fresh)], 1)
                o = ids.sort(dim=1, stable=True).indices
                o = o.gather(1, key.gather(1, o).sort(dim=1, stable=True).indices)[:, :cap]
                ids, key, done = ids.gather(1, o), key.gather(1, o), done.gather(1, o)
            wide = min(L, key.shape[1])
            ok = key[:, :wide] < (1 << 58)
            d64 = torch.where(ok, true_dist(live, ids[:, :wide].clamp(max=n - 1)), math.inf)
            o = ids[:, :wide].sort(dim=1, stable=True).indices
            o = o.gather(1, d64.gather(1, o).sort(dim=1, stable=True).indices)
            d64, top = d64.gather(1, o), ids[:, :wide].gather(1, o)
            count = ok.sum(1)
            root = d64.sqrt()
            dmax = root.gather(1, (count - 1).clamp(min=0)[:, None])[:, 0]
            dk = root[:, k - 1] if wide >= k else torch.full((b,), math.inf, device=dev, dtype=torch.float64)
            gap = torch.where(dmax == 0, 0.0, (dmax - dk) / dmax)
            end = ((count > k) & (gap <= case["eps"])) | (p + 1 == len(w))
            t = min(k, wide)
            out_ids[live[end], :t] = torch.where(d64[end, :t] < math.inf, top[end, :t], -1).int()
            out_d[live[end], :t] = d64[end, :t]
            out_L[live[end]] = L
            stay = ~end
            if not bool(stay.any()):
                return
            carried = (seen[stay], ids[stay], key[stay], done[stay])
            live = live[stay]

    per = max(1, min(nq, (1 << 33) // (n + 1), (1 << 28) // (case["R"] * case["d"])))
    for c in torch.arange(nq, device=dev).split(per):
        chunk(c)
    out = dict(ids=out_ids, dists=out_d, final_L=out_L)
    if case["counters"]:
        out.update(expansions=E.int(), scored=S.int())
    return out
