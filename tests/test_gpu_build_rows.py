"""The rows that the library's graph construction writes, edge by edge, against
plain constructions of the same graph: in numpy at sizes around the tiles of the
distance kernels (every list length and attribute type), and in torch, with whole
tables of distances, at sizes above the sample of the thresholds (4,096) and
above what keeps all distances (11,500 points), where the distances come in
panels of 6,144 rows by 6,144 columns and the lists are saved between them. The
vectors are whole numbers, so that every distance is exact in float32 in any
order, and equal distances (many) are decided by id."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PAD = 0xFFFFFFFF
LEVEL_Q = (0.001, 0.01, 0.05, 0.2)


def _prune(D, cand, dists, budget, alpha2):
    kept = []
    for c, du in zip(cand, dists):
        if len(kept) == budget:
            break
        if not any(alpha2 * D[w, c] <= du for w in kept):
            kept.append(c)
    return kept


def _nearest(D, u, ids, K):
    ids = np.asarray([i for i in ids if i != u], dtype=np.int64)
    o = np.lexsort((ids, D[u, ids]))[:K]
    return ids[o], D[u, ids[o]]


def _rows(x, attrs, f32_cols, R, alpha, levels):
    n, m = attrs.shape
    xf = x.astype(np.float64)
    D = ((xf[:, None, :] - xf[None, :, :]) ** 2).sum(-1).astype(np.float32)
    alpha2 = np.float32(alpha) * np.float32(alpha)
    levels = levels if R >= 8 else 0
    b_lvl = max(1, R // 8)
    budget = max(1, R - 1 - levels * b_lvl)
    K = min(2 * R, 128, n - 1)
    everyone = np.arange(n)
    fwd = []
    for u in range(n):
        c, du = _nearest(D, u, everyone, K)
        fwd.append(_prune(D, c, du, budget, alpha2))
    rev = [[] for _ in range(n)]
    for u in range(n):
        for v in fwd[u]:
            rev[v].append(u)
    rows = []
    for u in range(n):
        c, du = _nearest(D, u, sorted(set(fwd[u]) | set(rev[u])), 256)
        rows.append(_prune(D, c, du, budget, alpha2))
    rk = np.empty((n, m), dtype=np.int64)
    for j in range(m):
        col = attrs[:, j].view(np.float32) if j in f32_cols else attrs[:, j]
        rk[:, j] = np.searchsorted(np.sort(col), col, side="left")
    S = min(4096, n)
    smp = (np.arange(S) * n) // S
    for u in range(n):
        gap = np.abs(rk - rk[u]).max(1)
        g = np.sort(gap[smp])
        for q in LEVEL_Q[:levels]:
            t = g[max(0, int(np.ceil(q * S)) - 1)]
            c, du = _nearest(D, u, np.flatnonzero(gap <= t), min(4 * b_lvl, 32, n - 1))
            for v in _prune(D, c, du, b_lvl, alpha2):
                if len(rows[u]) < R - 1 and v not in rows[u]:
                    rows[u].append(v)
    return rows


@pytest.mark.parametrize("n,d,R,m,u8,levels,alpha", [
    (2, 16, 8, 1, True, 4, 1.2), (65, 4, 8, 2, False, 4, 1.2), (128, 20, 16, 3, False, 2, 1.0),
    (129, 48, 16, 2, True, 4, 1.2), (300, 96, 64, 3, False, 4, 1.2), (300, 144, 64, 8, True, 3, 2.0),
    (257, 260, 33, 1, False, 1, 1.2), (500, 32, 7, 2, True, 4, 1.2)])
def test_rows_equal_a_plain_construction(n, d, R, m, u8, levels, alpha):
    import paper_2609_16175_amd as boa
    g = np.random.default_rng(n + d)
    x = (g.integers(0, 4, size=(n, d)) * g.integers(1, 5, size=d)).astype(np.uint8 if u8 else np.float32)
    attrs = g.integers(0, 40, size=(n, m)).astype(np.int32)
    types = np.zeros(m, dtype=np.int32)
    f32_cols = [m - 1] if m > 1 else []
    for j in f32_cols:
        types[j] = boa.ATTR_F32
        attrs[:, j] = np.round(g.normal(size=n), 1).astype(np.float32).view(np.int32)
    ix = boa.Index(x, attrs, types, None, -1, R=R, alpha=alpha, attr_levels=levels)
    adj, _, repaired = ix.graph()
    ix.close()
    extra = 0
    for u, want in enumerate(_rows(x, attrs, f32_cols, R, alpha, levels)):
        got = [int(v) for v in adj[u] if v != PAD]
        assert got[:len(want)] == [int(v) for v in want], (u, got, want)
        extra += len(got) - len(want)
    assert extra == repaired


def _nearest_table(D, allowed, K):
    """(ids, distances) n x K of each row's K nearest allowed columns by
    (distance, id); -1 past their number. allowed(rows): bool per column."""
    import torch
    n = D.shape[0]
    col = torch.arange(n, device=D.device)
    ids, dist = [], []
    for rows in col.split(1024):
        ok = allowed(rows)
        ok[torch.arange(len(rows), device=D.device), rows] = False
        key = torch.where(ok, D[rows].long() << 15 | col, 1 << 62)
        key = torch.topk(key, K, dim=1, largest=False, sorted=True).values
        ids.append(torch.where(key < 1 << 62, key & 32767, -1))
        dist.append((key >> 15).float())
    return torch.cat(ids), torch.cat(dist)


def _prune_table(D, ids, dist, budget, alpha2):
    """Greedy alpha-pruning of every row's candidates (ids n x C, -1 past their
    number, nearest first): bool n x C of the kept ones."""
    import torch
    kept = torch.zeros(ids.shape, dtype=torch.bool, device=D.device)
    step = max(1, (1 << 28) // (ids.shape[1] ** 2))
    for r0 in range(0, len(ids), step):
        c, du, k = ids[r0:r0 + step], dist[r0:r0 + step], kept[r0:r0 + step]
        safe = c.clamp(min=0)
        pair = alpha2 * D[safe[:, :, None], safe[:, None, :]]
        for j in range(c.shape[1]):
            dominated = (k & (pair[:, :, j] <= du[:, j, None])).any(1)
            k[:, j] = (c[:, j] >= 0) & ~dominated & (k.sum(1) < budget)
    return kept


def _rows_table(x, attrs, f32_cols, R, alpha, levels):
    import torch
    dev = torch.device("cuda:0")
    n, m = attrs.shape
    X = torch.from_numpy(x.astype(np.float32)).to(dev)
    D = torch.empty((n, n), dtype=torch.float32, device=dev)
    for r in torch.arange(n, device=dev).split(256):   # (whole numbers below 2^24: exact)
        D[r] = ((X[r][:, None, :] - X[None, :, :]) ** 2).sum(-1)
    alpha2 = float(np.float32(alpha) * np.float32(alpha))
    b_lvl = R // 8
    budget = R - 1 - levels * b_lvl
    everyone = lambda rows: torch.ones((len(rows), n), dtype=torch.bool, device=dev)  # noqa: E731
    ids, dist = _nearest_table(D, everyone, min(2 * R, 128))
    keep = _prune_table(D, ids, dist, budget, alpha2)
    # forward rows and their reverse
    joined = torch.zeros((n, n), dtype=torch.bool, device=dev)
    u = torch.arange(n, device=dev)[:, None].expand_as(ids)[keep]
    joined[u, ids[keep]] = True
    joined |= joined.T.clone()
    most = int(joined.sum(1).max())
    ids, dist = _nearest_table(D, lambda rows: joined[rows].clone(), min(most, 256))
    keep = _prune_table(D, ids, dist, budget, alpha2)
    rows = [c[k].tolist() for c, k in zip(ids.cpu(), keep.cpu())]
    rk = np.empty((n, m), dtype=np.int32)
    for j in range(m):
        col = attrs[:, j].view(np.float32) if j in f32_cols else attrs[:, j]
        rk[:, j] = np.searchsorted(np.sort(col), col, side="left")
    rk = torch.from_numpy(rk).to(dev)
    gap = lambda rows: (rk[rows][:, None, :] - rk[None, :, :]).abs().amax(-1)  # noqa: E731
    S = min(4096, n)
    smp = torch.arange(S, device=dev) * n // S
    srt = torch.cat([gap(r)[:, smp].sort(1).values for r in torch.arange(n, device=dev).split(1024)])
    for q in LEVEL_Q[:levels]:
        t = srt[:, max(0, int(np.ceil(q * S)) - 1)]
        ids, dist = _nearest_table(D, lambda r: gap(r) <= t[r][:, None], min(4 * b_lvl, 32))
        keep = _prune_table(D, ids, dist, b_lvl, alpha2)
        for row, c, k in zip(rows, ids.cpu(), keep.cpu()):
            for v in c[k].tolist():
                if len(row) < R - 1 and v not in row:
                    row.append(v)
    return rows


@pytest.mark.parametrize("n,d,R,m,u8,levels", [
    (5000, 24, 24, 2, False, 4),       # all distances kept, a sample of the points for the thresholds
    (11_585, 16, 16, 1, True, 2),      # just above what is kept: two panels, two chunks of columns
    (12_400, 24, 24, 2, False, 4),     # three of each, 112 rows and columns left over
    (12_400, 32, 32, 3, True, 4),
    (18_500, 16, 64, 1, False, 3)])    # four of each, lists of 128
def test_large_rows_equal_a_plain_construction(n, d, R, m, u8, levels):
    import torch

    import paper_2609_16175_amd as boa
    g = np.random.default_rng(n + d)
    x = (g.integers(0, 4, size=(n, d)) * g.integers(1, 5, size=d)).astype(np.uint8 if u8 else np.float32)
    attrs = g.integers(0, 5000, size=(n, m)).astype(np.int32)
    types = np.zeros(m, dtype=np.int32)
    f32_cols = [m - 1] if m > 1 else []
    for j in f32_cols:
        types[j] = boa.ATTR_F32
        attrs[:, j] = np.round(g.normal(size=n), 3).astype(np.float32).view(np.int32)
    ix = boa.Index(x, attrs, types, None, -1, R=R, attr_levels=levels)
    adj, _, repaired = ix.graph()
    ix.close()
    extra = 0
    for u, want in enumerate(_rows_table(x, attrs, f32_cols, R, 1.2, levels)):
        got = [int(v) for v in adj[u] if v != PAD]
        assert got[:len(want)] == want, (u, got, want)
        extra += len(got) - len(want)
    assert extra == repaired
    torch.cuda.empty_cache()
