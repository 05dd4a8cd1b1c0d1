"""The rows that the library's graph construction writes, edge by edge, against
a plain numpy construction of the same graph: sizes around the tiles of the
distance kernels and the sample of the thresholds, every list length and
attribute type. The vectors are whole numbers, so that every distance is exact
in float32 in any order, and equal distances (many) are decided by id."""
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
