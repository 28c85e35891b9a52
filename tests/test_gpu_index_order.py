"""The order of the retrieved tokens: those above the threshold bin ascending, then the admitted ones of that bin best first.  The
edges of the bins are single-precision arithmetic on the score bounds and 1024 sampled scores, repeated here in numpy, so that the
output is compared position by position."""
import numpy as np
import pytest
import torch

import oracle
from paper_2407_12820_amd import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
F = np.float32
FINE, HIGH, SAMPLE_BINS = 1791, 256, 256


@pytest.fixture(scope="module")
def pqc():
    from paper_2407_12820_amd import binding
    binding.load()
    return binding


def _w(**kw):
    base = dict(name="order", batch=1, n_q_heads=2, n_kv_heads=2, head_dim=128, n_tokens=131072, pq_m=4, pq_centroids=256,
                topk=13107, n_init=4, n_local=64, dtype="f32", kmeans_iters=1, recipe="plain")
    base.update(kw)
    return wl.Workload(**base)


def _sampled(w):
    nmid = w.n_tokens - w.n_init - w.n_local
    n = min(nmid, 1024)
    return w.n_init + (np.arange(n, dtype=np.int64) * nmid) // n


def _layout(w, scores, lo, hi):
    """(c0, slope, c1, slope above it) from the score bounds and the scores of the sampled tokens."""
    s = scores[_sampled(w)]
    nmid, n = w.n_tokens - w.n_init - w.n_local, len(s)
    pr = w.topk / nmid
    centre, hw = pr * n, 5.0 * np.sqrt(n * pr * (1.0 - pr)) + 2.0
    rank_hi, rank_lo = int(np.floor(centre - hw)), int(np.ceil(centre + hw))
    width = F(hi) - F(lo)
    in_range = lambda x: 1e-30 < x < 3e38
    scale = F(SAMPLE_BINS) / width if in_range(width) else F(0)
    counts = np.bincount(np.clip(((s - lo) * scale).astype(np.int64), 0, SAMPLE_BINS - 1), minlength=SAMPLE_BINS)
    reached = np.cumsum(counts[::-1])  # samples in the bins from the top one down
    bin_of = lambda rank: SAMPLE_BINS - 1 - int(np.searchsorted(reached, rank))
    wu = width * F(1.0 / SAMPLE_BINS)
    edge = lambda b: F(np.float64(b) * np.float64(wu) + np.float64(lo))  # a fused multiply-add
    q_hi = hi if rank_hi < 1 else edge(bin_of(rank_hi) + 1)
    q_lo = lo if rank_lo > n else edge(bin_of(rank_lo))
    c0, c1 = max(F(lo), q_lo), min(F(hi), q_hi)
    if not c1 > c0:
        c0, c1 = F(lo), F(hi)
    slope = lambda bins, x: F(bins) / x if in_range(x) else F(0)
    return c0, slope(FINE, c1 - c0), c1, slope(HIGH, F(hi) - c1)


def _bins(s, layout):
    c0, ic, c1, ih = layout
    fine = 1 + np.minimum(((s - c0) * ic).astype(np.int64), FINE - 1)
    high = 1 + FINE + np.minimum(((s - c1) * ih).astype(np.int64), HIGH - 1)
    return np.where(s < c0, 0, np.where(s > c1, high, fine))


def _expected(w, scores, lo, hi):
    I, K, N, L = w.n_init, w.topk, w.n_tokens, w.n_local
    mid = np.arange(I, N - L)
    s = scores[mid]
    bins = _bins(s, _layout(w, scores, lo, hi))
    kth = np.sort(bins)[len(bins) - K]
    above, at = mid[bins > kth], mid[bins == kth]
    best = at[np.lexsort((at, -scores[at]))][:K - len(above)]
    return np.concatenate([np.arange(I), above, best, np.arange(N - L, N)])


@pytest.mark.parametrize("n_tokens, topk", [(131072, 13107), (32768, 6553), (20011, 2001), (5003, 500)])
def test_scores_at_the_edges_of_bins(pqc, n_tokens, topk):
    # half of the scores inside the window are moved to the first value of a bin or the last one of the bin below it
    w = _w(n_tokens=n_tokens, topk=topk, n_q_heads=6, n_kv_heads=6)
    rng = np.random.default_rng(n_tokens)
    scores = rng.standard_normal((1, 6, n_tokens)).astype(F)
    scores[0, 2] += F(20.0)
    scores[0, 3] *= F(1e-4)
    scores[0, 4] *= F(37.5)
    want = []
    for g in range(6):
        s = scores[0, g]
        m = slice(w.n_init, n_tokens - w.n_local)
        lo, hi = s[m].min(), s[m].max()
        c0, ic, c1, _ = layout = _layout(w, s, lo, hi)
        inside = (s > c0) & (s < c1) & (rng.random(n_tokens) < 0.5) & ~np.isin(np.arange(n_tokens), _sampled(w))
        b = _bins(s[inside], layout)
        first = (np.float64(c0) + (b - 1) / np.float64(ic)).astype(F)
        for _ in range(64):  # to the lowest value of the bin
            down = np.nextafter(first, F(-np.inf))
            first = np.where(_bins(first, layout) < b, np.nextafter(first, F(np.inf)), np.where(_bins(down, layout) >= b, down, first))
        assert (_bins(first, layout) == b).all() and (_bins(np.nextafter(first, F(-np.inf)), layout) < b).all()
        s[inside] = np.where(rng.random(len(b)) < 0.5, first, np.nextafter(first, F(-np.inf)))
        want.append(_expected(w, s, lo, hi))
    print(f"[case] scores at edges n={n_tokens}", flush=True)
    got = pqc.PQCache(w, DEV).topk(torch.from_numpy(scores).to(DEV)).cpu().numpy()
    np.testing.assert_array_equal(got[0], np.stack(want))


@pytest.mark.parametrize("kw", [dict(n_tokens=60001, topk=6000, n_kv_heads=16), dict(n_tokens=12289, topk=1200, pq_centroids=64, n_kv_heads=16),
                                dict(n_tokens=7001, topk=1400, pq_centroids=64, n_kv_heads=32), dict(n_tokens=30001, topk=3000, pq_m=2, n_kv_heads=8),
                                dict(n_tokens=9003, topk=900, pq_m=2, pq_centroids=48, n_kv_heads=8), dict(n_tokens=30001, topk=6000, pq_m=2, pq_centroids=64, n_kv_heads=8),
                                dict(n_tokens=11003, topk=1100, pq_m=2, pq_centroids=48, n_kv_heads=8), dict(n_tokens=20002, topk=2000, pq_m=8),
                                dict(n_tokens=60001, topk=6000, pq_m=2, pq_centroids=64, n_kv_heads=8)],
                         ids=lambda kw: ",".join(f"{k}={v}" for k, v in kw.items()))
def test_decode(pqc, kw):
    w = _w(n_q_heads=kw.get("n_kv_heads", 2), **kw)
    H, N, M, C = w.n_kv_heads, w.n_tokens, w.pq_m, w.pq_centroids
    gen = torch.Generator(device=DEV)
    gen.manual_seed(N)
    q, k, v = (torch.randn(s, generator=gen, device=DEV) for s in ((1, H, 128), (1, H, N, 128), (1, H, N, 128)))
    cent = torch.randn((1, H, M, C, 128 // M), generator=gen, device=DEV)
    codes = torch.randint(0, C, (1, H, N, M), generator=gen, device=DEV, dtype=torch.uint8)
    print(f"[case] order of a step {w}", flush=True)
    ctx = pqc.PQCache(w, DEV)
    idx, _ = ctx.decode(q, cent, codes, k, v)
    table = ctx.lut(q, cent).cpu().numpy()
    scores, _ = oracle.scores(q.cpu().numpy(), "f32", cent.cpu().numpy(), codes.cpu().numpy())
    for g in range(H):
        lo, hi = F(0), F(0)
        for j in range(M):  # bounds are added in the order of a score's terms
            lo, hi = lo + table[0, g, j].min(), hi + table[0, g, j].max()
        np.testing.assert_array_equal(idx[0, g].cpu().numpy(), _expected(w, scores[0, g], lo, hi))
