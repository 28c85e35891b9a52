"""GPU parity of PQ construction (K-Means) and of the appended-token code against the oracle.

The GPU evaluates distances in fp32, the oracle in double, so a code may legitimately
differ where a token is (nearly) equidistant from two centroids: a differing code is
accepted only if the oracle's distances to the two centroids agree within 1e-5 relative.
Centroid means are compared with a tolerance that covers the 2^-20 fixed-point grid."""
import numpy as np
import pytest
import torch

import oracle
from paper_2407_12820_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def pqc():
    from paper_2407_12820_amd import binding
    binding.load()
    return binding


def _codes_agree(keys_f32, cent, codes_gpu, codes_ref, M):
    """All differing codes must be near-ties in the oracle's metric. Returns their count."""
    B, Hkv, N, D = keys_f32.shape
    Dm = D // M
    diff = np.argwhere(codes_gpu != codes_ref)
    for b, g, t, j in diff:
        x = keys_f32[b, g, t, j * Dm:(j + 1) * Dm].astype(np.float64)
        da = ((x - cent[b, g, j, codes_gpu[b, g, t, j]].astype(np.float64)) ** 2).sum()
        db = ((x - cent[b, g, j, codes_ref[b, g, t, j]].astype(np.float64)) ** 2).sum()
        assert abs(da - db) <= 1e-5 * max(da, db), (b, g, t, j, da, db)
    return len(diff)


CASES = {
    "tiny_f32": dict(n_tokens=1500),
    "llama8b_32k": dict(n_tokens=3001),
    "batch8_32k": dict(batch=2, n_tokens=2500),
}


@pytest.mark.parametrize("name", list(CASES))
def test_assign_and_one_update_match_oracle(pqc, name):
    w = wl.get(name, **CASES[name])
    print(f"[case] pq assign/update {w}", flush=True)
    d = wl.generate(w, seed=11)
    init = wl.kmeans_init_indices(w, seed=11)
    kf = wl.to_f32(d["k"], w.dtype)
    keys = pqc.to_device(d["k"], w.dtype, DEV)
    init_d = torch.from_numpy(init).to(DEV)
    # zero iterations: centroids are the sampled sub-vectors, codes their nearest centroids
    c0_ref, cd0_ref, _ = oracle.pq_build(d["k"], w.dtype, w.pq_m, w.pq_centroids, 0, init)
    c0, cd0 = pqc.pq_build(w, keys, init_d, iters=0)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(c0.cpu().numpy(), c0_ref)
    n0 = _codes_agree(kf, c0_ref, cd0.cpu().numpy(), cd0_ref, w.pq_m)
    # one iteration: the new centroids are the member means of that assignment
    c1_ref, cd1_ref, _ = oracle.pq_build(d["k"], w.dtype, w.pq_m, w.pq_centroids, 1, init)
    c1, cd1 = pqc.pq_build(w, keys, init_d, iters=1)
    torch.cuda.synchronize()
    if n0 == 0:
        np.testing.assert_allclose(c1.cpu().numpy(), c1_ref, rtol=2e-6, atol=2e-6)
    # assignment against given centroids (the oracle's), the step K-Means repeats
    cd = pqc.pq_assign(w, keys, torch.from_numpy(c1_ref).to(DEV))
    torch.cuda.synchronize()
    n1 = _codes_agree(kf, c1_ref, cd.cpu().numpy(), cd1_ref, w.pq_m)
    assert n0 + n1 <= 1e-3 * cd1_ref.size


@pytest.mark.parametrize("name", ["tiny_f32", "llama8b_32k", "batch8_32k"])
def test_centroid_update_with_keys_of_large_magnitude(pqc, name):
    # The centroid sums are taken in fixed point; values of 2048 and more take another way through the kernel than
    # small ones.  A tenth of the tokens is scaled into that range, a few far beyond it, with both signs.  Expected:
    # the member means (double precision) under the codes the GPU itself assigned in round 0, so that no near-tie
    # between two centroids can blur the comparison.
    w = wl.get(name, **CASES[name])
    print(f"[case] pq update, large keys {w}", flush=True)
    d = wl.generate(w, seed=13)
    rng = np.random.default_rng(13)
    kf = wl.to_f32(d["k"], w.dtype).copy()
    big = rng.random(kf.shape[:3]) < 0.1
    kf[big] *= 1500.0
    huge = rng.random(kf.shape[:3]) < 0.002
    kf[huge] *= -3.0e5
    keys_h = np.ascontiguousarray(kf, dtype=np.float32) if w.dtype == "f32" else wl.f32_to_bf16_bits(kf)
    kf = wl.to_f32(keys_h, w.dtype)
    assert np.abs(kf).max() > 1e6 and (np.abs(kf) >= 2048).mean() > 0.01
    init = wl.kmeans_init_indices(w, seed=13)
    keys, init_d = pqc.to_device(keys_h, w.dtype, DEV), torch.from_numpy(init).to(DEV)
    c0, cd0 = pqc.pq_build(w, keys, init_d, iters=0)
    c1, _ = pqc.pq_build(w, keys, init_d, iters=1)
    torch.cuda.synchronize()
    c0, cd0, c1 = c0.cpu().numpy(), cd0.cpu().numpy(), c1.cpu().numpy()
    Dm = w.sub_dim
    for b in range(w.batch):
        for g in range(w.n_kv_heads):
            for j in range(w.pq_m):
                x = kf[b, g, :, j * Dm:(j + 1) * Dm].astype(np.float64)
                for c in range(w.pq_centroids):
                    members = cd0[b, g, :, j] == c
                    want = x[members].mean(0) if members.any() else c0[b, g, j, c].astype(np.float64)
                    np.testing.assert_allclose(c1[b, g, j, c], want, rtol=2e-6, atol=2e-6, err_msg=f"{(b, g, j, c)}")


@pytest.mark.parametrize("name", ["llama8b_32k", "llama70b_128k"])
def test_kmeans_converges_like_the_oracle(pqc, name):
    w = wl.get(name, batch=1, n_tokens=4000)
    print(f"[case] pq build {w}", flush=True)
    d = wl.generate(w, seed=12)
    init = wl.kmeans_init_indices(w, seed=12)
    kf = wl.to_f32(d["k"], w.dtype)
    T = 6
    cent, codes = pqc.pq_build(w, pqc.to_device(d["k"], w.dtype, DEV), torch.from_numpy(init).to(DEV), iters=T)
    torch.cuda.synchronize()
    cent, codes = cent.cpu().numpy(), codes.cpu().numpy()
    _, _, inertia_ref = oracle.pq_build(d["k"], w.dtype, w.pq_m, w.pq_centroids, T, init)
    Dm = w.sub_dim
    for g in range(w.n_kv_heads):
        for j in range(w.pq_m):
            x = kf[0, g, :, j * Dm:(j + 1) * Dm].astype(np.float64)
            d2 = ((x[:, None, :] - cent[0, g, j][None].astype(np.float64)) ** 2).sum(-1)
            # returned codes are nearest centroids of the returned centroids (up to fp32 near-ties)
            chosen = d2[np.arange(len(x)), codes[0, g, :, j]]
            assert np.all(chosen <= d2.min(1) * (1 + 1e-5))
            # same quality of clustering as the oracle's run from the same start
            assert abs(chosen.sum() - inertia_ref[0, g, j, -1]) <= 2e-3 * inertia_ref[0, g, j, -1]


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name,T", [("llama8b_128k", 2), ("batch8_32k", 1)])
def test_build_at_full_length_matches_oracle(pqc, name, T):
    # The benchmark's own builds (131072 tokens x 8 heads with two partitions of 64 centroids; 32768 tokens x 64 heads
    # with four partitions of 256), so that token ranges and tiles are the ones bench.py builds with; the last head is
    # compared with the oracle, the others hold other keys.
    # Round by round, so that a legitimate near-tie in one round cannot hide behind the next: the start,
    # every round's centroids given the previous GPU codes are the oracle's member means, the final codes are
    # the oracle's nearest centroids of the GPU's own centroids.
    w0 = wl.get(name)
    w = wl.get(name, batch=1, n_q_heads=w0.group, n_kv_heads=1)
    print(f"[case] pq build at full length, T={T}: {w0}", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(15)
    d = wl.generate(w, seed=15)
    init = wl.kmeans_init_indices(w, seed=15)
    kf = wl.to_f32(d["k"], w.dtype)
    keys = torch.randn((w0.batch, w0.n_kv_heads, w0.n_tokens, w0.head_dim), generator=gen, device=DEV, dtype=torch.bfloat16)
    keys[-1:, -1:] = pqc.to_device(d["k"], w.dtype, DEV)
    init_d = torch.from_numpy(wl.kmeans_init_indices(w0, seed=16)).to(DEV)
    init_d[-1:, -1:] = torch.from_numpy(init).to(DEV)

    def build(iters):
        cent, codes = pqc.pq_build(w0, keys, init_d, iters=iters)
        return cent[-1:, -1:].cpu().numpy(), codes[-1:, -1:].cpu().numpy()

    def assign(cent):
        full = torch.randn((w0.batch, w0.n_kv_heads, *cent.shape[2:]), generator=gen, device=DEV)
        full[-1:, -1:] = torch.from_numpy(cent).to(DEV)
        return pqc.pq_assign(w0, keys, full)[-1:, -1:].cpu().numpy()

    near = 0
    # whole run against the oracle's run from the same start
    c_ref, cd_ref, inertia_ref = oracle.pq_build(d["k"], w.dtype, w.pq_m, w.pq_centroids, T, init)
    cent, codes = build(T)
    # (1) the final assignment is the stand-alone assignment, and every returned code is a nearest centroid of
    # the returned centroids (double-precision distances, up to fp32 near-ties)
    np.testing.assert_array_equal(assign(cent), codes)
    Dm = w.sub_dim
    for j in range(w.pq_m):
        cj = cent[0, 0, j].astype(np.float64)
        for t0 in range(0, w.n_tokens, 8192):
            x = kf[0, 0, t0:t0 + 8192, j * Dm:(j + 1) * Dm].astype(np.float64)
            d2 = (x * x).sum(-1)[:, None] - 2.0 * x @ cj.T + (cj * cj).sum(-1)[None]
            chosen = d2[np.arange(len(x)), codes[0, 0, t0:t0 + 8192, j]]
            assert np.all(chosen <= d2.min(1) * (1 + 1e-5) + 1e-9)
    # (2) round 0 of both sides: same start, same codes up to near-ties
    c0, cd0 = build(0)
    c0_ref, cd0_ref, _ = oracle.pq_build(d["k"], w.dtype, w.pq_m, w.pq_centroids, 0, init)
    np.testing.assert_array_equal(c0, c0_ref)
    near += _codes_agree(kf, c0_ref, cd0, cd0_ref, w.pq_m)
    # (3) one update: member means of that assignment (exact agreement of the codes makes the means comparable)
    c1, _ = build(1)
    c1_ref, cd1_ref, _ = oracle.pq_build(d["k"], w.dtype, w.pq_m, w.pq_centroids, 1, init)
    if near == 0:
        np.testing.assert_allclose(c1, c1_ref, rtol=2e-6, atol=2e-6)
    # (4) assignment against the oracle's final centroids
    near += _codes_agree(kf, c_ref, assign(c_ref), cd_ref, w.pq_m)
    assert near <= 1e-3 * cd_ref.size
    # (5) the GPU's own run ends with the oracle's clustering quality, and with its centroids and codes when no
    # near-tie moved a token on the way
    for j in range(w.pq_m):
        x = kf[0, 0, :, j * Dm:(j + 1) * Dm].astype(np.float64)
        chosen = ((x - cent[0, 0, j][codes[0, 0, :, j]].astype(np.float64)) ** 2).sum(-1)
        assert abs(chosen.sum() - inertia_ref[0, 0, j, -1]) <= 1e-4 * inertia_ref[0, 0, j, -1]
    if np.allclose(cent, c_ref, rtol=2e-6, atol=2e-6):
        near += _codes_agree(kf, c_ref, codes, cd_ref, w.pq_m)
    else:  # a near-tie of an earlier round moved a token to the other centroid: the runs part by a few tokens
        assert near > 0 or T > 1
        assert (codes != cd_ref).mean() <= 1e-3
    print(f"[result] {name}: {near} near-tie codes of {cd_ref.size}", flush=True)


# One round and the assignment at the edges of the kernels' tiles and ranges: fewer tokens than a 16-token tile, one more than a
# tile, one range and several per (unit, partition), accumulators that do not fit LDS (two partitions of 256), centroids staged in
# groups (one partition of 256), 16-dimensional sub-vectors, centroid counts that are not a multiple of 16, fp32 keys of every
# sub-vector length; "huge": keys beyond 2^30, which are converted another way; "crowd": most tokens are one and the same.
# Few (unit, partition) pairs are cut into ranges of a few tokens; 256 of them get one range each, which is what brings a range
# past a batch of its workgroup's sixteen waves.
@pytest.mark.parametrize("dtype,m,c,n,units,kind", [
    ("bf16", 2, 64, 1, 1, ""), ("bf16", 2, 64, 17, 3, ""), ("bf16", 4, 256, 2049, 2, ""), ("bf16", 4, 7, 129, 2, ""),
    ("bf16", 4, 256, 300, 96, ""), ("bf16", 2, 256, 1000, 2, ""), ("bf16", 1, 256, 700, 2, ""), ("bf16", 1, 20, 2100, 1, ""),
    ("bf16", 8, 200, 500, 2, ""), ("f32", 8, 33, 257, 2, ""), ("f32", 4, 256, 1000, 1, ""), ("f32", 2, 64, 15, 2, ""),
    ("f32", 1, 256, 600, 1, ""), ("f32", 1, 9, 513, 2, ""), ("bf16", 2, 48, 1600, 2, "huge"), ("f32", 4, 16, 400, 2, "huge"),
    ("bf16", 4, 32, 900, 2, "twins"), ("bf16", 2, 32, 900, 2, "twins"), ("f32", 2, 32, 900, 2, "twins"),
    # one range of tokens per (unit, partition), so that the vector kernel has whole tokens per lane: one and two at a time (two for
    # 16 and 32 dimensions), a batch and a little of the next, fewer centroids than run side by side
    ("f32", 2, 9, 2063, 128, ""), ("f32", 4, 17, 4111, 64, ""), ("f32", 4, 3, 1100, 64, "huge"), ("bf16", 8, 20, 4099, 32, ""),
    ("bf16", 8, 2, 1031, 32, "twins"), ("f32", 1, 9, 519, 256, ""), ("f32", 1, 2, 1024, 256, "huge"), ("f32", 8, 18, 2048, 32, "twins"),
    # four lanes per token, several batches of 256 (128 dimensions: 128) tokens
    ("f32", 2, 9, 700, 128, ""), ("f32", 1, 5, 300, 256, ""), ("bf16", 8, 7, 530, 32, "crowd"),
    # the matrix-core kernel with two tiles per wave, a batch of 512 tokens and some of the next
    ("bf16", 4, 17, 700, 64, ""), ("bf16", 2, 9, 900, 128, ""), ("bf16", 1, 20, 700, 256, ""),
    # with eight, five and three tiles per wave (32, 64 and 128 dimensions): batches of 2048, 1280 and 768 tokens and some of the next,
    # several such ranges, large and equal keys
    ("bf16", 4, 17, 2100, 64, ""), ("bf16", 2, 9, 1303, 128, ""), ("bf16", 1, 20, 900, 256, ""), ("bf16", 2, 20, 5200, 32, ""),
    ("bf16", 4, 9, 2100, 64, "huge"), ("bf16", 2, 9, 1303, 128, "huge"), ("bf16", 1, 9, 900, 256, "huge"),
    ("bf16", 4, 9, 2100, 64, "crowd"), ("bf16", 2, 9, 1303, 128, "crowd"), ("bf16", 4, 16, 1000, 3, "crowd"), ("f32", 4, 9, 2100, 64, "crowd"),
])
def test_round_edges(pqc, dtype, m, c, n, units, kind):
    w = wl.Workload(name="round", batch=units, n_q_heads=1, n_kv_heads=1, head_dim=128, n_tokens=n, pq_m=m, pq_centroids=c,
                    topk=1 if n < 80 else n // 4, n_init=0, n_local=0, dtype=dtype, kmeans_iters=1, recipe="plain")
    print(f"[case] round edges {dtype} m={m} c={c} n={n} units={units} {kind}", flush=True)
    d = wl.generate(w, seed=n + c)
    rng = np.random.default_rng(n)
    kf = wl.to_f32(d["k"], dtype).copy()
    if kind == "huge":
        kf[rng.random(kf.shape[:3]) < 0.05] *= 3.0e9
    if kind == "crowd":
        same = rng.random(kf.shape[:3]) < 0.7
        kf = np.where(same[..., None], kf[:, :, :1], kf)
    keys_h = kf if dtype == "f32" else wl.f32_to_bf16_bits(kf)
    kf = wl.to_f32(keys_h, dtype)
    init = wl.kmeans_init_indices(w, seed=3)
    if kind == "twins":  # every centroid twice: the lower index must take all members
        init[..., 1::2] = init[..., 0::2]
    keys, init_d = pqc.to_device(keys_h, dtype, DEV), torch.from_numpy(init).to(DEV)
    c0, cd0 = pqc.pq_build(w, keys, init_d, iters=0)
    c1, cd1 = pqc.pq_build(w, keys, init_d, iters=1)
    torch.cuda.synchronize()
    c0, cd0, c1, cd1 = c0.cpu().numpy(), cd0.cpu().numpy(), c1.cpu().numpy(), cd1.cpu().numpy()
    c0_ref, cd0_ref, _ = oracle.pq_build(keys_h, dtype, m, c, 0, init)
    np.testing.assert_array_equal(c0, c0_ref)
    if kind == "twins":
        assert np.all(cd0 % 2 == 0)
    if kind != "huge":  # (|c|^2 - 2 x.c of magnitudes far apart: the comparison rule of near-ties does not fit)
        assert _codes_agree(kf, c0_ref, cd0, cd0_ref, m) <= 1 + 1e-3 * cd0.size
        want = np.stack([oracle.nearest_codes(np.ascontiguousarray(keys_h[:, :, t]), dtype, c1) for t in range(n)], axis=2)
        assert _codes_agree(kf, c1, cd1, want, m) <= 1 + 1e-3 * cd1.size
    Dm = 128 // m
    for u in range(units):
        for j in range(m):
            x = kf[u, 0, :, j * Dm:(j + 1) * Dm].astype(np.float64)
            members = (cd0[u, 0, :, j][:, None] == np.arange(c)).astype(np.float64)  # [n][c]
            count = members.sum(0)
            want = np.where(count[:, None] > 0, members.T @ x / np.maximum(count, 1.0)[:, None], c0[u, 0, j].astype(np.float64))
            # 2^-20 per key and one fp32 rounding; the mean of keys of both signs may cancel
            tol = 2e-6 * (1.0 + np.abs(want)) + 2.0 ** -20
            if kind == "huge":
                largest = np.stack([np.abs(x[members[:, k] > 0]).max(initial=1.0) for k in range(c)])
                tol = 2e-6 * (1.0 + np.abs(want)) + largest[:, None] * 2.0 ** -24
            assert np.all(np.abs(c1[u, 0, j] - want) <= tol), (u, j)


# A key value that is not a number adds nothing to the sum of its centroid (its token still counts as a member) and leaves
# every other dimension alone, whichever conversion the kernel takes for the values around it.
@pytest.mark.parametrize("dtype,m,c,n,units", [
    ("bf16", 4, 16, 700, 1), ("bf16", 2, 64, 700, 1), ("bf16", 1, 32, 700, 1), ("bf16", 1, 256, 700, 1), ("f32", 2, 16, 700, 1),
    # one range per (unit, partition): eight, five and three tiles per wave, one and two tokens per lane
    ("bf16", 4, 16, 2100, 64), ("bf16", 2, 16, 1303, 128), ("bf16", 1, 16, 900, 256), ("bf16", 8, 16, 2100, 32), ("f32", 2, 16, 1100, 128),
])
def test_round_passes_over_what_is_not_a_number(pqc, dtype, m, c, n, units):
    Dm = 128 // m
    w = wl.Workload(name="round", batch=units, n_q_heads=1, n_kv_heads=1, head_dim=128, n_tokens=n, pq_m=m, pq_centroids=c,
                    topk=n // 4, n_init=0, n_local=0, dtype=dtype, kmeans_iters=1, recipe="plain")
    print(f"[case] not a number {dtype} m={m} c={c} n={n} units={units}", flush=True)
    d = wl.generate(w, seed=c)
    init = wl.kmeans_init_indices(w, seed=3)
    kf = wl.to_f32(d["k"], dtype).copy()
    bad = np.setdiff1d(np.arange(n), init.ravel())[::37]
    kf[:, 0, bad, (5 * bad) % 128] = np.nan
    keys = pqc.to_device(kf if dtype == "f32" else wl.f32_to_bf16_bits(kf), dtype, DEV)
    init_d = torch.from_numpy(init).to(DEV)
    _, cd0 = pqc.pq_build(w, keys, init_d, iters=0)
    c1, _ = pqc.pq_build(w, keys, init_d, iters=1)
    torch.cuda.synchronize()
    cd0, c1 = cd0.cpu().numpy(), c1.cpu().numpy()
    for u in {0, units // 2, units - 1}:
        x = np.nan_to_num(keys[u, 0].float().cpu().numpy().astype(np.float64), nan=0.0)
        for j in range(m):
            for k in np.unique(cd0[u, 0, :, j]):
                want = x[cd0[u, 0, :, j] == k, j * Dm:(j + 1) * Dm].mean(0)
                # 2^-20 per key and one fp32 rounding
                assert np.all(np.abs(c1[u, 0, j, k] - want) <= 2.0 ** -20 + 2e-6 * (1.0 + np.abs(want))), (u, j, k)


# A workspace taken once serves every length, also one that holds a single set of sums per (unit, partition): ranges of tokens
# then add to it with atomics, which gives the sums of the sets bit for bit.
@pytest.mark.parametrize("dtype,m,c,units", [("bf16", 2, 64, 8), ("bf16", 4, 48, 3), ("bf16", 2, 256, 2), ("f32", 2, 64, 9), ("f32", 8, 20, 1)])
def test_build_in_the_smallest_workspace_at_several_lengths(pqc, dtype, m, c, units):
    import ctypes
    lib = pqc.load()
    ws = None
    for n in (20011, 700, 4096):
        w = wl.Workload(name="round", batch=units, n_q_heads=1, n_kv_heads=1, head_dim=128, n_tokens=n, pq_m=m, pq_centroids=c,
                        topk=n // 4, n_init=0, n_local=0, dtype=dtype, kmeans_iters=3, recipe="plain")
        print(f"[case] smallest workspace {dtype} m={m} c={c} n={n} units={units}", flush=True)
        gen = torch.Generator(device=DEV)
        gen.manual_seed(n)
        keys = torch.randn((units, 1, n, 128), generator=gen, device=DEV, dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
        init = torch.from_numpy(wl.kmeans_init_indices(w, seed=3)).to(DEV)
        if ws is None:
            up = lambda b: (b + 255) // 256 * 256
            sets = units * m * c
            ws = torch.full((up(8 * sets * w.sub_dim) + up(4 * sets),), 0xa5, dtype=torch.uint8, device=DEV)
        cent = torch.empty((units, 1, m, c, w.sub_dim), dtype=torch.float32, device=DEV)
        codes = torch.empty((units, 1, n, m), dtype=torch.uint8, device=DEV)
        rc = lib.pqc_pq_build(ctypes.byref(pqc.make_config(w)), keys.data_ptr(), init.data_ptr(), 3, cent.data_ptr(), codes.data_ptr(),
                              ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        want_cent, want_codes = pqc.pq_build(w, keys, init)
        torch.cuda.synchronize()
        assert torch.equal(cent, want_cent) and torch.equal(codes, want_codes), n


# Rounds that take the means of the round in front themselves (sums in three places in turn, centroids in two) against a launch for
# the means after each round, which the smallest workspace asks for: the same bits after any number of rounds.
@pytest.mark.parametrize("dtype,m,c,n,units", [("bf16", 2, 64, 1031, 1), ("bf16", 4, 256, 5003, 1), ("bf16", 2, 50, 40009, 2), ("bf16", 1, 64, 9001, 3),
                                               ("bf16", 8, 20, 3001, 2), ("f32", 2, 64, 2048, 1), ("f32", 4, 33, 70001, 2)])
def test_linked_rounds(pqc, dtype, m, c, n, units):
    import ctypes
    lib = pqc.load()
    w = wl.Workload(name="round", batch=units, n_q_heads=1, n_kv_heads=1, head_dim=128, n_tokens=n, pq_m=m, pq_centroids=c,
                    topk=n // 4, n_init=0, n_local=0, dtype=dtype, kmeans_iters=3, recipe="plain")
    cfg = ctypes.byref(pqc.make_config(w))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n)
    keys = torch.randn((units, 1, n, 128), generator=gen, device=DEV, dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    init = torch.from_numpy(wl.kmeans_init_indices(w, seed=3)).to(DEV)
    init[:, :, :, 1] = init[:, :, :, 0]  # the second of two equal centroids has no members and stays as it is
    up = lambda b: (b + 255) // 256 * 256
    least = up(8 * units * m * c * w.sub_dim) + up(4 * units * m * c)
    for iters in (0, 1, 2, 3, 4, 7):
        got = []
        for nbytes in (lib.pqc_pq_build_workspace_bytes(cfg), least):
            ws = torch.full((nbytes,), 0xa5, dtype=torch.uint8, device=DEV)
            cent = torch.empty((units, 1, m, c, w.sub_dim), dtype=torch.float32, device=DEV)
            codes = torch.empty((units, 1, n, m), dtype=torch.uint8, device=DEV)
            assert lib.pqc_pq_build(cfg, keys.data_ptr(), init.data_ptr(), iters, cent.data_ptr(), codes.data_ptr(), ws.data_ptr(), nbytes,
                                    torch.cuda.current_stream().cuda_stream) == 0
            torch.cuda.synchronize()
            got.append((cent, codes))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), iters


# As many sets of sums are cleared as rounds add to them: none without rounds, the first two (or the one there is) at most.
@pytest.mark.parametrize("dtype,m,c,n,units", [("bf16", 2, 64, 20000, 2), ("f32", 4, 64, 3001, 1)])
def test_sums_nobody_reads_are_left_alone(pqc, dtype, m, c, n, units):
    import ctypes
    lib = pqc.load()
    w = wl.Workload(name="sums", batch=units, n_q_heads=1, n_kv_heads=1, head_dim=128, n_tokens=n, pq_m=m, pq_centroids=c,
                    topk=0, n_init=1, n_local=0, dtype=dtype, kmeans_iters=1, recipe="plain")
    cfg = ctypes.byref(pqc.make_config(w))
    keys = torch.randn((units, 1, n, 128), device=DEV, dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    init = torch.from_numpy(wl.kmeans_init_indices(w, seed=3)).to(DEV)
    nbytes, a_set = lib.pqc_pq_build_workspace_bytes(cfg), 8 * units * 128 * c
    for iters, sets in ((0, 0), (1, 1), (2, 2)):
        ws = torch.full((nbytes,), 0xa5, dtype=torch.uint8, device=DEV)
        cent = torch.empty((units, 1, m, c, w.sub_dim), dtype=torch.float32, device=DEV)
        codes = torch.empty((units, 1, n, m), dtype=torch.uint8, device=DEV)
        assert lib.pqc_pq_build(cfg, keys.data_ptr(), init.data_ptr(), iters, cent.data_ptr(), codes.data_ptr(), ws.data_ptr(), nbytes,
                                torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        untouched = [bool((ws[x * a_set:(x + 1) * a_set] == 0xa5).all()) for x in range(3)]
        assert untouched == [x >= sets for x in range(3)], iters


# A build recorded into a HIP graph: every replay starts from its own cleared sums, whatever ran in the workspace in between.
@pytest.mark.parametrize("dtype,m,c,units", [("bf16", 2, 64, 1), ("bf16", 2, 64, 8), ("bf16", 2, 256, 1), ("f32", 4, 20, 3)])
def test_recorded_build_replays(pqc, dtype, m, c, units):
    import ctypes
    n = 5000
    w = wl.Workload(name="round", batch=units, n_q_heads=1, n_kv_heads=1, head_dim=128, n_tokens=n, pq_m=m, pq_centroids=c,
                    topk=n // 4, n_init=0, n_local=0, dtype=dtype, kmeans_iters=3, recipe="plain")
    lib, cfg = pqc.load(), ctypes.byref(pqc.make_config(w))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n)
    keys = torch.randn((units, 1, n, 128), generator=gen, device=DEV, dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    init = torch.from_numpy(wl.kmeans_init_indices(w, seed=3)).to(DEV)
    ws = torch.full((lib.pqc_pq_build_workspace_bytes(cfg),), 0x5a, dtype=torch.uint8, device=DEV)
    cent = torch.empty((units, 1, m, c, w.sub_dim), dtype=torch.float32, device=DEV)
    codes = torch.empty((units, 1, n, m), dtype=torch.uint8, device=DEV)

    def build():
        assert lib.pqc_pq_build(cfg, keys.data_ptr(), init.data_ptr(), 3, cent.data_ptr(), codes.data_ptr(), ws.data_ptr(),
                                ws.numel(), torch.cuda.current_stream().cuda_stream) == 0

    build()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        build()
    for _ in range(4):
        keys.copy_(torch.randn(keys.shape, generator=gen, device=DEV, dtype=keys.dtype))
        want_cent, want_codes = pqc.pq_build(w, keys, init)
        ws.fill_(0xa5)
        cent.zero_()
        codes.fill_(255)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(cent, want_cent) and torch.equal(codes, want_codes)


def test_build_on_another_stream_keeps_its_workspace(pqc):
    # the workspace belongs to the call: memory asked for on the current stream right after it must be other memory while the
    # build waits on its own stream
    w = wl.Workload(name="round", batch=1, n_q_heads=1, n_kv_heads=1, head_dim=128, n_tokens=20000, pq_m=2, pq_centroids=64,
                    topk=100, n_init=0, n_local=0, dtype="bf16", kmeans_iters=3, recipe="plain")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    keys = torch.randn((1, 1, w.n_tokens, 128), generator=gen, device=DEV, dtype=torch.bfloat16)
    init = torch.from_numpy(wl.kmeans_init_indices(w, seed=3)).to(DEV)
    want_cent, want_codes = pqc.pq_build(w, keys, init)
    nbytes = pqc.load().pqc_pq_build_workspace_bytes(pqc._config(w))
    side, busy = torch.cuda.Stream(), torch.randn((4096, 4096), device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(20):  # a few ms
            busy = (busy @ busy).clamp_(-1.0, 1.0)
    cent, codes = pqc.pq_build(w, keys, init, stream=side)
    others = []
    for _ in range(200):  # written over and over while the build runs
        others = [torch.full((nbytes,), 0x7f, dtype=torch.uint8, device=DEV) for _ in range(4)]
    torch.cuda.synchronize()
    del others
    assert torch.equal(cent, want_cent) and torch.equal(codes, want_codes)


def _shortest(fn):
    """Milliseconds of one call: the shortest of eight runs of ten."""
    best = float("inf")
    for _ in range(9):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(10):
            fn()
        t1.record()
        t1.synchronize()
        best = min(best, t0.elapsed_time(t1) / 10)
    return best


# The vector kernel on long inputs, against a copy of the keys (read and written once) on the same card: with four lanes per token
# whatever the length, and one range per unit on 128 compute units at most, these took 2.1 and 9.4 copies (1.0 and 3.1 now).
@pytest.mark.parametrize("dtype,m,c,units,copies", [("bf16", 8, 16, 8, 1.5), ("f32", 1, 64, 1, 5.0)])
def test_assignment_of_long_inputs_keeps_up(pqc, dtype, m, c, units, copies):
    n = 131072
    w = wl.Workload(name="round", batch=units, n_q_heads=1, n_kv_heads=1, head_dim=128, n_tokens=n, pq_m=m, pq_centroids=c,
                    topk=n // 4, n_init=0, n_local=0, dtype=dtype, kmeans_iters=1, recipe="plain")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1)
    keys = torch.randn((units, 1, n, 128), generator=gen, device=DEV, dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    cent = torch.randn((units, 1, m, c, 128 // m), generator=gen, device=DEV)
    copy = torch.empty_like(keys)
    took, ref = _shortest(lambda: pqc.pq_assign(w, keys, cent)), _shortest(lambda: copy.copy_(keys))
    print(f"[result] {dtype} m={m} c={c}: {took * 1e3:.1f} us, a copy {ref * 1e3:.1f} us", flush=True)
    assert took <= copies * ref


# Keys of which all share a centroid (padding, a repeated token) against keys that spread: lanes that add to one address add one
# after the other, which took up to 3.4 times as long before the additions of a wave were spread over the dimensions.
@pytest.mark.parametrize("dtype,m,c", [("bf16", 4, 16), ("bf16", 4, 256), ("bf16", 2, 64), ("bf16", 8, 16), ("f32", 4, 64)])
def test_equal_keys_build_as_fast_as_others(pqc, dtype, m, c):
    n, units = 131072, 8
    w = wl.Workload(name="round", batch=units, n_q_heads=1, n_kv_heads=1, head_dim=128, n_tokens=n, pq_m=m, pq_centroids=c,
                    topk=n // 4, n_init=0, n_local=0, dtype=dtype, kmeans_iters=2, recipe="plain")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(2)
    keys = torch.randn((units, 1, n, 128), generator=gen, device=DEV, dtype=torch.float32 if dtype == "f32" else torch.bfloat16)
    init = torch.from_numpy(wl.kmeans_init_indices(w, seed=3)).to(DEV)
    spread = _shortest(lambda: pqc.pq_build(w, keys, init))
    keys[:] = keys[:, :, :1].clone()
    equal = _shortest(lambda: pqc.pq_build(w, keys, init))
    print(f"[result] {dtype} m={m} c={c}: {spread * 1e3:.1f} us, equal keys {equal * 1e3:.1f} us", flush=True)
    assert equal <= 1.5 * spread
    # and the sums are right: after one round the lowest of the equal centroids is the mean of all tokens, and codes are all alike
    cent, codes = pqc.pq_build(w, keys, init, iters=1)
    want = keys[:, 0, 0].float().view(units, m, w.sub_dim)
    assert (cent[:, 0, :, 0] - want).abs().max() <= 2.0 ** -20 + 2e-6 * want.abs().max()
    assert torch.equal(codes, codes[:, :, :1].expand_as(codes))


def test_encode_token_writes_nearest_codes_in_place(pqc):
    w = wl.get("batch8_32k", batch=3, n_tokens=700)
    d = wl.generate(w, seed=13)
    init = wl.kmeans_init_indices(w, seed=13)
    cent, codes, _ = oracle.pq_build(d["k"], w.dtype, w.pq_m, w.pq_centroids, 2, init)
    pos = 650
    key = np.ascontiguousarray(d["k"][:, :, pos])  # re-encode an existing token: its code must be reproduced
    codes_d = torch.from_numpy(codes).to(DEV)
    before = codes_d.clone()
    codes_d[:, :, pos] = 255
    pqc.pq_encode_token(w, pqc.to_device(key, w.dtype, DEV), torch.from_numpy(cent).to(DEV), codes_d, pos)
    torch.cuda.synchronize()
    want = oracle.nearest_codes(key, w.dtype, cent)
    got = codes_d.cpu().numpy()
    kf = wl.to_f32(d["k"], w.dtype)
    mism = _codes_agree(kf[:, :, pos:pos + 1], cent, got[:, :, pos:pos + 1], want[:, :, None, :], w.pq_m)
    assert mism <= 1
    mask = np.ones(w.n_tokens, bool)
    mask[pos] = False
    np.testing.assert_array_equal(got[:, :, mask], before.cpu().numpy()[:, :, mask])


def test_decode_after_gpu_pq_build(pqc):
    # End to end on GPU-built PQ structures: the decode path must agree with the oracle run on the same structures.
    from parity_utils import ATTN_TOL, Problem, attn_error, check_indices
    w = wl.get("llama8b_128k", n_tokens=12000)
    d = wl.generate(w, seed=14)
    keys = pqc.to_device(d["k"], w.dtype, DEV)
    cent, codes = pqc.pq_build(w, keys, torch.from_numpy(wl.kmeans_init_indices(w, 14)).to(DEV), iters=4)
    ctx = pqc.PQCache(w, DEV)
    idx, out = ctx.decode(pqc.to_device(d["q"], w.dtype, DEV), cent, codes, keys, pqc.to_device(d["v"], w.dtype, DEV))
    torch.cuda.synchronize()
    p = Problem(w, d["q"], d["k"], d["v"], cent.cpu().numpy(), codes.cpu().numpy(), list(range(w.n_kv_heads)))
    assert check_indices(p, idx.cpu().numpy()) == 0
    assert attn_error(p, idx.cpu().numpy(), out.cpu().numpy()) <= ATTN_TOL[w.dtype]
    planted = d["planted"]
    got = idx.cpu().numpy()
    found = np.mean([np.isin(planted[0, g], got[0, g]).mean() for g in range(w.n_kv_heads)])
    assert found > 0.9, f"only {found:.2f} of the planted tokens were retrieved"


@pytest.mark.parametrize("block,k_cache", [(128, 20), (128, 0), (64, 7), (2047, 3), (1, 300), (100, 79)])
def test_block_stats_match_oracle(pqc, block, k_cache):
    # per-block counts of the attended tokens and the k_cache fullest blocks (Section 3.4)
    w = wl.Workload(name="blocks", batch=2, n_q_heads=4, n_kv_heads=2, head_dim=128, n_tokens=7900, pq_m=2, pq_centroids=16,
                    topk=900, n_init=4, n_local=64, dtype="bf16", kmeans_iters=1, recipe="plain")
    rng = np.random.default_rng(block * 1000 + k_cache)
    # clumped selections, so that counts differ and tie at the same time
    idx = np.stack([np.sort(rng.choice(np.arange(0, w.n_tokens, 3) if u % 2 else w.n_tokens, size=w.n_selected, replace=False))
                    for u in range(4)]).reshape(2, 2, -1).astype(np.int32)
    nb = (w.n_tokens + block - 1) // block
    k_cache = min(k_cache, nb)
    counts, blocks = pqc.block_stats(w, torch.from_numpy(idx).to(DEV), block, k_cache)
    torch.cuda.synchronize()
    want_c = oracle.block_counts(idx, w.n_tokens, block)
    np.testing.assert_array_equal(counts.cpu().numpy(), want_c)
    want_b = oracle.block_topk(want_c, k_cache)
    np.testing.assert_array_equal(blocks.cpu().numpy(), want_b)  # same blocks in the same order: fullest first, lower index on ties


# the edges of the count kernel: blocks whose counts still fit LDS and one more, more blocks above the cut than are ranked by
# counting, an unsorted list (no runs of equal blocks), a list with entries that are no tokens
@pytest.mark.parametrize("n,n_idx,block,k_cache,order", [
    (16384, 3000, 1, 2900, "sorted"), (16385, 3000, 1, 2900, "sorted"), (16385, 3000, 1, 17, "shuffled"), (40000, 20000, 64, 300, "shuffled"),
    (40000, 20000, 64, 200, "sorted"), (40000, 1, 64, 3, "sorted"), (5000, 4999, 2047, 3, "shuffled"), (9000, 1025, 7, 100, "foreign"),
])
def test_block_stats_edges(pqc, n, n_idx, block, k_cache, order):
    w = wl.Workload(name="blocks", batch=1, n_q_heads=4, n_kv_heads=2, head_dim=128, n_tokens=n, pq_m=2, pq_centroids=16,
                    topk=100, n_init=4, n_local=64, dtype="bf16", kmeans_iters=1, recipe="plain")
    print(f"[case] block stats n={n} n_idx={n_idx} block={block} k_cache={k_cache} {order}", flush=True)
    rng = np.random.default_rng(n + n_idx + block)
    rows = []
    for _ in range(2):  # counts grow towards the end of the range, so that many differ
        r = rng.choice(n, size=n_idx, replace=False, p=(np.arange(n) + 1.0) / (n * (n + 1.0) / 2.0))
        rows.append(r if order == "shuffled" else np.sort(r))
    idx = np.stack(rows).reshape(1, 2, -1).astype(np.int32)
    given = idx.copy()
    if order == "foreign":
        given[0, :, ::5] = np.where(np.arange(given[0, :, ::5].shape[-1]) % 2, -3, n + 2)
        idx = np.delete(idx, np.s_[::5], axis=-1)
    counts, blocks = pqc.block_stats(w, torch.from_numpy(given).to(DEV), block, k_cache)
    torch.cuda.synchronize()
    want_c = oracle.block_counts(np.ascontiguousarray(idx), n, block)
    np.testing.assert_array_equal(counts.cpu().numpy(), want_c)
    np.testing.assert_array_equal(blocks.cpu().numpy(), oracle.block_topk(want_c, k_cache))


@pytest.mark.parametrize("policy", ["lru", "lfu"])
@pytest.mark.parametrize("n_slots,k_cache,block", [(32, 32, 128), (1, 1, 128), (5, 3, 64), (4, 9, 256), (16, 0, 128),
                                                   (1024, 200, 16), (100, 1024, 4)])
def test_block_cache_refresh_matches_oracle(pqc, policy, n_slots, k_cache, block):
    # Section 3.4 over a run of decode steps: look-up, then refresh with the fullest blocks; the state evolves
    # on both sides from the same start and must stay identical
    w = wl.Workload(name="cache", batch=2, n_q_heads=4, n_kv_heads=2, head_dim=128, n_tokens=8190, pq_m=2, pq_centroids=16,
                    topk=800, n_init=4, n_local=64, dtype="bf16", kmeans_iters=1, recipe="plain")
    nb = (w.n_tokens + block - 1) // block
    k_cache = min(k_cache, nb)
    rng = np.random.default_rng(n_slots * 7 + k_cache)
    dev_state = [torch.full((2, 2, n_slots), -1, dtype=torch.int32, device=DEV)] + [
        torch.zeros((2, 2, n_slots), dtype=torch.int32, device=DEV) for _ in range(2)]
    host_state = [t.cpu().numpy() for t in dev_state]
    hot = rng.choice(w.n_tokens, 600, replace=False)  # tokens that keep coming back, so that some blocks stay hot
    for step in range(1, 13):
        idx = np.stack([np.sort(np.concatenate([rng.choice(hot, 300, replace=False),
                                                rng.choice(np.setdiff1d(np.arange(w.n_tokens), hot), w.n_selected - 300, replace=False)]))
                        for _ in range(4)]).reshape(2, 2, -1).astype(np.int32)
        counts, blocks = pqc.block_stats(w, torch.from_numpy(idx).to(DEV), block, k_cache)
        if step % 4 == 0 and k_cache > 2:  # now and then some entries that are not block numbers: they are skipped
            blocks[:, :, 1] = -1
            blocks[:, 0, 2] = nb + 5
        stats = pqc.block_cache_update(w, block, policy, step, counts, blocks, *dev_state)
        torch.cuda.synchronize()
        # the oracle runs on its own counts and its own request list (fullest block first): which blocks survive when
        # the requests outnumber the slots depends on that order
        want_counts = oracle.block_counts(idx, w.n_tokens, block)
        np.testing.assert_array_equal(counts.cpu().numpy(), want_counts)
        req = oracle.block_topk(want_counts, k_cache)
        if step % 4 == 0 and k_cache > 2:  # the same entries spoilt on the oracle's side
            req = req.copy()
            req[:, :, 1] = -1
            req[:, 0, 2] = nb + 5
        np.testing.assert_array_equal(blocks.cpu().numpy(), req)
        *host_state, want_stats = oracle.block_cache_update(*host_state, want_counts, req, step, policy)
        for got, want, name in zip(dev_state, host_state, ("block", "stamp", "uses")):
            np.testing.assert_array_equal(got.cpu().numpy(), want, err_msg=f"step {step}: slot_{name}")
        np.testing.assert_array_equal(stats.cpu().numpy(), want_stats, err_msg=f"step {step}: stats")
    if k_cache and n_slots >= 4:
        assert want_stats[..., 0].min() > 0  # the hot tokens do get hits


# The nearest centroid by |c|^2 - 2 x.c with sub-vectors of 32 dimensions: x.c is a finished sum before |c|^2 = 1.5 * 2^24 (of which
# the last bit is 2) comes in.  Three bf16 terms of a centroid contribute -0.9 each, which added one by one to |c|^2 are lost, or
# taken for -2 each, whichever way the sum is rounded; together they are -2.7.  Against them a centroid at |c|^2 and one at |c|^2 - 4.
@pytest.mark.parametrize("n", [40, 9001, 70000])  # ranges of a few tokens, of two tiles per wave, of eight
@pytest.mark.parametrize("rival", [0.0, 4.0])
def test_products_are_summed_before_the_norm(pqc, n, rival):
    C, M = 20, 4
    w = wl.Workload(name="sum", batch=1, n_q_heads=1, n_kv_heads=1, head_dim=128, n_tokens=n, pq_m=M, pq_centroids=C, topk=0, n_init=1,
                    n_local=0, dtype="bf16", kmeans_iters=1, recipe="plain")
    x = np.zeros(32, np.float32)
    x[1], x[2], x[3] = 28.75, 14720.0, 14720.0
    x[4], x[5], x[8] = 7536640.0, 7536640.0, 128.0
    near, other = np.zeros(32, np.float32), np.zeros(32, np.float32)
    near[[0, 6, 7]] = other[[0, 6, 7]] = 4096.0, 2048.0, 2048.0  # |c|^2 = 1.5 * 2^24
    near[1] = 2.0 ** -6
    near[2], near[3] = 2.0 ** -6 + 2.0 ** -15, -(2.0 ** -6)                              # differ in the second term
    near[4], near[5] = 2.0 ** -6 + 2.0 ** -15 + 2.0 ** -24, -(2.0 ** -6 + 2.0 ** -15)    # differ in the third term
    other[8] = rival / 256.0
    assert np.array_equal(wl.to_f32(wl.f32_to_bf16_bits(x), "bf16"), x)
    d = [(c.astype(np.float64) ** 2).sum() - 2.0 * (x.astype(np.float64) * c).sum() for c in (other, near)]
    assert abs(d[0] - 1.5 * 2 ** 24 + rival) < 0.1 and abs(d[1] - 1.5 * 2 ** 24 + 2.7) < 0.1
    cent = np.zeros((1, 1, M, C, 32), np.float32)
    cent[..., 0] = 8192.0  # far
    cent[..., 3, :], cent[..., 11, :] = other, near
    keys = torch.from_numpy(np.tile(x, M)).to(DEV).to(torch.bfloat16).repeat(1, 1, n, 1).contiguous()
    codes = pqc.pq_assign(w, keys, torch.from_numpy(cent).to(DEV))
    assert torch.equal(codes, torch.full_like(codes, 11 if rival == 0.0 else 3))


# Assignments against 64-bit arithmetic, keys with the channel means that real caches have: the squared distances of the assigned and
# of the nearest centroid differ by no more than the errors of their two scores, each (3 products per 32 dimensions + 1) roundings
# of at most 2^-23 of the numbers that are added, |c|^2 + 2 |x|.|c|.
@pytest.mark.parametrize("m,c,n", [(4, 256, 30000), (4, 64, 2000), (2, 64, 30000), (2, 256, 1000), (1, 64, 30000), (1, 256, 3000)])
def test_assignments_are_nearest_to_rounding(pqc, m, c, n):
    H, dm = 8, 128 // m
    w = wl.Workload(name="near", batch=1, n_q_heads=H, n_kv_heads=H, head_dim=128, n_tokens=n, pq_m=m, pq_centroids=c, topk=0, n_init=1,
                    n_local=0, dtype="bf16", kmeans_iters=2, recipe="plain")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(n + c)
    randn = lambda *s: torch.randn(s, generator=gen, device=DEV)
    keys = (randn(1, H, n, 128) + 4.0 * randn(1, H, 1, 128)).to(torch.bfloat16)
    cent, codes = pqc.pq_build(w, keys, torch.from_numpy(wl.kmeans_init_indices(w, seed=1)).to(DEV))
    off = 0
    for h in range(H):
        for j in range(m):
            x, ce = keys[0, h, :, j * dm:(j + 1) * dm].double().contiguous(), cent[0, h, j].double()
            score = ce.square().sum(-1) - 2.0 * torch.mm(x, ce.t().contiguous())
            size = ce.square().sum(-1) + 2.0 * torch.mm(x.abs(), ce.abs().t().contiguous())
            best, at = score.min(-1)
            got = codes[0, h, :, j].long().unsqueeze(1)
            bound = (3 * dm // 32 + 1) * 2.0 ** -23 * (size.gather(1, got) + size.gather(1, at.unsqueeze(1))).squeeze(1)
            excess = score.gather(1, got).squeeze(1) - best
            off += int((excess > 0).sum())
            assert bool((excess <= bound).all())
    print(f"[case] {m}x{c} n={n}: {off} of {H * m * n} not the nearest", flush=True)
