"""GPU parity of decode steps without a histogram kernel (short caches) at the edges of its tiles and of the rule that chooses
it, and of thresholds outside the sampled window on both forms, against the CPU oracle: index sets equal, attention within the
tolerance of tests/parity_utils.py.  Which lengths take it is counted in the launches of a recorded step."""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2407_12820_amd import workloads as wl

from parity_utils import ATTN_TOL, attn_error, build_problem, check_indices, check_structure, count_launches

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def pqc():
    from paper_2407_12820_amd import binding
    binding.load()
    return binding


def _w(**kw):
    base = dict(name="short", batch=1, n_q_heads=4, n_kv_heads=2, head_dim=128, n_tokens=3000, pq_m=2, pq_centroids=64,
                topk=300, n_init=4, n_local=64, dtype="bf16", kmeans_iters=1, recipe="plain")
    base.update(kw)
    return wl.Workload(**base)


def _decode_and_check(pqc, p):
    w = p.w
    every = list(range(w.batch * w.n_kv_heads))
    dev = [pqc.to_device(p.q, w.dtype, DEV), torch.from_numpy(p.centroids).to(DEV), torch.from_numpy(p.codes).to(DEV),
           pqc.to_device(p.k, w.dtype, DEV), pqc.to_device(p.v, w.dtype, DEV)]
    ctx = pqc.PQCache(w, DEV)
    for _ in range(2):  # the second step finds the workspace as the first left it
        idx, out = ctx.decode(*dev)
    torch.cuda.synchronize()
    idx, out = idx.cpu().numpy(), out.cpu().numpy()
    assert check_indices(p, idx, units=every) == 0
    err = attn_error(p, idx, out, units=every)
    assert err <= ATTN_TOL[w.dtype], f"attention error {err:.3e}"
    check_structure(p, idx, out)


@pytest.mark.parametrize("kw", [
    dict(n_tokens=513, topk=60),                                                    # a workgroup with one token
    dict(n_tokens=16385, topk=1600, n_q_heads=2, n_kv_heads=1),                     # one chunk beyond a step of the scan
    dict(n_tokens=16384, topk=1600),
    dict(n_tokens=22528, topk=2250, batch=4),
    dict(n_tokens=24576, topk=2400),
    dict(n_tokens=24577, topk=2400),
    dict(n_tokens=11264, topk=1100, pq_m=4, n_q_heads=4),                           # the last short length of a few units, 4 x 64
    dict(n_tokens=12288, topk=1200, pq_m=4, n_q_heads=8, n_kv_heads=8),             # of more units
    dict(n_tokens=12288, topk=1200, pq_m=4, n_q_heads=16),                          # G = 8
    dict(n_tokens=12289, topk=1200, pq_m=4, n_q_heads=2, dtype="f32"),
    dict(n_tokens=8192, topk=800, pq_m=4, pq_centroids=256),                        # 4 x 256
    dict(n_tokens=8191, topk=800, pq_m=4, pq_centroids=129, n_q_heads=2, dtype="f32"),
    dict(n_tokens=16384, topk=3200, pq_centroids=256, n_q_heads=8),                 # 2 x 256
    dict(n_tokens=3001, batch=3, n_q_heads=5, n_kv_heads=5, topk=700, pq_centroids=48),  # units at every alignment of the codes
    dict(n_tokens=2999, batch=5, n_q_heads=5, n_kv_heads=5, topk=150, pq_m=4, n_init=0, n_local=1),
    dict(n_tokens=300, batch=75, n_q_heads=4, n_kv_heads=4, topk=30),               # more units than workgroups fit at once
    dict(n_tokens=2048, batch=66, n_q_heads=8, n_kv_heads=4, topk=1980),            # every token; 264 units of 512 tokens a workgroup
], ids=lambda kw: ",".join(f"{k}={v}" for k, v in kw.items()))
def test_short_caches(pqc, kw):
    w = _w(**kw)
    print(f"[case] short cache {w}", flush=True)
    _decode_and_check(pqc, build_problem(w, seed=3, checked_units=[]))


# Steps that count the code pairs of their unit (two partitions of up to 64 centroids): units at every alignment of the codes, middle tokens
# beside whole chunks of eight, none of these.
@pytest.mark.parametrize("kw", [
    dict(n_tokens=10241, topk=1000, n_init=3, n_local=5, batch=2),
    dict(n_tokens=10247, topk=1000, n_q_heads=5, n_kv_heads=5, pq_centroids=48, n_init=0, n_local=0),
    dict(n_tokens=9285, topk=900, n_q_heads=2, n_kv_heads=1, pq_centroids=33),
    dict(n_tokens=33861, topk=3000, n_q_heads=2, n_kv_heads=1, pq_centroids=17),
    dict(n_tokens=49152, topk=9000, n_q_heads=8, n_kv_heads=1),                           # the last length of a few units; G = 8
    dict(n_tokens=77, topk=2, n_init=30, n_local=40, batch=3),
    dict(n_tokens=20011, topk=2000, n_q_heads=4, dtype="f32", batch=2),
    dict(n_tokens=11000, topk=600, n_init=4001, n_local=6003),                            # more window tokens than middle ones
    dict(n_tokens=10300, topk=3, n_init=5000, n_local=5295, n_q_heads=2, n_kv_heads=1),   # five middle tokens
    dict(n_tokens=12289, topk=0),
    dict(n_tokens=11111, topk=11043, n_q_heads=2, n_kv_heads=1),                          # all of them
    dict(n_tokens=14336, topk=1400, n_q_heads=8, n_kv_heads=8, batch=16),                 # one workgroup per compute unit
], ids=lambda kw: ",".join(f"{k}={v}" for k, v in kw.items()))
def test_counted_pairs(pqc, kw):
    w = _w(**kw)
    print(f"[case] counted pairs {w}", flush=True)
    _decode_and_check(pqc, build_problem(w, seed=5, checked_units=[]))


# Whole chunks of middle tokens at both sides of what is counted beside the table (1152), and of that and one turn of what is under way
# afterwards (3072 more).
@pytest.mark.parametrize("n_tokens, chunks", [(9293, 1152), (9301, 1153), (33869, 4224), (33877, 4225)])
def test_counted_pairs_at_the_hand_overs(pqc, n_tokens, chunks):
    w = _w(n_tokens=n_tokens, topk=n_tokens // 10, n_q_heads=2, n_kv_heads=1, pq_centroids=33)
    assert (n_tokens - w.n_local) // 8 - -(-w.n_init // 8) == chunks  # (one unit: its chunks start at token 0)
    print(f"[case] hand-over {w}", flush=True)
    _decode_and_check(pqc, build_problem(w, seed=5, checked_units=[]))


# Code tensors whose bytes are no multiple of 16, or fewer than 16: the last bytes reach the last unit's last tokens on every form.
@pytest.mark.parametrize("m, c, n_tokens", [(2, 64, 5), (2, 64, 1003), (2, 64, 4099), (2, 200, 1005), (2, 200, 17003), (4, 64, 3), (4, 64, 1001), (4, 64, 1002),
                                            (4, 64, 12291), (8, 16, 1), (8, 16, 515), (1, 64, 1001), (1, 64, 1014), (1, 64, 13)])
@pytest.mark.parametrize("heads", [1, 3])
def test_ragged_end_of_the_codes(pqc, m, c, n_tokens, heads):
    w = _w(n_tokens=n_tokens, topk=max(1, n_tokens // 3), n_q_heads=heads, n_kv_heads=heads, pq_m=m, pq_centroids=c, n_init=0, n_local=0)
    print(f"[case] ragged end {w}", flush=True)
    _decode_and_check(pqc, build_problem(w, seed=9, checked_units=[]))


@pytest.mark.parametrize("share", [0.3, 0.6, 1.0])
def test_counted_pairs_of_repeated_codes(pqc, share):
    # lanes that meet in one address are counted in one go; a fraction of the tokens carries one pair, or all do
    w = _w(n_tokens=12293, topk=1200, n_init=5)
    p = build_problem(w, seed=7, checked_units=[])
    rng = np.random.default_rng(8)
    codes = np.where(rng.random((1, 2, w.n_tokens, 1)) < share, np.array([13, 60], np.uint8), p.codes)
    print(f"[case] repeated codes {share} {w}", flush=True)
    _decode_and_check(pqc, dataclasses.replace(p, codes=np.ascontiguousarray(codes)))


@pytest.mark.parametrize("n_tokens", [6007, 30001, 60001])  # without and (the last one) with a histogram kernel
@pytest.mark.parametrize("where", ["below", "above"])
def test_threshold_outside_the_window(pqc, n_tokens, where):
    # The sampled tokens (every nmid / 1024-th) all score best or all score worst, so that the K-th largest score lies below or
    # above the window that the sample puts around it: slower, but the same selection.
    w = _w(n_tokens=n_tokens, topk=2000, n_init=5, n_local=33)
    p0 = build_problem(w, seed=4, checked_units=[])
    codes = p0.codes.copy()
    s32, _ = oracle.scores(p0.q, w.dtype, p0.centroids, p0.codes)
    nmid = n_tokens - w.n_init - w.n_local
    sampled = w.n_init + (np.arange(1024) * nmid) // 1024
    for g in range(w.n_kv_heads):
        mid = np.arange(w.n_init, n_tokens - w.n_local)
        order = mid[np.argsort(s32[0, g, mid], kind="stable")]
        codes[0, g, sampled] = p0.codes[0, g, order[-1] if where == "below" else order[0]]
    p = dataclasses.replace(p0, codes=codes)
    print(f"[case] threshold {where} the window {w}", flush=True)
    _decode_and_check(pqc, p)
    # and the stand-alone top-k on the same scores
    s32, _ = oracle.scores(p.q, w.dtype, p.centroids, p.codes)
    idx = pqc.PQCache(w, DEV).topk(torch.from_numpy(s32).to(DEV)).cpu().numpy()
    np.testing.assert_array_equal(np.sort(idx, -1), np.sort(oracle.select(s32, w.topk, w.n_init, w.n_local), -1))


@pytest.mark.parametrize("low, high", [(0.9, 0.0), (0.3, 0.0), (0.0, 0.02), (0.4, 0.4), (0.5, 0.5), (1.0, 0.0)])
def test_topk_of_infinite_scores(pqc, low, high):
    # Masked tokens (-inf) and overflowed ones (+inf), few and many of them: the map from scores to bins keeps their order, also
    # where the window that the sample puts around the K-th largest score has infinite ends.
    w = _w(n_tokens=20068, topk=5000)
    rng = np.random.default_rng(12)
    s32 = rng.standard_normal((1, 2, w.n_tokens)).astype(np.float32)
    x = rng.random(s32.shape)
    s32[x < low] = -np.inf
    s32[x >= 1.0 - high] = np.inf
    print(f"[case] infinite scores low={low} high={high}", flush=True)
    idx = pqc.PQCache(w, DEV).topk(torch.from_numpy(s32).to(DEV)).cpu().numpy()
    np.testing.assert_array_equal(np.sort(idx, -1), np.sort(oracle.select(s32, w.topk, w.n_init, w.n_local), -1))


@pytest.mark.parametrize("units, n_tokens, topk", [(64, 32768, 30000), (33, 4100, 4000), (3, 60001, 59000), (70, 600, 500)])
def test_lists_copied_by_several_waves(pqc, units, n_tokens, topk):
    # few, long lists per unit: waves share one, beyond what they request up front; and lists of which a wave takes several
    w = _w(batch=units, n_q_heads=1, n_kv_heads=1, n_tokens=n_tokens, topk=topk, n_local=33)
    s32 = np.random.default_rng(units).standard_normal((units, 1, n_tokens)).astype(np.float32)
    print(f"[case] long lists {units} {n_tokens}", flush=True)
    idx = pqc.PQCache(w, DEV).topk(torch.from_numpy(s32).to(DEV)).cpu().numpy()
    np.testing.assert_array_equal(np.sort(idx, -1), np.sort(oracle.select(s32, w.topk, w.n_init, w.n_local), -1))


@pytest.mark.parametrize("units, n_tokens, m, c, den, launches", [
    (1, 2048, 2, 64, 10, 2), (7, 49152, 2, 64, 10, 2), (7, 49153, 2, 64, 10, 3), (8, 49153, 2, 48, 10, 2), (15, 53249, 2, 48, 10, 3),
    (16, 57344, 2, 64, 10, 2), (31, 57345, 2, 64, 10, 3), (32, 65536, 2, 64, 5, 2), (32, 65537, 2, 64, 10, 3), (1, 11264, 4, 64, 10, 2),
    (1, 11265, 4, 64, 10, 3), (8, 12288, 4, 64, 10, 2), (8, 12289, 4, 64, 10, 3), (1, 8192, 4, 256, 10, 2), (1, 8193, 4, 256, 10, 3),
    (1, 16384, 2, 65, 10, 2), (1, 16385, 2, 256, 10, 3), (8, 2048, 8, 64, 10, 3), (8, 2048, 1, 64, 10, 3), (96, 20000, 2, 64, 20, 3),
    (80, 20000, 2, 64, 10, 2), (80, 20000, 2, 64, 5, 2), (128, 12288, 2, 64, 5, 3), (128, 16384, 2, 64, 5, 2),
    (207, 8192, 2, 64, 5, 2), (208, 8192, 2, 64, 5, 3), (208, 8192, 2, 64, 7, 2), (256, 8191, 2, 64, 5, 2),
    # lengths around which steps that score every token (not its code pair) give way to the histogram kernel
    (1, 16384, 2, 64, 10, 2), (1, 16385, 2, 64, 10, 2), (7, 16385, 2, 48, 10, 2), (8, 16385, 2, 64, 10, 2), (1, 24576, 2, 64, 10, 2),
    (8, 22528, 2, 64, 10, 2), (8, 22529, 2, 64, 10, 2)])
def test_launches_of_a_step(pqc, units, n_tokens, m, c, den, launches):
    w = _w(batch=units, n_q_heads=1, n_kv_heads=1, n_tokens=n_tokens, pq_m=m, pq_centroids=c, topk=n_tokens // den)
    print(f"[case] launches {w}", flush=True)
    new = lambda shape, dtype: torch.zeros(shape, dtype=dtype, device=DEV)
    kv = torch.bfloat16
    k = new((units, 1, n_tokens, 128), kv)
    args = [new((units, 1, 128), kv), new((units, 1, m, c, 128 // m), torch.float32), new((units, 1, n_tokens, m), torch.uint8), k, k]
    ctx = pqc.PQCache(w, DEV)
    outs = ctx.empty_outputs()
    assert count_launches(lambda: ctx.decode(*args, *outs)) == launches


# A workspace that holds the plan of every other call but not that of the step without a histogram kernel: the step takes the
# general form, with the same result.
@pytest.mark.parametrize("kw", [dict(n_tokens=10755, topk=1000, pq_m=4, batch=16), dict(n_tokens=2147, topk=200, batch=50)])
def test_smallest_workspace(pqc, kw):
    lib = pqc.load()
    w = _w(**kw)
    p = build_problem(w, seed=6, checked_units=[])
    cfg = pqc.make_config(w)
    dev = [pqc.to_device(p.q, w.dtype, DEV), torch.from_numpy(p.centroids).to(DEV), torch.from_numpy(p.codes).to(DEV),
           pqc.to_device(p.k, w.dtype, DEV), pqc.to_device(p.v, w.dtype, DEV)]
    got, launches = [], []
    full = lib.pqc_workspace_bytes(ctypes.byref(cfg))
    room = torch.full((full,), 0xa5, dtype=torch.uint8, device=DEV)

    def create(nbytes):
        h = ctypes.c_void_p()
        return h if lib.pqc_create(ctypes.byref(h), ctypes.byref(cfg), room.data_ptr(), nbytes) == 0 else None

    least = full
    while (h := create(least - 256)) is not None:
        lib.pqc_destroy(h)
        least -= 256
    assert least < full
    for nbytes in (full, least):
        room.fill_(0xa5)
        h = create(nbytes)
        idx = torch.empty((w.batch, w.n_kv_heads, w.n_selected), dtype=torch.int32, device=DEV)
        out = torch.empty((w.batch, w.n_q_heads, 128), dtype=torch.float32, device=DEV)

        def call():
            assert lib.pqc_decode(h, *[t.data_ptr() for t in dev], idx.data_ptr(), out.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0

        launches.append(count_launches(call))
        call()
        torch.cuda.synchronize()
        lib.pqc_destroy(h)
        got.append((idx.cpu().numpy(), out.cpu().numpy()))
    assert launches == [2, 3]
    np.testing.assert_array_equal(got[0][0], got[1][0])
    assert check_indices(p, got[1][0], units=list(range(0, w.batch * w.n_kv_heads, 7))) == 0
    for idx, out in got:
        assert attn_error(p, idx, out, units=list(range(0, w.batch * w.n_kv_heads, 7))) <= ATTN_TOL[w.dtype]
