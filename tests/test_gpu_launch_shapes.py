"""Launch shapes of a decode step, read from a recorded graph: which select kernel runs and on how many tokens per workgroup, how many
workgroups finish a step, and how many of them share a compute unit.  Results do not depend on any of it (the other tests compare
those); speed does."""
import ctypes

import pytest
import torch

from paper_2407_12820_amd import workloads as wl

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _NodeParams(ctypes.Structure):  # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("args", ctypes.c_void_p), ("lds", ctypes.c_uint)]


@pytest.fixture(scope="module")
def pqc():
    from paper_2407_12820_amd import binding
    binding.load()
    return binding


def _kernels(pqc, call):
    """Launches of `call`, in order: (workgroups per unit, units, threads, dynamic LDS, workgroups resident per compute unit)."""
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph, stream=torch.cuda.Stream(device=DEV)):
        call()
    hip, raw = pqc.load(), ctypes.c_void_p(graph.raw_cuda_graph())  # (the library is linked to the HIP runtime)
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(n)) == 0
    out = []
    for node in nodes:
        p, resident = _NodeParams(), ctypes.c_int(0)
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        assert hip.hipOccupancyMaxActiveBlocksPerMultiprocessor(ctypes.byref(resident), ctypes.c_void_p(p.func), ctypes.c_int(p.block.x),
                                                                ctypes.c_size_t(p.lds)) == 0
        out.append((p.grid.x, p.grid.y, p.block.x, p.lds, resident.value))
    return out


def _step(pqc, units, group, n_tokens, m, c, den, dtype, indexed):
    w = wl.Workload(name="launches", batch=units, n_q_heads=group, n_kv_heads=1, head_dim=128, n_tokens=n_tokens, pq_m=m, pq_centroids=c,
                    topk=n_tokens // den, n_init=4, n_local=64, dtype=dtype, kmeans_iters=1, recipe="plain")
    print(f"[case] {w} indexed={indexed}", flush=True)
    kv = torch.bfloat16 if dtype == "bf16" else torch.float32
    new = lambda shape, t: torch.zeros(shape, dtype=t, device=DEV)
    k = new((units, 1, n_tokens, 128), kv)
    q, cent, codes = new((units, group, 128), kv), new((units, 1, m, c, 128 // m), torch.float32), new((units, 1, n_tokens, m), torch.uint8)
    ctx = pqc.PQCache(w, DEV)
    outs = ctx.empty_outputs()
    if indexed:
        counts = pqc.pair_counts(w, codes)
        return _kernels(pqc, lambda: ctx.decode_indexed(q, cent, codes, counts, k, k, *outs))
    return _kernels(pqc, lambda: ctx.decode(q, cent, codes, k, k, *outs))


@pytest.mark.parametrize("units, group, n_tokens, m, c", [(64, 4, 2048, 2, 64), (200, 2, 2056, 2, 64), (8, 8, 8000, 1, 64), (40, 1, 20011, 4, 64)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_workgroups_that_finish_a_step_share_a_compute_unit(pqc, units, group, n_tokens, m, c, dtype):
    assert _step(pqc, units, group, n_tokens, m, c, 10, dtype, False)[-1][4] >= 2


@pytest.mark.parametrize("units, group, n_tokens, m, c, workgroups", [
    (8, 4, 32768, 2, 64, 16 + 6), (12, 4, 20011, 4, 64, 16 + 4), (7, 8, 4096, 4, 64, 32 + 4), (24, 8, 20011, 4, 64, 8 + 2), (16, 8, 4096, 2, 64, 8 + 6),
    (64, 1, 20000, 4, 256, 1 + 2), (2, 1, 3000, 2, 64, 4 + 4), (32, 8, 4096, 4, 256, 8 + 4),
    # large tie classes: four workgroups per head up to two per compute unit
    (24, 4, 40000, 1, 256, 16 + 4), (14, 8, 8000, 1, 64, 32 + 4), (8, 8, 131072, 2, 64, 32 + 4), (64, 1, 8000, 1, 64, 4 + 2)])
def test_workgroups_that_finish_a_unit(pqc, units, group, n_tokens, m, c, workgroups):
    grid, y, threads, _, _ = _step(pqc, units, group, n_tokens, m, c, 10, "bf16", False)[-1]
    assert (grid, y, threads) == (workgroups, units, 512)


def test_tokens_of_a_workgroup_end_with_the_unit(pqc):
    # more units than workgroups fit at once: a select workgroup's list (two bytes per token, and one entry per thread behind it) is that of the next
    # power of two, not of the largest workgroup
    for units, n_tokens, tokens in ((520, 600, 1024), (520, 1024, 1024), (520, 1025, 2048), (8, 600, 512)):
        grid, _, threads, lds, _ = _step(pqc, units, 1, n_tokens, 8, 16, 10, "bf16", False)[1]
        assert (grid, threads, lds) == (-(-n_tokens // tokens), 256, 2 * (tokens + 256))
    lists = [_step(pqc, units, 4, n_tokens, 2, 64, 10, "bf16", False)[0][3] for units, n_tokens in ((264, 600), (264, 2048), (264, 4097))]
    assert (lists[1] - lists[0], lists[2] - lists[0]) == (2 * 1024, 2 * 7168)


@pytest.mark.parametrize("units, group, n_tokens, dtype, grid, threads, resident", [
    (8, 4, 4096, "bf16", 8, 512, 1), (64, 1, 16384, "bf16", 4, 512, 1), (100, 1, 16384, "bf16", 2, 512, 1), (256, 2, 2048, "bf16", 1, 512, 1),
    (264, 4, 2048, "bf16", 1, 256, 2), (264, 8, 8192, "bf16", 1, 256, 2), (130, 2, 20000, "bf16", 3, 256, 2), (100, 1, 9000, "bf16", 5, 256, 2),
    (8, 2, 4096, "f32", 8, 512, 2), (100, 1, 20000, "f32", 5, 512, 2), (600, 2, 600, "f32", 1, 512, 2), (300, 4, 2048, "f32", 1, 256, 2)])
def test_select_kernel_of_a_step_with_given_pair_counts(pqc, units, group, n_tokens, dtype, grid, threads, resident):
    x, y, t, _, r = _step(pqc, units, group, n_tokens, 2, 64, 10, dtype, True)[0]
    assert (x, y, t) == (grid, units, threads) and r >= resident
