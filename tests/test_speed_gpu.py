"""Sizes at which a call once took a multiple of what a call of the same traffic takes: each is held to a multiple of such
a neighbour, timed beside it on the same device (GPU time of graph replays, the best of several)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _us(call, calls=4):
    """GPU time of one call, us."""
    import torch
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(calls):
            call()
    best = float("inf")
    for _ in range(8):
        start, stop = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        start.record()
        graph.replay()
        stop.record()
        torch.cuda.synchronize()
        best = min(best, start.elapsed_time(stop) / calls * 1e3)
    return best


def _embedding_us(ids, D, V, dtype, presorted=True):
    import torch
    from paper_2411_00999_amd import binding
    B, T = ids.shape
    ids = torch.from_numpy(np.ascontiguousarray(ids, dtype=np.int64)).cuda()
    g = (torch.randn(B, T, D, device="cuda") * 1e-3).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    out = dict(w=torch.empty(V, D, device="cuda"), s=torch.empty(B, device="cuda"), big_sq=torch.empty(1, device="cuda"),
               workspace=torch.empty(binding.load().embedding_pegn_workspace_bytes(B, T, D, V), dtype=torch.uint8, device="cuda"))
    if not presorted:
        return _us(lambda: binding.embedding_pegn(ids, g, V, **out))
    in_order = binding.embedding_sort_ids(ids, V)
    return _us(lambda: binding.embedding_pegn_presorted(*in_order, g, V, **out))


@pytest.mark.parametrize("B,T,D,V,dtype,times", [
    (69, 4815, 26, 920, "bf16", 2.0),        # with one workgroup for all of an id's rows: 6.7 times
    (36, 4546, 64, 2096, "f32", 1.8),        # 2.6
    (73, 4476, 1, 6, "f32", 2.0),            # 3.3
])
def test_embedding_of_one_id(B, T, D, V, dtype, times):
    """A batch of one id against one whose ids all occur about equally often."""
    spread = np.random.default_rng(1).integers(0, V, (B, T))
    one, many = _embedding_us(np.full((B, T), V - 1), D, V, dtype), _embedding_us(spread, D, V, dtype)
    assert one < times * many, (one, many)


@pytest.mark.parametrize("B,T,D,V,times", [
    (8, 1024, 8, 1000000, 3.0),              # with a search per row and rows far apart: 12 times
    (2, 36, 3, 1263217, 6.0),                # 14
])
def test_embedding_over_a_large_vocabulary(B, T, D, V, times):
    """Rows that no id selects cost what filling memory costs: the call against the call over a small vocabulary and a
    fill of as much memory."""
    import torch
    ids = np.random.default_rng(2).integers(0, 200, (B, T))
    large, small = _embedding_us(ids, D, V, "bf16"), _embedding_us(ids, D, 200, "bf16")
    w = torch.empty(V, D, device="cuda")
    fill = _us(lambda: w.zero_())
    assert large < small + times * fill, (large, small, fill)


def test_embedding_of_rows_that_end_inside_a_line():
    """Against rows of 32 bytes more, which are whole lines (1.06 to 1.09 times in twelve pairs; with the shares of the fill meeting
    inside a line 1.23 to 1.25)."""
    ids = np.random.default_rng(3).permutation(50257)[np.random.default_rng(4).zipf(1.2, (3, 705)) % 50257]
    inside, whole = _embedding_us(ids, 1688, 50257, "bf16", False), _embedding_us(ids, 1696, 50257, "bf16", False)
    assert inside < 1.15 * whole, (inside, whole)


def _linear_us(B, T, K, L, dtype, accumulate=False, less=0):
    import torch
    from paper_2411_00999_amd import binding
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x, g = torch.randn(B, T, K, device="cuda").to(dt), torch.randn(B, T, L, device="cuda").to(dt)
    nbytes = max(256, binding.load().linear_pegn_workspace_bytes(B, T, K, L, binding.BF16 if dtype == "bf16" else binding.F32))
    out = dict(w=torch.empty(K, L, device="cuda"), s=torch.empty(B, device="cuda"), big_sq=torch.empty(1, device="cuda"),
               workspace=torch.empty(nbytes - less, dtype=torch.uint8, device="cuda"))
    if accumulate:
        out["w"].zero_()
    return _us(lambda: binding.linear_pegn(x, g, accumulate=accumulate, **out), calls=10)


@pytest.mark.parametrize("B,T,K,L,dtype,times", [
    (2, 4, 9, 3, "bf16", 2.0),               # on the matrix cores: 3.4 times
    (1, 8, 257, 300, "f32", 2.2),            # 3.4
    (3, 8, 1000, 499, "bf16", 3.2),          # 4.5
])
def test_linear_of_a_few_short_ragged_examples(B, T, K, L, dtype, times):
    """Against the smallest call there is."""
    few, least = _linear_us(B, T, K, L, dtype), _linear_us(1, 1, 1, 1, "f32")
    assert few < times * least, (few, least)


def test_forward_of_ragged_rows_with_gamma_of_the_other_type():
    """fp32 gamma and beta over bf16 rows cost what bf16 ones do (element by element: 3.3 times)."""
    import torch
    from paper_2411_00999_amd import binding
    B, T, D = 8, 500, 1001
    x = torch.randn(B, T, D, device="cuda").bfloat16()
    y, mean, rstd = torch.empty_like(x), torch.empty(B, T, device="cuda"), torch.empty(B, T, device="cuda")
    us = {}
    for dt in (torch.bfloat16, torch.float32):
        gamma, beta = torch.ones(D, device="cuda", dtype=dt), torch.zeros(D, device="cuda", dtype=dt)
        us[dt] = _us(lambda: binding.ln_fwd(x, gamma, beta, 1e-5, y=y, mean=mean, rstd=rstd), calls=10)
    assert us[torch.float32] < 2.0 * us[torch.bfloat16], us


def _deferred_us(B, T, D, dtype, layers=16):
    """GPU time of the deferred reduction of some layers, us."""
    import torch
    from paper_2411_00999_amd import binding
    dt, code = (torch.bfloat16, binding.BF16) if dtype == "bf16" else (torch.float32, binding.F32)
    x, dy, gamma = torch.randn(B, T, D, device="cuda").to(dt), torch.randn(B, T, D, device="cuda").to(dt), torch.ones(D, device="cuda", dtype=dt)
    workspaces = [binding.alloc_workspace(B, T, D, code) for _ in range(layers)]
    keep = [binding.ln_bwd_pegn(x, dy, gamma, 1e-5, workspace=w, deferred=True) for w in workspaces]
    us = _us(lambda: binding.reduce_deferred(workspaces, B, T, D, code), calls=10)
    return us, keep


def test_deferred_reduction_of_many_short_examples():
    """512 examples of a chunk each against 64 of eight chunks each: the same sums of the same 512 chunks (with a
    workgroup sent for every example in vain: 1.7 times)."""
    many, few = _deferred_us(512, 64, 1024, "bf16")[0], _deferred_us(64, 512, 1024, "bf16")[0]
    assert many < 1.45 * few, (many, few)


@pytest.mark.parametrize("B,T,K,L", [(1, 1822, 640, 2624), (4, 97, 7360, 11520), (9, 160, 5632, 11136), (1, 2006, 1848, 408)])
def test_linear_accumulated_by_the_larger_tile(B, T, K, L):
    """Adding to w costs the reading of it: 1.0 to 1.4 times the call (load by load, each waited for: 2.3 to 4.7 times)."""
    added, written = _linear_us(B, T, K, L, "bf16", accumulate=True), _linear_us(B, T, K, L, "bf16")
    assert added < 1.7 * written, (added, written)



@pytest.mark.parametrize("B,T,K,L", [(15, 513, 7296, 8), (8, 503, 7488, 64), (3, 695, 16, 3776), (90, 153, 2368, 8)])
def test_linear_of_narrow_matrices_in_the_larger_tile(B, T, K, L):
    """Against the smaller tile, which runs in one byte less of workspace (0.81 to 0.99 times; with whole tiles in the splits' sums
    1.16 to 1.23)."""
    larger, smaller = _linear_us(B, T, K, L, "bf16"), _linear_us(B, T, K, L, "bf16", less=1)
    assert larger < 1.08 * smaller, (larger, smaller)
