"""The zero fill of w' beside the sort, kernel A and kernel B: a w' of less than the first share, rows of widths that end off a
16-byte boundary at its end, unaligned w', a w' whose fill is shared by all three, in rows that
are a line of 128 bytes by fours, by eights and not at all.  Every element of w' is compared, from a
buffer that held something else."""
import numpy as np
import pytest

from paper_2411_00999_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,T,D,V,off", [
    ("bf16", 2, 50, 24, 700, 0), ("f32", 2, 50, 7, 3001, 0), ("f32", 1, 3, 1, 5, 0), ("bf16", 3, 33, 1001, 8400, 0),
    ("bf16", 3, 33, 1002, 8500, 0), ("f32", 4, 64, 128, 50257, 0), ("f32", 2, 40, 64, 9000, 1), ("bf16", 5, 1000, 520, 50257, 0),
    ("f32", 8, 36, 840, 37197, 0), ("bf16", 3, 100, 36, 999999, 0), ("f32", 8, 600, 552, 50257, 0), ("bf16", 4, 64, 2049, 30001, 0),
    ("bf16", 2, 100, 840, 37197, 4)])
def test_every_row_is_written(dtype, B, T, D, V, off):
    import torch
    from paper_2411_00999_amd import binding
    ids, g = workloads.make_embedding_inputs(3, B, T, D, V, dtype)
    i, x = torch.from_numpy(ids).cuda(), workloads.to_device(g, dtype)
    want = torch.zeros((V, D), dtype=torch.float64, device="cuda")
    want.index_add_(0, i.reshape(-1), x.double().reshape(-1, D))
    scale = torch.zeros((V, D), dtype=torch.float64, device="cuda")
    scale.index_add_(0, i.reshape(-1), x.double().abs().reshape(-1, D))
    order = binding.embedding_sort_ids(i, V)
    for sort in (False, True):
        w = torch.full((V * D + off,), 7.0, dtype=torch.float32, device="cuda")[off:].view(V, D)
        if sort:
            binding.embedding_pegn_presorted(*order, x, V, w=w)
        else:
            binding.embedding_pegn(i, x, V, w=w)
        torch.cuda.synchronize()
        # a sum of n fp32 values, each addition rounded: (n-1) 2^-24 of the sum of their magnitudes at most
        n = int(np.bincount(ids.ravel()).max())
        assert bool(((w.double() - want).abs() <= n * 2.0 ** -24 * scale).all())
        assert bool((w[scale == 0] == 0).all())
