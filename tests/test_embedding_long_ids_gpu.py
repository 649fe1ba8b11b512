"""embedding_pegn with ids that fill hundreds to thousands of positions: their parked sums are shared out over workgroups
in parts of 1024 sorted positions (16385 to 65536 positions; 4096 below that, 2048 and more above), cut only where an id
has 64 positions on either side."""
import numpy as np
import pytest

import parity_util as pu
from paper_2411_00999_amd import workloads

pytestmark = pytest.mark.gpu

EDGES = [63, 64, 65, 100, 127, 128, 129, 130, 191, 900, 959, 960, 961, 1023, 1024, 1025, 1087, 1088, 1089, 1090, 2047,
         2048, 2200, 3100, 4031, 4160, 4161, 5000]


def _ids(rng, n, V, lengths):
    """n ids in ascending order whose segments have these lengths (the last takes what is left)."""
    names = np.sort(rng.choice(V, size=len(lengths) + 1, replace=False))
    flat = np.concatenate([np.full(m, v) for m, v in zip(lengths, names)])[:n]
    return np.concatenate([flat, np.full(n - len(flat), names[-1])]).astype(np.int64)


def _check(ids, g, V, dtype, w0=None):
    import torch
    from oracle import embedding_pegn_oracle as emb
    from paper_2411_00999_amd import binding
    keep = (ids >= 0) & (ids < V)
    ref = emb.embedding_pegn(np.where(keep, ids, 0), g * keep[..., None], V)
    want_w = ref["w"] + (0 if w0 is None else w0.astype(np.float32).astype(np.float64))
    idd, gd = torch.from_numpy(ids).cuda(), pu.to_device(g, dtype)
    runs = []
    for _ in range(3):                               # whichever workgroup arrives last, the bits are the same
        w = None if w0 is None else torch.from_numpy(w0.astype(np.float32)).cuda()
        runs.append(binding.embedding_pegn(idd, gd, V, w=w, accumulate=w0 is not None))
    sk, sp = binding.embedding_sort_ids(idd, V)
    w = None if w0 is None else torch.from_numpy(w0.astype(np.float32)).cuda()
    runs.append(binding.embedding_pegn_presorted(sk, sp, gd, V, w=w, accumulate=w0 is not None))
    torch.cuda.synchronize()
    for again in runs[1:]:
        assert all(torch.equal(p, q) for p, q in zip(runs[0], again))
    got_w, s, big = (pu.to_host64(t) for t in runs[0])
    pu.check_close("w", got_w, want_w, pu.TOL_SUMS)
    np.testing.assert_allclose(s, ref["s"], rtol=pu.TOL_SUMS)
    np.testing.assert_allclose(big, [np.sum(got_w ** 2)], rtol=pu.TOL_SUMS)


@pytest.mark.parametrize("dtype,D", [("bf16", 8), ("f32", 26), ("bf16", 520), ("f32", 516), ("bf16", 1100)])
@pytest.mark.parametrize("B,T,order", [(1, 17001, "sorted"), (3, 5667, "sorted"), (3, 5667, "mixed"), (17001, 1, "mixed"),
                                       (600, 30, "mixed"), (3, 5003, "sorted"), (7, 2001, "mixed")])
def test_segments_around_the_cuts(dtype, D, B, T, order):
    """Segments of every length near the cuts' limits, from random places; runs over several parts (one example, or ids
    in the order of the positions), several runs to a part, and runs of one position."""
    rng = np.random.default_rng(workloads.BASE_SEED + B + D)
    n, V = B * T, 200
    lengths = []
    while sum(lengths) < n:
        lengths += [int(rng.integers(1, 80))] * int(rng.integers(0, 4)) + [int(rng.choice(EDGES))]
    flat = _ids(rng, n, V, lengths)
    if order == "mixed":
        flat = rng.permutation(flat)
    ids = flat.reshape(B, T)
    ids[rng.random((B, T)) < 0.01] = V + 7           # skipped
    _, g = workloads.make_embedding_inputs(85, B, T, D, 50, dtype)
    _check(ids, g, V, dtype)
    if D in (26, 520):
        _check(ids, g, V, dtype, w0=rng.normal(0, 1e-2, (V, D)))


@pytest.mark.parametrize("before", [0, 1, 895, 896, 897, 959, 960, 961, 1023, 1024, 1025])
@pytest.mark.parametrize("length", [65, 127, 128, 129, 1087, 1088, 1089, 1153, 2113])
def test_one_long_id_at_every_offset_from_a_cut(before, length):
    """One id behind `before` others, over examples that end at odd places."""
    rng = np.random.default_rng(before * 10000 + length)
    B, T, D, V = 3, 5511, 16, 5000
    flat = np.arange(B * T, dtype=np.int64)[:before]
    rest = 4000 + np.arange(B * T - before - length, dtype=np.int64) % 900
    flat = np.concatenate([flat, np.full(length, 3900), np.sort(rest)])[:B * T]
    ids = rng.permutation(flat) if before % 2 else flat
    _, g = workloads.make_embedding_inputs(86, B, T, D, 50, "f32")
    _check(ids.reshape(B, T), g, V, "f32")


@pytest.mark.parametrize("B,T,D", [(130, 1031, 8), (1, 134030, 8), (2, 1100000, 4)])
def test_one_id_beyond_the_own_sort(B, T, D):
    """The counters' place in the other workspace layout, and (the last) more parts than a wave lists at a time."""
    V = 7
    _, g = workloads.make_embedding_inputs(87, B, T, D, V, "f32")
    ids = np.full((B, T), 3, dtype=np.int64)
    ids[:, ::1000] = 5
    _check(ids, g, V, "f32")


@pytest.mark.parametrize("V,D,off,kind", [
    (70001, 8, 0, "few"), (70001, 1, 3, "few"), (1000, 3, 1, "few"), (64, 5, 2, "all"), (65, 5, 1, "all but one"),
    (200, 4, 0, "every other"), (300, 7, 1, "every other"), (129, 260, 0, "crowded"), (500, 2, 2, "crowded"),
    (5000, 1021, 3, "few"), (9, 20000, 1, "few"), (1, 12, 1, "few"), (3000, 64, 0, "out of range"),
])
def test_rows_no_id_selects_are_zero(V, D, off, kind):
    """The fill over rows of any width and address, with none, some, most of 64 neighbouring rows present, many positions
    among them, and nothing outside w' touched."""
    import torch
    from paper_2411_00999_amd import binding
    rng = np.random.default_rng(V + D)
    if kind == "few":
        ids = rng.integers(0, V, (2, 30))
        ids[0, 0], ids[0, 1] = 0, V - 1
    elif kind == "all":
        ids = rng.permutation(np.arange(V)).reshape(2, -1)
    elif kind == "all but one":
        ids = rng.permutation(np.delete(np.arange(V), V // 2)).reshape(2, -1)
    elif kind == "every other":
        ids = np.arange(V // 2)[None] * 2
    elif kind == "crowded":                          # more than 512 positions on the rows of one wave
        ids = rng.choice([3, 5, 6, 63, 64, V - 2], (3, 400))
    else:
        ids = np.full((2, 20), V + 1)
    ids = ids.astype(np.int64)
    g = torch.ones((*ids.shape, D), device="cuda")
    flat = torch.full((V * D + off + 5,), 7.0, device="cuda")
    w = flat[off:off + V * D].view(V, D)
    _, s, big = binding.embedding_pegn(torch.from_numpy(ids).cuda(), g, V, w=w)
    torch.cuda.synchronize()
    count = np.bincount(ids[ids < V].reshape(-1), minlength=V)
    np.testing.assert_array_equal(w.cpu().numpy(), np.repeat(count[:, None], D, 1).astype(np.float32))
    assert bool((flat[:off] == 7).all()) and bool((flat[off + V * D:] == 7).all())


def test_positions_just_below_the_limit():
    """Nearly 2^28 positions: the workgroups of the runs, the medium segments and the fill are more than one launch holds.
    Whole numbers, so sums are exact in any order."""
    import torch
    from paper_2411_00999_amd import binding
    n, D, V = (1 << 28) - 200000, 1, 1 << 24
    ids = torch.randint(0, V // 2, (1, n), device="cuda", dtype=torch.int32) * 2      # about 32 positions to an id
    ids[0, :5000], ids[0, -300:] = 8, 1
    g = torch.randint(-1, 2, (1, n, D), device="cuda", dtype=torch.int8).to(torch.bfloat16)
    w, s, big = binding.embedding_pegn(ids, g, V)
    want = torch.zeros(V, device="cuda").index_add_(0, ids[0], g.view(-1).float())
    assert torch.equal(w.view(-1), want)
    square = float(want.double().square().sum())
    np.testing.assert_allclose([float(s[0]), float(big[0])], square, rtol=pu.TOL_SUMS)
