"""The linear layer's larger tile at the shapes where it can go wrong: one column of tiles and edges in both directions, examples
whose last stage is short, of one stage and of two, whole rounds of tiles alone and beside split and unsplit ones, one and many
splits, accumulation, an infinity that must stay in its example, less workspace than it asks for (the smaller tile's).  That the
larger tile runs, and with which shares, is asserted by the plan.

Reference: the products in fp64 on the device.  Every product is exact in fp32, so an output of n additions is off by at most
n 2^-24 of the sum of its terms' magnitudes; the norms, sums of squares of such outputs, are held to 1e-5 like those of the
other linear kernels."""
import pytest

pytestmark = pytest.mark.gpu


def _inputs(B, T, K, L, seed=1):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    x = torch.randn((B, T, K), generator=gen, device="cuda").bfloat16()
    g = (torch.randn((B, T, L), generator=gen, device="cuda") * 1e-3 + torch.randn((T, L), generator=gen, device="cuda") * 5e-4).bfloat16()
    return x, g


def _check(x, g, got, w0=None):
    import torch
    B, T, K = x.shape
    w = torch.zeros((K, g.shape[2]), dtype=torch.float64, device="cuda") if w0 is None else w0.double()
    size = w.abs()
    s = []
    for b in range(B):
        xt, gb = x[b].double().t().contiguous(), g[b].double()
        wb = torch.mm(xt, gb)
        s.append(wb.square().sum())
        w = w + wb
        size = size + torch.mm(xt.abs(), gb.abs())
    torch.cuda.synchronize()
    assert bool(((got[0].double() - w).abs() <= (T + B) * 2.0 ** -24 * size + 1e-30).all())
    torch.testing.assert_close(got[1].double(), torch.stack(s), rtol=1e-5, atol=0)
    torch.testing.assert_close(got[2].double(), w.square().sum().reshape(1), rtol=1e-5, atol=0)


def _shares(B, T, K, L):
    """Tiles that a workgroup finishes whatever the splits, other tiles, splits of those."""
    from paper_2411_00999_amd import binding
    plan = binding.linear_plan_query(B, T, K, L, binding.BF16)
    assert plan["kernel"] == "matrix_larger_tile", plan
    return plan["whole_tiles"], plan["tiles"] - plan["whole_tiles"], plan["splits"]


@pytest.mark.parametrize("B,T,K,L,shares", [
    (2, 1000, 8, 8, (0, 1, 2)), (2, 2048, 264, 200, (0, 4, 2)), (3, 1025, 768, 584, (0, 12, 3)), (4, 601, 1032, 3000, (0, 80, 2)),
    (5, 515, 2056, 2600, (0, 126, 2)), (2, 640, 4104, 4000, (256, 101, 2)), (3, 545, 4096, 3080, (256, 16, 3)),
    (13, 700, 64, 1000, (0, 6, 13)), (1, 3000, 1496, 8000, (0, 252, 1)),
    (6, 100, 5224, 6232, (512, 181, 1)), (8, 33, 4904, 1632, (0, 180, 1)), (40, 64, 776, 3000, (0, 64, 4)),
    (16, 16, 3072, 4032, (0, 252, 1)), (24, 1, 1936, 6048, (256, 0, 1)), (12, 64, 1928, 6000, (256, 0, 1)),
    (16, 33, 2048, 6144, (256, 0, 1))])
def test_linear_larger_tile(B, T, K, L, shares):
    import torch
    from paper_2411_00999_amd import binding
    assert _shares(B, T, K, L) == shares
    x, g = _inputs(B, T, K, L)
    got = binding.linear_pegn(x, g)
    _check(x, g, got)
    again = binding.linear_pegn(x, g)
    assert all(torch.equal(a, b) for a, b in zip(got, again))            # the same bits
    w0 = torch.randn((K, L), device="cuda") * 1e-2
    _check(x, g, binding.linear_pegn(x, g, w=w0.clone(), accumulate=True), w0=w0)


@pytest.mark.parametrize("B,T,K,L", [(4, 601, 1032, 3000), (2, 2048, 264, 200)])
def test_linear_larger_tile_in_less_workspace(B, T, K, L):
    import torch
    from paper_2411_00999_amd import binding
    assert _shares(B, T, K, L)[2] == 2
    x, g = _inputs(B, T, K, L)
    need = binding.load().linear_pegn_workspace_bytes(B, T, K, L, binding.BF16)
    for nbytes in (need, need - 1, need // 2, need // 4):
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        try:
            _check(x, g, binding.linear_pegn(x, g, workspace=ws))
        except binding.LnpegnError as e:                               # less than the smaller tile's
            assert e.status == 3 and nbytes <= need // 2


def test_linear_larger_tile_keeps_infinities_to_their_example():
    import torch
    from paper_2411_00999_amd import binding
    assert _shares(3, 1025, 768, 584) == (0, 12, 3)
    x, g = _inputs(3, 1025, 768, 584)
    g[1, 1024, 583] = float("inf")                                         # the last row and column of an example
    _, s, _ = binding.linear_pegn(x, g)
    torch.cuda.synchronize()
    assert not bool(torch.isfinite(s[1])) and bool(torch.isfinite(s[[0, 2]]).all())


@pytest.mark.parametrize("B,T,K,L", [(2, 1025, 2048, 2560), (2, 1025, 2048, 5120)])
def test_linear_larger_tile_norm_of_an_infinite_gradient(B, T, K, L):
    """An infinity in x meets the zeros behind the last tile's 64 columns: outputs that are not there, and not counted."""
    import torch
    from paper_2411_00999_amd import binding
    _shares(B, T, K, L)
    x, g = _inputs(B, T, K, L)
    x[1, 1, K - 1] = float("inf")
    g[1, 1] = g[1, 1].abs() + 1e-4                                         # no zeros, whose product would be no number in truth
    _, s, big_sq = binding.linear_pegn(x, g)
    torch.cuda.synchronize()
    assert bool(torch.isinf(s[1])) and bool(torch.isfinite(s[0])) and bool(torch.isinf(big_sq[0]))


@pytest.mark.parametrize("B,T,K,L", [(5, 515, 72, 2600), (3, 1025, 768, 584), (13, 700, 64, 1000), (3, 545, 4096, 3080)])
def test_linear_larger_tile_reads_no_sums_that_it_has_not_written(B, T, K, L):
    """The parts of a tile behind the matrix are not in the splits' sums; the workspace holds no numbers before the call."""
    import torch
    from paper_2411_00999_amd import binding
    assert _shares(B, T, K, L)[2] > 1
    x, g = _inputs(B, T, K, L)
    ws = torch.full((binding.load().linear_pegn_workspace_bytes(B, T, K, L, binding.BF16),), 255, dtype=torch.uint8, device="cuda")
    _check(x, g, binding.linear_pegn(x, g, workspace=ws))
