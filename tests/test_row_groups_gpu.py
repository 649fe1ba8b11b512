"""The row kernel's launch shapes around the lines of the planning rules: eight row groups a workgroup for rows of one wave
(chunks of two rows a group and just below, chunks that do not come out even, ragged rows) and half as many workgroups
for narrow rows.  Against the oracle, with the tolerances of the other parity tests."""
import pytest

from paper_2411_00999_amd import binding, workloads
import parity_util as pu
import test_parity_gpu as tp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,D,dtype,groups", [
    (3, 16, 768, "bf16", 8), (3, 15, 768, "bf16", 4), (5, 33, 520, "bf16", 8), (2, 47, 1001, "bf16", 8),
    (130, 31, 768, "bf16", 8), (100, 24, 520, "bf16", 8), (40, 17, 1024, "f32", 8), (34, 500, 520, "bf16", 4),
    (8, 1024, 264, "bf16", 4), (8, 1024, 500, "f32", 4), (3, 2731, 250, "bf16", 4)])
def test_row_groups(B, T, D, dtype, groups):
    code = binding.BF16 if dtype == "bf16" else binding.F32
    vectors = D % (8 if dtype == "bf16" else 4) == 0
    assert binding.plan_query(B, T, D, code, aligned=vectors)["row_groups"] == groups
    inp = workloads.make_inputs(2, B=B, T=T, D=D, dtype=dtype, signal=1e-3)
    ref = tp._oracle(inp)
    for saved in (False, True):
        pu.compare_with_oracle(inp, pu.run_gpu(inp, saved_stats=saved), ref)
    pu.compare_with_oracle(inp, pu.run_gpu(inp, pegn=False), ref, pegn=False)
