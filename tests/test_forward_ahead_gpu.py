"""The forward that loads rows ahead: one row more than the waves there are (rows of one wave), two to four rows a
workgroup and one beyond (rows of two waves), full and partly empty lanes, gamma of both types, with and without beta."""
import numpy as np
import pytest

import oracle
from paper_2411_00999_amd import workloads
import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,D,dtype", [
    (5, 3277, 136, "bf16"), (5, 3277, 520, "bf16"), (17, 964, 1024, "bf16"), (5, 3277, 600, "f32"),
    (1, 2049, 1032, "bf16"), (3, 1000, 2048, "bf16"), (8, 1024, 1288, "bf16"), (1, 8193, 1032, "bf16"), (1, 2049, 1028, "f32")])
def test_forward_ahead(B, T, D, dtype):
    import torch
    from paper_2411_00999_amd import binding
    inp = workloads.make_inputs(2, B=B, T=T, D=D, dtype=dtype)
    x, gamma, beta = (pu.to_device(a, inp.dtype) for a in (inp.x, inp.gamma, inp.beta))
    bf = dtype == "bf16"
    tol = pu.TOL_BF16 if bf else pu.TOL_F32
    y, mean, rstd = binding.ln_fwd(x, gamma, beta, inp.eps)
    other = torch.float32 if bf else torch.bfloat16
    z, _, _ = binding.ln_fwd(x, gamma.to(other), beta.to(other), inp.eps)
    v, rms = binding.rms_fwd(x, gamma, inp.eps)
    m2, r2 = binding.ln_fwd_stats(x, inp.eps)
    torch.cuda.synchronize()
    pu.check_close("y", pu.to_host64(y), oracle.ln_fwd(inp.x, inp.gamma, inp.beta, inp.eps), tol, bf16_output=bf)
    assert torch.equal(m2, mean) and torch.equal(r2, rstd)
    want = oracle.ln_fwd(inp.x, pu.to_host64(gamma.to(other)), pu.to_host64(beta.to(other)), inp.eps)
    pu.check_close("y, gamma of the other type", pu.to_host64(z), want, tol, bf16_output=bf)
    want, want_rstd = oracle.rms_fwd(inp.x, inp.gamma, inp.eps)
    pu.check_close("rms y", pu.to_host64(v), want, tol, bf16_output=bf)
    np.testing.assert_allclose(pu.to_host64(rms), want_rstd, rtol=pu.TOL_F32)
