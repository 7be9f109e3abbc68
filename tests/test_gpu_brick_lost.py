"""A launch of bricks that lost a value between its workgroups is an error, also
where a number of cycles was asked for and no residual is looked at; the
context's next solve launches its passes, with the bits they have."""
import ctypes

import numpy as np
import pytest

from paper_1302_3663_amd import _lib as L
from paper_1302_3663_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("restart", [0, 3])
@pytest.mark.parametrize("precision", [L.IBB_FP64, L.IBB_FP32_REFINED])
def test_lost_value_is_an_error(precision, restart):
    from paper_1302_3663_amd import ibmg
    print("precision", precision, "restart", restart, flush=True)
    case = synth.tiny_3d(n=(16, 16, 32))
    case = dict(case, params=dict(case["params"], krylov_restart=restart))
    ctx = ibmg.from_case(case, precision=precision, inner_cycles=2)
    b = torch.as_tensor(np.random.default_rng(3).standard_normal(ctx.n_face), device="cuda:0")
    x0 = torch.zeros_like(b)
    want, _ = ctx.mg_solve(1, b, x0, exact=2)
    fn = ctx.lib.ibmg_bricks_lose
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int]
    assert fn(ctx.ctx, 1) == 0   # the count a workgroup leaves behind; nothing is lost here
    with pytest.raises(L.IbbError) as e:
        ctx.mg_solve(1, b, x0, exact=2)
    assert e.value.status == L.IBB_ENUMERIC
    got, _ = ctx.mg_solve(1, b, x0, exact=2)
    assert torch.equal(got, want) and bool(torch.isfinite(got).all())
    ctx.close()
