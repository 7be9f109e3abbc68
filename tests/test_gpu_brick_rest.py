"""A context whose launch of bricks did not find its workgroups together takes
the next solve pass by pass and then returns to bricks; the bits are the same."""
import ctypes

import numpy as np
import pytest

from paper_1302_3663_amd import _lib as L
from paper_1302_3663_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SMOOTH_U = {L.IBB_FP64: 0, L.IBB_FP32_REFINED: 2}   # launched colour passes of the velocity on the finest level


@pytest.mark.parametrize("restart", [0, 3])
@pytest.mark.parametrize("precision", [L.IBB_FP64, L.IBB_FP32_REFINED])
def test_bricks_come_back(precision, restart):
    from paper_1302_3663_amd import ibmg
    print("precision", precision, "restart", restart, flush=True)
    case = synth.tiny_3d(n=(16, 16, 32))
    case = dict(case, params=dict(case["params"], krylov_restart=restart))
    ctx = ibmg.from_case(case, precision=precision, inner_cycles=2)
    b = torch.as_tensor(np.random.default_rng(3).standard_normal(ctx.n_face), device="cuda:0")
    x0 = torch.zeros_like(b)
    fn = ctx.lib.ibmg_bricks_control
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_longlong, ctypes.POINTER(ctypes.c_int),
                   ctypes.POINTER(ctypes.c_int)]

    def solve(limit=-1):
        """The iterate, the launched passes of the finest level and the launches on one workgroup so far."""
        solo = ctypes.c_int()
        assert fn(ctx.ctx, 1, limit, None, None) == 0
        ctx.profile_enable(True)
        x, _ = ctx.mg_solve(1, b, x0, exact=3)
        launched = ctx.profile_read(SMOOTH_U[precision])["launches"]
        ctx.profile_enable(False)
        assert fn(ctx.ctx, 1, -1, None, ctypes.byref(solo)) == 0
        return x, launched, solo.value

    ctx._solver_scratch()
    want, launched, solo = solve()
    assert launched == 0 and solo == 0
    slow, launched, solo = solve(limit=1)      # 10 ns to find the others
    assert launched > 0 and solo == 1          # the first iteration alone, the others pass by pass
    rest, launched, solo = solve()
    assert launched > 0 and solo == 1
    back, launched, solo = solve()
    assert launched == 0 and solo == 1
    for x in (slow, rest, back):
        assert torch.equal(x, want)
    ctx.close()
