"""Kernels that walk rows by waves: the momentum right-hand side (inner points
apart from those near an end of the domain) against the oracle; the velocity
residual and, on large boxes, the interpolation against the passes of a group,
which number the points through: the same bits."""
import numpy as np
import pytest

import oracle as O
from oracle import step as S
from paper_1302_3663_amd import _lib as L
from paper_1302_3663_amd import synth

from parity import rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def periodic(n):
    case = synth.tiny_3d(n=n, periodic_z=True, periodic_x=True)
    case["params"] = dict(case["params"], omega=1.5 * case["params"]["h"])
    return case


# no inner point, one, rows shorter and longer than a wave, every kind of end
GRIDS = {
    "2d_4x4": lambda: synth.tiny_2d(nx=4, ny=4),
    "2d_6x10": lambda: synth.tiny_2d(nx=6, ny=10),
    "2d_inout_130x6": lambda: synth.tiny_2d(nx=130, ny=6, inout=True),
    "3d_4x6x6": lambda: synth.tiny_3d(n=(4, 6, 6)),
    "3d_72x6x8": lambda: synth.tiny_3d(n=(72, 6, 8)),
    "3d_periodic_72x8x8": lambda: periodic((72, 8, 8)),
}


@pytest.mark.parametrize("name", sorted(GRIDS))
def test_momentum_rhs(name):
    from paper_1302_3663_amd import ibmg
    case = GRIDS[name]()
    rng = np.random.default_rng(3)
    case["u0"] = case["u0"] + 0.1 * rng.standard_normal(len(case["u0"]))
    print("case", name, flush=True)
    ctx = ibmg.from_case(case)
    st = S.State(case["params"], case["u0"], case["p0"], case["X"], case["ij"], case["rest"], case["K"])
    S.setup(st)
    got = host(ctx.momentum_rhs())
    ctx.close()
    # 1e-12: the bound of the other right-hand sides against the oracle
    assert rel(got, O.momentum_rhs(case["params"], st.u, st.rho, st.mu_c, st.mu_e, st.f)) < 1e-12


LARGE = {
    "3d_72x16x16": lambda: synth.tiny_3d(n=(72, 16, 16)),
    "3d_periodic_72x16x16": lambda: periodic((72, 16, 16)),
    # interpolation by rows on the finest level: 2^21 points and odd remainders
    "2d_2050x1026": lambda: synth.tiny_2d(nx=2050, ny=1026, inout=True),
    "2d_2048x1024": lambda: synth.tiny_2d(nx=2048, ny=1024),
}


@pytest.mark.parametrize("name", sorted(LARGE))
@pytest.mark.parametrize("precision", [L.IBB_FP64, L.IBB_FP32_REFINED])
def test_group_equals_solo(name, precision):
    from paper_1302_3663_amd import ibmg
    case = LARGE[name]()
    # launched passes on every level; two cycles, converged or not
    case["params"] = dict(case["params"], wg_coarse_max=-1, max_cycles=2, max_levels=3, rtol=1e-300)
    print("case", name, "precision", precision, flush=True)
    out = []
    for grouped in (False, True):
        ctx = ibmg.from_case(case, precision=precision, inner_cycles=2)
        g = ibmg.Group([ctx]) if grouped else None
        (g or ctx).projection_step(check=False)
        u, p = ctx.get_state()
        out.append((host(u), host(p)))
        if g:
            g.close()
        ctx.close()
    for a, b in zip(*out):
        assert np.all(np.isfinite(a)) and np.array_equal(a, b)
