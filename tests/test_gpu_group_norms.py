"""A member's residual norms in a group are those of its own solves, bit for
bit, also where the norm is summed by rows (2^20 points a component and more),
beside a small member; and on a 3D grid large enough for every pass by rows
(2^21 points) the fields are."""
import numpy as np
import pytest

from paper_1302_3663_amd import _lib as L
from paper_1302_3663_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


# just below 2^20 points a component and just above, walls and open ends; 3D with remainders of waves and rounds
# (periodic extents even on every level: an odd one puts two neighbours into one colour, and the passes of a group
# then depend on timing)
GRIDS = {
    "2d_1024x1022": lambda: synth.tiny_2d(nx=1024, ny=1022),
    "2d_inout_1040x1024": lambda: synth.tiny_2d(nx=1040, ny=1024, inout=True),
    "3d_128x128x144": lambda: synth.tiny_3d(n=(128, 128, 144)),
    "3d_periodic_160x112x128": lambda: synth.tiny_3d(n=(160, 112, 128), periodic_z=True, periodic_x=True),
}


@pytest.mark.parametrize("name", sorted(GRIDS))
@pytest.mark.parametrize("precision", [L.IBB_FP64, L.IBB_FP32_REFINED])
def test_norms_of_a_large_member(name, precision):
    from paper_1302_3663_amd import ibmg
    print("case", name, "precision", precision, flush=True)
    out = []
    for grouped in (False, True):
        case = GRIDS[name]()
        # steps of one cycle each: sums in another order agree to the last bit most of the time, but not always
        case["params"] = dict(case["params"], max_cycles=1, max_levels=4, rtol=1e-300)
        ctx = ibmg.from_case(case, precision=precision, inner_cycles=1)
        small = ibmg.from_case(synth.tiny_2d(), precision=precision, inner_cycles=1)
        g = ibmg.Group([small, ctx]) if grouped else None
        norms = []
        for _ in range(12):
            s = g.projection_step(check=False)[1] if grouped else ctx.projection_step(check=False)
            norms += [s["relres_u"], s["relres_p"]]
        u, p = ctx.get_state()
        out.append((host(u), host(p), norms))
        if grouped:
            g.close()
        ctx.close()
        small.close()
    for a, b in zip(out[0][:2], out[1][:2]):
        assert np.all(np.isfinite(a)) and np.array_equal(a, b)
    assert out[0][2] == out[1][2], (out[0][2], out[1][2])
