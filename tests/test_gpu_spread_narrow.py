"""Lattices of more than 65536 points with a narrow periodic axis, where a box
of points looks at every bin of the axis and a point only at some: the nodes
are added up in the order of the spread without a context, bit for bit."""
import numpy as np
import pytest

from paper_1302_3663_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda:0").contiguous()


@pytest.mark.parametrize("n,width_h", [((16, 66, 66), 2.6),    # 6 bins along x
                                       ((16, 66, 66), 3.2),    # 5, the fewest that a point sees in part
                                       ((16, 66, 66), 4.0),    # 4: every point sees all
                                       ((24, 66, 66), 2.0),    # 12: one box and the bins around it
                                       ((32, 66, 40), 2.6),    # 12 and 15, neither whole
                                       ((66, 66, 16), 2.0)])   # 8 along z, where boxes are two points deep
def test_order_of_nodes(n, width_h):
    from paper_1302_3663_amd import ibmg
    print("grid", n, "width", width_h, flush=True)
    p = dict(synth.tiny_3d(n=n, periodic_z=True, periodic_x=True)["params"])
    h = p["h"]
    p["omega"] = h
    L = np.array([p["n"][d] * h for d in range(3)])[:, None]
    rng = np.random.default_rng(9)
    # few enough for a table to have room, close together along the long axes and all along the short ones
    X = rng.random((3, 1200)) * L
    for d in range(3):
        if n[d] > 40:
            X[d] = 20 * h + rng.random(1200) * 14 * h
    F = rng.standard_normal(X.shape)
    ctx = ibmg.Context(p, X.shape[1], 1)
    got = ctx.spread(width_h * h, dev(X), dev(F))
    want = ibmg.spread_static(p, width_h * h, dev(X), dev(F))[0]
    torch.cuda.synchronize()
    print("largest difference", float((got - want).abs().max()), "of", float(want.abs().max()), flush=True)
    assert bool(torch.isfinite(got).all()) and torch.equal(got, want)
    ctx.close()
