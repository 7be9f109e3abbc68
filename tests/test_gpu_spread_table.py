"""Lattices of more than 65536 points are spread through a table of the nodes'
factors, a wave to a box of points: the same bits as the spread without a
context, which works out every factor at every point."""
import numpy as np
import pytest

from paper_1302_3663_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda:0").contiguous()


# remainders of the boxes (8 x 4 x 2, 8 x 8) along every axis, every kind of end
GRIDS = {
    "2d_260x254": lambda: synth.tiny_2d(nx=260, ny=254),
    "2d_inout_1030x66": lambda: synth.tiny_2d(nx=1030, ny=66, inout=True),
    "3d_46x38x42": lambda: synth.tiny_3d(n=(46, 38, 42)),
    "3d_periodic_64x32x40": lambda: synth.tiny_3d(n=(64, 32, 40), periodic_z=True, periodic_x=True),
}


@pytest.mark.parametrize("name", sorted(GRIDS))
@pytest.mark.parametrize("kernel", [0, 1])
@pytest.mark.parametrize("width_h", [1.0, 2.6])
def test_table_matches_direct(name, kernel, width_h):
    from paper_1302_3663_amd import ibmg
    p = dict(GRIDS[name]()["params"], kernel=kernel)
    D, h = p["dim"], p["h"]
    p["omega"] = h
    L = np.array([p["n"][d] * h for d in range(D)])[:, None]
    rng = np.random.default_rng(5)
    spread = rng.random((D, 500)) * 1.1 * L - 0.05 * L          # over the domain and a little beyond
    dense = 0.3 * L + 3 * h * rng.random((D, 700))              # many nodes to a bin
    ends = np.where(rng.random((D, 64)) < 0.5, 0.0, L)          # on the ends of the axes
    lost = np.full((D, 2), np.nan)
    lost[:, 1] = 1e12
    X = np.concatenate([spread, dense, ends, lost], axis=1)
    if any(p["axis_bc"][d] == 0 for d in range(D)):
        X = X[:, :-2]                                           # a periodic axis wraps every node
    F = rng.standard_normal(X.shape)
    print("grid", name, "kernel", kernel, "width", width_h, flush=True)
    ctx = ibmg.Context(p, X.shape[1], 1)
    got = ctx.spread(width_h * h, dev(X), dev(F))
    want = ibmg.spread_static(p, width_h * h, dev(X), dev(F))[0]
    torch.cuda.synchronize()
    print("largest difference", float((got - want).abs().max()), "of", float(want.abs().max()), flush=True)
    assert bool(torch.isfinite(got).all()) and torch.equal(got, want)
    # the table lies in memory of the pressure solve, which follows unharmed
    ctx.set_nodes(dev(dense))
    ctx.update_coefficients()
    b = dev(rng.standard_normal(ctx.n_cell))
    x0 = torch.zeros_like(b)
    first, _ = ctx.mg_solve(0, b, x0, exact=2)
    ctx.spread(width_h * h, dev(X), dev(F))
    again, _ = ctx.mg_solve(0, b, x0, exact=2)
    assert torch.equal(first, again) and bool(torch.isfinite(first).all())
    ctx.close()
