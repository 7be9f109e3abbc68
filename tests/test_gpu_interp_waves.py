"""Interpolation with a wave to a node (supports of up to 16 lattice indices an
axis) and with a block (wider ones) against the oracle, on both sides of the
rule, at every kind of end of an axis."""
import numpy as np
import pytest

import oracle as O
from paper_1302_3663_amd import synth

from parity import rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda:0").contiguous()


GRIDS = {
    "2d": lambda: synth.tiny_2d(nx=34, ny=18),
    "2d_inout": lambda: synth.tiny_2d(nx=30, ny=22, inout=True),
    "3d": lambda: synth.tiny_3d(n=(18, 16, 20)),
    "3d_periodic": lambda: synth.tiny_3d(n=(16, 18, 32), periodic_z=True, periodic_x=True),
}


@pytest.mark.parametrize("name", sorted(GRIDS))
@pytest.mark.parametrize("kernel", [0, 1])
@pytest.mark.parametrize("width_h", [1.0, 1.3, 3.25, 3.3])
def test_interp_matches_oracle(name, kernel, width_h):
    from paper_1302_3663_amd import ibmg
    p = dict(GRIDS[name]()["params"], kernel=kernel)
    D, h = p["dim"], p["h"]
    p["omega"] = h
    L = np.array([p["n"][d] * h for d in range(D)])[:, None]
    rng = np.random.default_rng(11)
    ends = np.where(rng.random((D, 9)) < 0.5, 0.0, L)
    X = np.concatenate([rng.random((D, 70)) * L, ends, np.round(rng.random((D, 6)) * L / h) * h], axis=1)
    u = rng.standard_normal(sum(O.face_counts(p)))
    print("grid", name, "kernel", kernel, "width", width_h, flush=True)
    ctx = ibmg.Context(p, X.shape[1], 1)
    got = ctx.interp(width_h * h, dev(X), dev(u)).cpu().numpy()
    ctx.close()
    # a sum of up to 16^3 products of order one: 1e-12 as for the other transfers
    assert rel(got, O.interp_vec(p, width_h * h, X, u)) < 1e-12
