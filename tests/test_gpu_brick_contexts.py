"""Contexts of different sizes share the kernels of the bricks: one with small
windows that comes later takes nothing away from one with large windows, whose
graphs are captured anew afterwards and replay the same bits."""
import numpy as np
import pytest

from paper_1302_3663_amd import _lib as L
from paper_1302_3663_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [L.IBB_FP64, L.IBB_FP32_REFINED])
def test_small_context_between_solves_of_a_large_one(precision):
    from paper_1302_3663_amd import ibmg
    print("precision", precision, flush=True)
    rng = np.random.default_rng(11)

    def context(n):
        ctx = ibmg.from_case(synth.tube_3d(seed=2, n=n, eta=100), precision=precision, inner_cycles=2)
        b = torch.as_tensor(rng.standard_normal(ctx.n_face), device="cuda:0")
        return ctx, b, torch.zeros_like(b)

    large, b, x0 = context((64, 64, 64))
    p = torch.as_tensor(rng.standard_normal(large.n_cell), device="cuda:0")
    want, _ = large.mg_solve(1, b, x0, exact=2)
    small, bs, xs = context((16, 16, 32))
    small.mg_solve(1, bs, xs, exact=1)
    got, _ = large.mg_solve(1, b, x0, exact=2)             # replayed
    assert torch.equal(got, want)
    y, _ = large.mg_solve(0, p, torch.zeros_like(p), exact=2)   # captured after the small context came
    fresh, _, _ = context((64, 64, 64))
    again, _ = fresh.mg_solve(0, p, torch.zeros_like(p), exact=2)
    assert torch.equal(y, again) and bool(torch.isfinite(y).all())
    # launched pass by pass: the same bits
    plain, _, _ = context((64, 64, 64))
    plain.scratch = torch.empty(0, device="cuda:0")
    for which, rhs, res in ((1, b, want), (0, p, y)):
        z, _ = plain.mg_solve(which, rhs, torch.zeros_like(rhs), exact=2)
        assert torch.equal(z, res)
    for ctx in (large, small, fresh, plain):
        ctx.close()
