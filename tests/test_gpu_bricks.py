"""The levels of a V-cycle run as bricks (one launch of many workgroups that
exchange the surfaces of their boxes) take exactly the passes of the launched
kernels: iterates agree bit for bit with the same context's launched passes,
on boxes that are whole and cut short, along walls, open and periodic axes, in
both precisions and for both systems.  A launch whose workgroups do not all
start in time runs on one of them, with the same bits."""
import ctypes

import numpy as np
import pytest

from paper_1302_3663_amd import _lib as L
from paper_1302_3663_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda:0").contiguous()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def control(ctx, on=1, limit=-1):
    """First brick level per system (-1: none) and the launches that ran on one workgroup."""
    ctx._solver_scratch()
    first, solo = (ctypes.c_int * 2)(), ctypes.c_int()
    fn = ctx.lib.ibmg_bricks_control
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_longlong, ctypes.POINTER(ctypes.c_int),
                   ctypes.POINTER(ctypes.c_int)]
    assert fn(ctx.ctx, on, limit, first, ctypes.byref(solo)) == 0
    return tuple(first), solo.value


CASES = {
    "2d_channel": lambda: synth.channel_2d(seed=1),
    "2d_inout": lambda: synth.tiny_2d(nx=48, ny=16, inout=True),
    "2d_wide": lambda: synth.channel_2d(seed=1, nx=40, ny=96),
    "3d_smallest": lambda: synth.tiny_3d(),
    "3d_tube": lambda: synth.tiny_3d(n=(32, 16, 32)),
    "3d_uneven": lambda: synth.tiny_3d(n=(24, 24, 40)),
    "3d_periodic_z": lambda: synth.tiny_3d(n=(16, 32, 32), periodic_z=True),
    "3d_periodic_xz": lambda: synth.tiny_3d(n=(16, 16, 32), periodic_z=True, periodic_x=True),
    "3d_tube_64": lambda: synth.tube_3d(seed=2, n=(64, 64, 64), eta=200),
}


def run(case, precision, on, limit=-1, inner=3, **params):
    from paper_1302_3663_amd import ibmg
    c = dict(case, params=dict(case["params"], **params))
    ctx = ibmg.from_case(c, precision=precision, inner_cycles=inner)
    first, _ = control(ctx, on, limit)
    rng = np.random.default_rng(7)
    out = []
    for vel, n in ((1, ctx.n_face), (0, ctx.n_cell)):
        b = rng.standard_normal(n)
        x0 = case["u0"] if vel else np.zeros(n)
        for cycles in (1, 3):
            x, _ = ctx.mg_solve(vel, dev(b), dev(x0), exact=cycles)
            out.append(host(x))
    s = ctx.projection_step(check=False)
    u, p = ctx.get_state()
    out += [host(u), host(p)]
    _, solo = control(ctx, on, limit)
    ctx.close()
    return out, (s["cycles_u"], s["cycles_p"]), first, solo


def same(a, b):
    assert all(np.all(np.isfinite(x)) for x in a)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("precision", [L.IBB_FP64, L.IBB_FP32_REFINED])
def test_bricks_match_launched(name, precision):
    print("case", name, "precision", precision, flush=True)
    case = CASES[name]()
    ref, cyc_ref, _, _ = run(case, precision, 0)
    got, cyc, first, solo = run(case, precision, 1)
    assert first[0] >= 0 and first[1] >= 0 and solo == 0
    assert cyc == cyc_ref
    same(got, ref)


@pytest.mark.parametrize("params", [dict(nu1=1, nu2=3), dict(nu1=3, nu2=1), dict(decoupled=1, mu_max=1.0),
                                    dict(krylov_restart=3), dict(gamma=[1.0, 0.7] + [1.0] * 14)])
@pytest.mark.parametrize("precision", [L.IBB_FP64, L.IBB_FP32_REFINED])
def test_bricks_options(params, precision):
    print("params", params, "precision", precision, flush=True)
    case = CASES["3d_tube"]()
    ref, cyc_ref, _, _ = run(case, precision, 0, **params)
    got, cyc, first, _ = run(case, precision, 1, **params)
    assert first == (0, 0) and cyc == cyc_ref
    same(got, ref)


@pytest.mark.parametrize("name", ["2d_channel", "3d_uneven", "3d_periodic_xz"])
@pytest.mark.parametrize("precision", [L.IBB_FP64, L.IBB_FP32_REFINED])
def test_bricks_on_one_workgroup(name, precision):
    """No time to wait for the others: the first workgroup of a launch that
    is not its last runs the cycle by itself, and the next launches too."""
    print("case", name, "precision", precision, flush=True)
    case = CASES[name]()
    ref, cyc_ref, _, _ = run(case, precision, 0)
    got, cyc, _, solo = run(case, precision, 1, limit=0)
    assert solo > 0 and cyc == cyc_ref
    same(got, ref)


def test_bricks_beside_another_solve():
    """While another context solves, iterations run pass by pass: two threads on two streams, same bits, and no
    launch is left waiting for its workgroups."""
    import threading

    from paper_1302_3663_amd import ibmg
    case = CASES["3d_tube"]()
    ref, _, _, _ = run(case, L.IBB_FP64, 0)
    rng = np.random.default_rng(7)
    ctx0 = ibmg.from_case(case)
    b = dev(rng.standard_normal(ctx0.n_face))
    x0 = dev(case["u0"])
    ctx0.close()
    got = [None, None]

    def work(i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            ctx = ibmg.from_case(case)
            for _ in range(5):
                x, _ = ctx.mg_solve(1, b, x0, exact=3)
            got[i] = (host(x), control(ctx)[1])
            ctx.close()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for x, solo in got:
        assert solo == 0 and np.array_equal(x, ref[1])


def test_without_solver_scratch():
    """Without the scratch every pass is launched; set between two solves, bricks take over, with the same bits."""
    from paper_1302_3663_amd import ibmg
    case = CASES["3d_tube"]()
    ref, _, _, _ = run(case, L.IBB_FP64, 0)
    ctx = ibmg.from_case(case)
    b = dev(np.random.default_rng(7).standard_normal(ctx.n_face))
    ctx.scratch = torch.empty(0, device="cuda:0")
    x, _ = ctx.mg_solve(1, b, dev(case["u0"]), exact=3)
    assert np.array_equal(host(x), ref[1])
    few = torch.empty(1024, dtype=torch.uint8, device="cuda:0")
    assert ctx.lib.ibb_set_solver_scratch(ctx.ctx, few.data_ptr(), 1024) != 0
    ctx.scratch = None
    assert control(ctx)[0] == (0, 0)
    assert ctx.lib.ibb_set_solver_scratch(ctx.ctx, ctx.scratch.data_ptr(), ctx.scratch.numel()) != 0
    x, _ = ctx.mg_solve(1, b, dev(case["u0"]), exact=3)
    assert np.array_equal(host(x), ref[1])
    ctx.close()
